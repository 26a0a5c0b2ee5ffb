"""The tracker's sum of term values (ph_accum.hpp), built for the host, against
exact rational sums: no further off than the chain of normalised additions that
the evaluation kernels and the oracle use, whatever the number of terms."""
import ctypes
from fractions import Fraction

import numpy as np
import pytest

from tests import host_cpp

SOURCE = r"""
#include "ph_accum.hpp"
using namespace ph;
template <int L> static void sums(int n, const double *u, double *acc, double *chain)
{
    Acc<L> s = acc_zero<L>();
    R<L> c = r_zero<L>();
    for (int i = 0; i < n; ++i) {
        R<L> x;
        for (int l = 0; l < L; ++l) x.v[l] = u[i * L + l];
        acc_add<L>(s, x);
        c = r_add<L>(c, x);
    }
    const R<L> v = acc_value<L>(s);
    for (int l = 0; l < L; ++l) { acc[l] = v.v[l]; chain[l] = c.v[l]; }
}
extern "C" void sums2(int n, const double *u, double *a, double *c) { sums<2>(n, u, a, c); }
extern "C" void sums4(int n, const double *u, double *a, double *c) { sums<4>(n, u, a, c); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_cpp.load(tmp_path_factory, "accum", SOURCE)


def _values(rng, n, L, spread):
    u = np.zeros((n, L))
    u[:, 0] = rng.normal(size=n) * 10.0 ** rng.uniform(-spread, spread, n)
    for l in range(1, L):
        u[:, l] = (rng.random(n) - 0.5) * np.spacing(np.abs(u[:, l - 1]))
    return u


def _sums(lib, u):
    n, L = u.shape
    a, c = np.zeros(L), np.zeros(L)
    p = lambda x: x.ctypes.data_as(ctypes.c_void_p)
    getattr(lib, f"sums{L}")(n, p(u), p(a), p(c))
    exact = sum((Fraction(x) for x in u.ravel()), Fraction(0))
    err = lambda v: abs(sum((Fraction(x) for x in v), Fraction(0)) - exact)
    return a, float(err(a)), float(err(c)), exact


@pytest.mark.parametrize("L", [2, 4])
@pytest.mark.parametrize("n", [1, 2, 8, 22, 64, 130, 1000])
def test_sum_is_no_further_off_than_normalised_additions(lib, L, n):
    rng = np.random.default_rng(17 * n + L)
    ea, ec = [], []
    for _ in range(60):
        u = _values(rng, n, L, 0.3)
        a, x, y, _ = _sums(lib, u)
        ea.append(x)
        ec.append(y)
        assert np.all(np.abs(a[1:]) <= np.spacing(np.abs(a[:-1])))  # limbs in order
    print(f"L={L} n={n}: median {np.median(ea):.1e} ({np.median(ec):.1e}), largest {max(ea):.1e} ({max(ec):.1e})")
    assert np.median(ea) <= np.median(ec) and max(ea) <= max(ec)


@pytest.mark.parametrize("L", [2, 4])
def test_cancelling_sums(lib, L):
    """Values that cancel to nothing or to a small tail.  Quad double: nothing is
    lost before the guard limb.  Double double: an addition may lose one rounding
    of each of two terms of the second limb's order, 2^-106 of the partial sum
    each."""
    rng = np.random.default_rng(L)
    for n in (3, 17, 64):
        u = _values(rng, n, L, 3.0)
        size = np.abs(u[:, 0]).sum()
        lost = n * size * 2.0 ** (-53 * (L + 1) + 4) if L == 4 else 2 * (2 * n + 1) * size * 2.0 ** -106
        for tail in (0.0, 1e-20, 1e-40, 1e-60):
            w = np.concatenate([u, -u[::-1], np.zeros((1, L))])
            w[-1, 0] = tail
            a, x, _, exact = _sums(lib, w)
            assert x <= max(2.0 ** (-53 * L + 1) * abs(float(exact)), lost)
