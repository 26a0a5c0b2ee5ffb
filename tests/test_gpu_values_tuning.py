"""Tuning of calls without a Jacobian (ph_eval_autotune with jac NULL; the Python
binding always passes one): the choice is theirs alone, in the handle and in the
cache file."""
import ctypes

import numpy as np
import pytest

import paper_1505_00383_amd as ph
from paper_1505_00383_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _tune_values(S, xs, npts, L, gamma):
    import torch
    val = torch.empty((S.n_eq * 2 * L, npts), dtype=torch.float64, device="cuda")
    g = (ctypes.c_double * 2)(gamma.real, gamma.imag)
    ms = ctypes.c_double(0.0)
    rc = ph.load_library().ph_eval_autotune(S.handle, None, g, L, npts, None, ctypes.c_void_p(xs.data_ptr()), npts,
                                            ctypes.c_void_p(val.data_ptr()), None, None, ctypes.byref(ms))
    assert rc == 0 and ms.value > 0
    return val


@pytest.mark.parametrize("long", [True, False])
@pytest.mark.parametrize("L", [1, 2, 4])
def test_values_choice_leaves_jacobian_calls_alone(L, long, tmp_path, monkeypatch):
    import torch
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("PH_AUTOTUNE_CACHE", str(cache))
    s = synth.SHAPED["cyclic10"]() if long else synth.eval_dense(seed=3, n=9, terms_per_eq=6, k=4)
    npts = 500
    x, _ = synth.torus_points(s, npts, L, np.random.default_rng(L))
    xs = ph.to_soa(x)
    gamma = synth.gamma_of(s)
    S = ph.System(s)
    v0, j0 = ph.eval_jac(S, xs, npts, L)
    w0, _ = ph.eval_jac(S, xs, npts, L, want_jac=False)
    tuned = _tune_values(S, xs, npts, L, gamma)
    line = cache.read_text().split()
    print(f"[gpu] L={L} long={long} values -> {line}", flush=True)
    assert torch.equal(tuned, w0) or L > 1   # double: one kernel, the bits of any tiling
    assert line[0] == "values" and line[4] in ("0", "1") and (L > 1 or line[4] == "1")
    assert ph.eval_get_config(S, L) == tuple(int(q) for q in line[4:7])
    for T in (S, ph.System(s)):              # this handle, and one that reads the file
        v1, j1 = ph.eval_jac(T, xs, npts, L)
        assert torch.equal(v1, v0) and torch.equal(j1, j0)
        w1, _ = ph.eval_jac(T, xs, npts, L, want_jac=False)
        assert torch.equal(w1, w0) or line[4] == "1"
    # a setting made by hand holds for both kinds of calls
    ph.eval_set_config(S, L, ph.EVAL_GENERAL, 2, 1)
    assert ph.eval_get_config(S, L) == (ph.EVAL_GENERAL, 2, 1)
    g1, _ = ph.eval_jac(S, xs, npts, L)
    g2, _ = ph.eval_jac(S, xs, npts, L, want_jac=False)
    assert (g1 - g2).abs().max() < 1e-12
