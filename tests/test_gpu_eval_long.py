"""Terms of 9 to 16 factors on the fast path (two records of half the factors
each) against the oracle: every factor count, next to shorter terms with and
without powers, with the total-degree and with an explicit start system; and the
equation groups a launch picks by itself give the bits of one group."""
import numpy as np
import pytest

import oracle
import paper_1505_00383_amd as ph
from paper_1505_00383_amd import synth
from tests.parity import TOL, scaled_error

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _system(rng, n, ks, power):
    eqs = []
    for i in range(n):
        eq = [(synth.unit_complex(rng), {int(v): 1 for v in rng.choice(n, size=k, replace=False)}) for k in ks]
        eq.append((synth.unit_complex(rng), {i: power, (i + 1) % n: 1}))
        eq.append((synth.unit_complex(rng), {}))
        eqs.append(eq)
    return synth.system_from_terms(n, eqs)


@pytest.mark.parametrize("n,ks,power", [(9, (9,), 1), (10, (10, 9, 3), 3), (12, (11, 12, 8), 2), (16, (13, 14, 15, 16), 1),
                                        (17, (16, 9, 17), 1), (18, (10,), 4)])
@pytest.mark.parametrize("L", [1, 2, 4])
@pytest.mark.parametrize("explicit", [False, True])
def test_long_terms_match_oracle(n, ks, power, L, explicit):
    rng = np.random.Generator(np.random.PCG64(31 * n + L))
    f = _system(rng, n, ks, power)
    g = _system(rng, n, ks[::-1], power) if explicit else None
    gamma = synth.unit_complex(rng)
    npts = 70
    x = synth.random_points(n, npts, L, rng, 0.8)
    t = rng.uniform(0, 1, npts)
    S = ph.System(f)
    G = ph.System(g) if explicit else None
    if explicit:
        ph.eval_prepare(S, L, start=G)
    import torch
    val, jac = ph.eval_jac(S, ph.to_soa(x), npts, L, torch.as_tensor(t).cuda(), gamma, start=G)
    only, _ = ph.eval_jac(S, ph.to_soa(x), npts, L, torch.as_tensor(t).cuda(), gamma, start=G, want_jac=False)
    ov, oj, sv, sj = oracle.eval_homotopy(f, L, x, t, gamma, start=g)
    ev = scaled_error(ph.from_soa(val, npts, (n, 2, L)), ov, sv)
    eo = scaled_error(ph.from_soa(only, npts, (n, 2, L)), ov, sv)
    ej = scaled_error(ph.from_soa(jac, npts, (n, n, 2, L)), oj, sj)
    print(f"[gpu] n={n} ks={ks} L={L} explicit={explicit} val {ev:.1e} values only {eo:.1e} jac {ej:.1e}", flush=True)
    assert max(ev, eo, ej) <= TOL[L]


@pytest.mark.parametrize("L", [1, 2, 4])
@pytest.mark.parametrize("npts", [1, 65, 700, 20001])
@pytest.mark.parametrize("n", [5, 12, 32])
def test_groups_chosen_give_the_bits_of_one_group(L, npts, n):
    import torch
    s = synth.eval_dense(seed=5, n=n, terms_per_eq=4, k=3)
    x, t = synth.torus_points(s, npts, L)
    S = ph.System(s)
    xs, tt = ph.to_soa(x), torch.as_tensor(t).cuda()
    a = ph.eval_jac(S, xs, npts, L, tt, synth.gamma_of(s))
    ph.eval_set_config(S, L, ph.EVAL_FAST, 1, 1)
    b = ph.eval_jac(S, xs, npts, L, tt, synth.gamma_of(s))
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
