"""ph_eval_autotune times a kernel's own choice of a tiling as well: five equations
at one tile of points run in one round of waves only with a group count that the
configurations by number do not have."""
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


@pytest.mark.parametrize("L", [2, 4])
def test_own_tiling_is_tried(L):
    import torch
    s = synth.eval_dense(seed=9, n=5, terms_per_eq=64, k=5)
    npts = 32
    x, t = synth.torus_points(s, npts, L)
    xs, tt = ph.to_soa(x), torch.as_tensor(t).cuda()
    gamma = synth.gamma_of(s)
    S = ph.System(s)
    v0, j0 = ph.eval_jac(S, xs, npts, L, tt, gamma)
    ms = ph.eval_autotune(S, xs, npts, L, tt, gamma)
    print(f"[gpu] L={L} {ms:.4f} ms {ph.eval_get_config(S, L)}", flush=True)
    assert ph.eval_get_config(S, L) == (ph.EVAL_FAST, 0, 0)
    v1, j1 = ph.eval_jac(S, xs, npts, L, tt, gamma)
    assert torch.equal(v0, v1) and torch.equal(j0, j1)
