"""The waves and groups that ph_eval_set_config names hold for the values kernels
too: one wave for 32 equations takes many times as long as the default launch,
with the same values."""
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
@pytest.mark.parametrize("kernel", [ph.EVAL_AUTO, ph.EVAL_FAST])
def test_named_tiling_is_taken(L, kernel):
    import torch
    s = synth.eval_dense()
    npts = 64
    x, t = synth.torus_points(s, npts, L)
    xs, tt = ph.to_soa(x), torch.as_tensor(t).cuda()
    gamma = synth.gamma_of(s)
    S = ph.System(s)

    def run():
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        for e in ev:
            v, _ = ph.eval_jac(S, xs, npts, L, tt, gamma, want_jac=False)
            e.record()
        torch.cuda.synchronize()
        return v, ev[0].elapsed_time(ev[1])

    v0, t0 = run()
    for W, G in ((1, 1), (3, 2), (0, 4), (2, 0), (8, 4)):
        ph.eval_set_config(S, L, kernel, W, G)
        v, ms = run()
        print(f"[gpu] L={L} kernel={kernel} waves={W} groups={G}: {ms:.3f} ms, default {t0:.3f} ms", flush=True)
        assert torch.equal(v, v0)
        if (W, G) == (1, 1):
            assert ms > 4 * t0
