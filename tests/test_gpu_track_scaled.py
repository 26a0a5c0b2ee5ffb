"""Both systems of a homotopy multiplied by a power of two: J and H scale by it,
the Newton corrections do not change by a bit, so endpoints, verdicts and step
counts are those of the unscaled homotopy, in both tracker kernels, where squares
of the Jacobian's entries are near the ends of the exponent range."""
import numpy as np
import pytest

import paper_1505_00383_amd as ph
from paper_1505_00383_amd import synth
from tests.starts import diagonal_roots, diagonal_start

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _times(s, e):
    eqs = [[(complex(c.real * 2.0 ** e, c.imag * 2.0 ** e), dict(m)) for c, m in s.terms(i)] for i in range(s.n_eq)]
    return synth.system_from_terms(s.n_var, eqs)


@pytest.mark.parametrize("n,lanes", [(3, 0), (3, 4), (12, 0), (17, 0), (17, 32)])
@pytest.mark.parametrize("L,mixed", [(1, 0), (2, 1), (2, 0), (4, 1), (4, 0)])
def test_scaled_homotopy_bitwise(n, lanes, L, mixed):
    rng = np.random.Generator(np.random.PCG64(n))
    f = synth.system_from_terms(n, [synth._equation_with_anchor(rng, list(range(n)), i, 2, 8) for i in range(n)])
    deg = [2] * n
    g, a, b = diagonal_start(rng, deg)
    gamma = synth.unit_complex(rng)
    paths = [0, 1, 5]
    x0 = ph.to_soa(diagonal_roots(a, b, deg, L, paths))
    kw = dict(prec=L, mixed=mixed, lanes_per_path=lanes)
    if n > 3 and L == 4 and not mixed:
        kw["max_steps"] = 6
    runs = {}
    for e in (0, -480, 480):
        print(f"[gpu] n={n} lanes={lanes} L={L} mixed={mixed} scale 2^{e}", flush=True)
        S, G = ph.System(_times(f, e)), ph.System(_times(g, e))
        ph.eval_prepare(S, L, start=G)
        runs[e] = ph.track(S, gamma, len(paths), ph.track_opts(**kw), x_start=x0, start=G)
    if "max_steps" not in kw:
        assert np.all(runs[0]["status"] == 1)
    for e in (-480, 480):
        for k in ("status", "reason", "steps"):
            assert np.array_equal(runs[e][k], runs[0][k]), (e, k)
        assert np.array_equal(runs[e]["x_end"].cpu().numpy(), runs[0]["x_end"].cpu().numpy()), e
