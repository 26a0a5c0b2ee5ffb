"""The tracker kernel that gives a whole wave to one path (lanes_per_path = 0
with few paths) against the kernel with one lane per equation (the natural lane
count asked for): every sum is made of the same additions in the same order, so
endpoints, verdicts and step counts agree bit for bit.  Sizes: the edges of the
lane counts (4, 8, 16, 32 rows), one and several chunks of terms, terms of up to
eight factors, columns in registers and in LDS, both schedules."""
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


def _same(a, b):
    assert np.array_equal(a["x_end"].cpu().numpy(), b["x_end"].cpu().numpy(), equal_nan=True)
    for k in ("status", "reason", "steps"):
        assert np.array_equal(a[k], b[k])
    assert {k: v for k, v in a["report"].items() if k != "seconds"} == \
        {k: v for k, v in b["report"].items() if k != "seconds"}


def _natural(n):
    return max(4, 1 << (n - 1).bit_length())


@pytest.mark.parametrize("n,d,terms", [(1, 3, 3), (2, 2, 4), (4, 3, 20), (5, 2, 9), (8, 3, 20), (9, 2, 12),
                                       (16, 2, 32), (17, 2, 10), (32, 2, 8)])
@pytest.mark.parametrize("L,mixed,order,schedule", [(1, 0, 1, 0), (2, 1, 4, 1), (2, 0, 1, 0), (4, 1, 1, 0), (4, 0, 2, 1)])
def test_wave_per_path_bitwise(n, d, terms, L, mixed, order, schedule):
    rng = np.random.Generator(np.random.PCG64(100 * n + L))
    eqs = [synth._equation_with_anchor(rng, list(range(n)), i, d, terms) for i in range(n)]
    gamma = synth.unit_complex(rng)
    S = ph.System(synth.system_from_terms(n, eqs))
    paths = min(d ** n, 24 if L < 4 or mixed else 3)
    kw = dict(prec=L, mixed=mixed, predictor_order=order, schedule=schedule)
    if n > 16 and L == 4 and not mixed:
        kw["max_steps"] = 5
    print(f"[gpu] n={n} d={d} L={L} mixed={mixed} order={order} schedule={schedule} paths={paths}", flush=True)
    _same(ph.track(S, gamma, paths, ph.track_opts(**kw)),
          ph.track(S, gamma, paths, ph.track_opts(lanes_per_path=_natural(n), **kw)))


@pytest.mark.parametrize("k", [3, 4, 5, 8])
@pytest.mark.parametrize("L,mixed", [(1, 1), (2, 1), (4, 1)])
def test_wave_per_path_long_terms_and_explicit_start(k, L, mixed):
    n = 8
    rng = np.random.Generator(np.random.PCG64(7 + k))
    eqs = []
    for i in range(n):
        eq = [(synth.unit_complex(rng), {i: k}), (synth.unit_complex(rng), {})]
        for q in range(1, k + 1):
            vs = rng.choice(n, size=q, replace=False)
            eq.append((0.3 * synth.unit_complex(rng), {int(v): 1 for v in vs}))
        eqs.append(eq)
    f = synth.system_from_terms(n, eqs)
    g, a, b = diagonal_start(rng, [k] * n)
    S, G = ph.System(f), ph.System(g)
    import torch
    paths = [0, 1, k, k * k + 1, k ** 5 - 1]
    x0 = ph.to_soa(diagonal_roots(a, b, [k] * n, L, paths))
    gamma = synth.unit_complex(rng)
    print(f"[gpu] k={k} L={L} mixed={mixed}", flush=True)
    kw = dict(prec=L, mixed=mixed)
    r = ph.track(S, gamma, len(paths), ph.track_opts(**kw), x_start=x0, start=G)
    _same(r, ph.track(S, gamma, len(paths), ph.track_opts(lanes_per_path=8, **kw), x_start=x0, start=G))
    assert np.all(r["status"] == 1)


def test_wave_per_path_mixed_classes_and_failures():
    """A batch of systems of 4, 8, 16 and 32 rows; paths that fail (a step
    budget, a divergence bound, a start point that is not finite)."""
    rng = np.random.Generator(np.random.PCG64(3))
    systems, gammas, lists = [], [], []
    for n in (3, 8, 13, 32):
        eqs = [synth._equation_with_anchor(rng, list(range(n)), i, 2, 7) for i in range(n)]
        systems.append(ph.System(synth.system_from_terms(n, eqs)))
        gammas.append(synth.unit_complex(rng))
        lists.append(np.arange(min(2 ** n, 20)))
    for kw in (dict(), dict(max_steps=20), dict(diverge_norm=1.05), dict(schedule=1, predictor_order=3)):
        print(f"[gpu] {kw}", flush=True)
        wide = ph.track_batch(systems, gammas, lists, ph.track_opts(prec=2, mixed=1, **kw))
        for s in range(4):
            n = systems[s].n_var
            one = ph.track(systems[s], gammas[s], len(lists[s]),
                           ph.track_opts(prec=2, mixed=1, lanes_per_path=_natural(n), **kw))
            a, b = int(wide["path_off"][s]), int(wide["path_off"][s + 1])
            assert np.array_equal(wide["x_end"][:n * 4, a:b].cpu().numpy(), one["x_end"].cpu().numpy(), equal_nan=True)
            assert np.array_equal(wide["reason"][a:b], one["reason"])
            assert np.array_equal(wide["steps"][a:b], one["steps"])
    x0 = ph.start_solutions(systems[1], 1, 0, 6)
    x0[3, 2] = float("nan")
    x0[0, 4] = float("inf")
    r = ph.track(systems[1], gammas[1], 6, ph.track_opts(prec=1), x_start=x0)
    _same(r, ph.track(systems[1], gammas[1], 6, ph.track_opts(prec=1, lanes_per_path=8), x_start=x0))
    assert r["status"][2] == -1 and r["status"][4] == -1
