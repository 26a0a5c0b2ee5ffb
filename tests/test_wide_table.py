"""The schedule of a wave over one path's terms (wide_table.cpp), built for the
host: every term is swept once, every partial and value is added once, in term
order, and an entry's partials of a chunk follow each other in one lane's list."""
import ctypes

import numpy as np
import pytest

from tests import host_cpp

SOURCE = r"""
#include "wide_table.cpp"
using namespace ph;
static ph::WideTable wt;
extern "C" int build(int n, const int *eq_off, const int *k, const int *fac_off, const unsigned *fac, int n_fac, int *sizes)
{
    std::vector<int32_t> eo(eq_off, eq_off + n + 1);
    std::vector<int4> td;
    std::vector<double> coef;
    for (int t = 0; t < eo[n]; ++t) {
        td.push_back(int4{k[t], fac_off[t], 0, 0});
        for (int c = 0; c < 8; ++c) coef.push_back(8 * t + c);
    }
    build_wide(n, eo, td, std::vector<uint32_t>(fac, fac + n_fac), coef, wt);
    sizes[0] = wt.rounds;
    sizes[1] = (int)wt.chunk.size();
    sizes[2] = (int)wt.list.size();
    return WIDE_ROUNDS;
}
extern "C" void tables(unsigned *meta, double *coef, int *chunk, unsigned *list)
{
    std::copy(wt.meta.begin(), wt.meta.end(), meta);
    std::copy(wt.coef.begin(), wt.coef.end(), coef);
    for (size_t c = 0; c < wt.chunk.size(); ++c) {
        chunk[3 * c] = wt.chunk[c].x;
        chunk[3 * c + 1] = wt.chunk[c].y;
        chunk[3 * c + 2] = wt.chunk[c].z;
    }
    for (size_t q = 0; q < wt.list.size(); ++q) {
        list[2 * q] = wt.list[q].x;
        list[2 * q + 1] = wt.list[q].y;
    }
}
"""
NONE, FIRST, LAST = 0xffffffff, 0x80000000, 0x40000000


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_cpp.load(tmp_path_factory, "wide_schedule", SOURCE)


@pytest.mark.parametrize("n,terms,kmax", [(1, 3, 1), (3, 6, 3), (4, 40, 4), (8, 24, 3), (8, 60, 8), (16, 20, 2), (17, 9, 5),
                                          (32, 14, 8), (5, 0, 2)])
def test_schedule(lib, n, terms, kmax):
    rng = np.random.default_rng(100 * n + terms)
    eqs = []
    for i in range(n):   # the order of the tables: by factors, then by extra powers
        eq = [sorted(((int(v), int(rng.integers(1, 4))) for v in rng.choice(n, size=min(n, int(rng.integers(0, kmax + 1))),
                                                                            replace=False)))
              for _ in range(int(rng.integers(0, terms + 1)))]
        eqs.append(sorted(eq, key=lambda t: (len(t), sum(e for _, e in t))))
    flat = [t for eq in eqs for t in eq]
    eq_of = [i for i, eq in enumerate(eqs) for _ in eq]
    off = np.cumsum([0] + [len(eq) for eq in eqs]).astype(np.int32)
    k = np.array([len(t) for t in flat] + [0], dtype=np.int32)
    fo = np.cumsum([0] + [len(t) for t in flat]).astype(np.int32)
    fac = np.array([v | (e << 16) for t in flat for v, e in t] + [0], dtype=np.uint32)
    sizes = (ctypes.c_int * 3)()
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    per = 64 * lib.build(n, p(off), p(k), p(fo), p(fac), len(fac), sizes)
    rounds, chunks, steps = sizes[0], sizes[1], sizes[2] // 64
    meta, coef = np.zeros(64 * rounds, np.uint32), np.zeros((rounds, 8, 64))
    chunk, lists = np.zeros((chunks, 3), np.int32), np.zeros((steps, 64, 2), np.uint32)
    lib.tables(p(meta), p(coef), p(chunk), p(lists))
    used = [q for q in range(64 * rounds) if meta[q] != NONE]
    assert used == list(range(len(flat)))
    term = [int(coef[q // 64, 0, q % 64]) // 8 for q in used]      # the term of slot q
    assert sorted(term) == used
    assert all(int(meta[q]) == len(flat[term[q]]) for q in used)
    np_ = max(4, 1 << (n - 1).bit_length())
    entries, values = {}, {}
    assert chunks == -(-len(flat) // per)
    for c, (first, length, gather) in enumerate(chunk):
        assert length % 4 == 0 and gather <= length
        seen = {}
        for lane in range(64):
            run = None
            for x, y in lists[first:first + length, lane]:
                if x != 0:
                    entry, slot, l = (int(x) >> 16) & 0x7ff, int(x) % per, (int(x) & 0xffff) // per
                    assert bool(x & FIRST) == (run is None) and (run is None or run == entry)
                    assert seen.setdefault(entry, lane) == lane
                    run = None if x & LAST else entry
                    t = term[c * per + slot]
                    assert entry == flat[t][l][0] * np_ + eq_of[t]
                    entries.setdefault(entry, []).append(t)
                if y != NONE:
                    t = term[c * per + int(y)]
                    assert eq_of[t] == lane // 2
                    values.setdefault(lane, []).append(t)
            assert run is None
            assert not lists[first + gather:first + length, lane, 0].any()
    for e, ts in entries.items():
        want = [t for t in range(len(flat)) for v, _ in flat[t] if v * np_ + eq_of[t] == e]
        assert ts == want
    for i in range(n):
        for lane in (2 * i, 2 * i + 1):
            assert values.get(lane, []) == [t for t in range(len(flat)) if eq_of[t] == i]
