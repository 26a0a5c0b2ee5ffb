"""Which tracker kernel a call takes (track_rule.hpp), built for the host: the line
between a wave per path and a lane per equation lies at a number of paths per
resident wave, times the ratio of the workgroups that the two kernels have
resident; fewer are where their LDS, the workgroups asked per CU or a bound on all
workgroups allow fewer."""
import ctypes

import numpy as np
import pytest

from tests import host_cpp

SOURCE = r"""
#include <cstring>
#include "track_rule.hpp"
using namespace ph;
extern "C" int rule(int nsys, const int *n, const int64_t *off, int kmax, int prec, int mixed, int lanes, int per_cu,
                    int blocks, int bounded, int *out)
{
    ph_track_opts o;
    std::memset(&o, 0, sizeof o);
    o.prec = prec;
    o.mixed = mixed;
    o.lanes_per_path = lanes;
    o.blocks_per_cu = per_cu;
    const LaneRule r = track_lane_rule(nsys, n, off, kmax, o, 256, blocks, bounded != 0);
    out[0] = r.wide;
    out[1] = r.lanes;
    return (int)track_wide_lds_bytes(prec, mixed, natural_lanes(n[0]), kmax);
}
"""


TUNE = r"""
extern "C" int tune(int nsys, const int *n, const int64_t *full, const int64_t *off, int kmax, int prec, int mixed,
                    int *out)
{
    ph_track_opts o;
    std::memset(&o, 0, sizeof o);
    o.prec = prec;
    o.mixed = mixed;
    o.rounds_per_launch = 32;
    int q = 0;
    for (const TuneCand &c : tune_candidates(nsys, n, full, off, kmax, o, 256, 0)) {
        const LaneRule whole = track_lane_rule(nsys, n, full, kmax, c.o, 256, 0, false);
        const LaneRule sample = track_lane_rule(nsys, n, off, kmax, c.o, 256, 0, false);
        const int row[8] = {c.o.schedule, c.o.blocks_per_cu, c.o.lanes_per_path, c.rule.wide, c.rule.lanes,
                            whole.wide == c.rule.wide && whole.lanes == c.rule.lanes, sample.wide,
                            (int)track_workgroups(nsys, n, off, c.rule)};
        for (int v : row) out[q++] = v;
    }
    return q / 8;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_cpp.load(tmp_path_factory, "track_rule", SOURCE + TUNE)


def _rule(lib, n, paths, kmax=2, prec=1, mixed=0, lanes=0, per_cu=0, blocks=0, bounded=0):
    ns = np.array(np.atleast_1d(n), dtype=np.int32)
    off = np.concatenate([[0], np.cumsum(np.atleast_1d(paths))]).astype(np.int64)
    out = (ctypes.c_int * 2)()
    lds = lib.rule(len(ns), ns.ctypes.data_as(ctypes.c_void_p), off.ctypes.data_as(ctypes.c_void_p), kmax, prec, mixed,
                   lanes, per_cu, blocks, bounded, out)
    return bool(out[0]), out[1], lds


# (n, factors, limbs, FP64 solves) -> workgroups per CU: wave per path, lane per equation
@pytest.mark.parametrize("n,kmax,prec,mixed,waves,other", [
    (3, 2, 1, 0, 8, 8), (8, 3, 2, 1, 8, 8), (16, 3, 2, 1, 8, 8), (8, 8, 4, 0, 2, 4), (8, 8, 2, 0, 4, 8), (16, 2, 4, 0, 3, 2),
    (16, 8, 4, 0, 1, 2), (16, 8, 2, 0, 3, 4), (24, 2, 2, 0, 3, 2), (32, 8, 4, 0, 1, 1), (32, 2, 1, 0, 6, 4)])
def test_line_lies_at_paths_per_resident_wave(lib, n, kmax, prec, mixed, waves, other):
    f = 1 if n <= 4 else (8 if n <= 8 else (11 if n <= 16 else 22))
    kw = dict(kmax=kmax, prec=prec, mixed=mixed)
    assert min(8, 160 * 1024 // _rule(lib, n, 1, **kw)[2]) == waves

    def on_line(w, o, **more):
        line = f * w * w // o
        return _rule(lib, n, line, **kw, **more)[0] and not _rule(lib, n, line + 1, **kw, **more)[0]

    assert on_line(256 * waves, 256 * other)
    for per_cu in (1, 2, 16):   # workgroups per CU as asked
        assert on_line(256 * min(waves, per_cu), 256 * min(other, per_cu), per_cu=per_cu)
    assert on_line(10, 10, blocks=10)
    line = f * 256 * waves * waves // other
    # a batch: the shares add up
    half = line // 2
    assert _rule(lib, [n, n], [half, half], **kw)[0] and not _rule(lib, [n, n], [half, half + 2], **kw)[0]


def test_lanes_asked_for_and_doubled_lanes(lib):
    for lanes in (4, 8, 16, 32):
        assert _rule(lib, 8, 10, lanes=lanes)[:2] == (False, lanes)
    # few paths whose history must fit the other kernel's buffer: twice the
    # natural lanes below one wave per SIMD, the natural count beyond
    assert _rule(lib, 8, 8191, bounded=1)[:2] == (False, 16)
    assert _rule(lib, 8, 8192, bounded=1)[:2] == (False, 0)
    assert _rule(lib, 32, 10, bounded=1)[:2] == (False, 0)
    assert _rule(lib, 3, 2049)[:2] == (False, 8)
    assert _rule(lib, 3, 16384)[:2] == (False, 0)
    # doubled lanes only where every path is resident with them
    assert _rule(lib, 8, 2048, kmax=8, prec=4, bounded=1)[:2] == (False, 16)
    assert _rule(lib, 8, 2049, kmax=8, prec=4, bounded=1)[:2] == (False, 0)


@pytest.mark.parametrize("n,full,prec,mixed", [([8], [200000], 2, 1), ([3, 8, 16], [1000, 40000, 160000], 2, 1),
                                               ([8], [6561], 2, 1), ([16], [65536], 4, 0), ([3], [8], 1, 0),
                                               ([24], [300000], 1, 0)])
def test_autotuner_times_the_kernel_of_the_whole_run(lib, n, full, prec, mixed):
    ns = np.array(n, dtype=np.int32)
    total = sum(full)
    frac = min(1.0, 16384 / total)
    whole = np.concatenate([[0], np.cumsum(full)]).astype(np.int64)
    off = np.concatenate([[0], np.cumsum([max(1, int(np.ceil(f * frac))) for f in full])]).astype(np.int64)
    out = (ctypes.c_int * 4096)()
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    rows = lib.tune(len(ns), p(ns), p(whole), p(off), 3, prec, mixed, out)
    cands = np.array(out[:8 * rows]).reshape(rows, 8)
    sched, per_cu, lanes, wide, got, same, sample_wide, need = cands.T
    assert np.all(same == 1)                     # a candidate runs as the whole run would
    if total > 100000:                           # ... where the sample by itself would not
        assert np.all(wide == 0) and np.any(sample_wide[lanes == 0] == 1)
    # the natural count is among them, as 0 or by name
    assert np.any((wide == 0) & ((got == 0) | (got == 4)))
    assert set(lanes) <= {0, 4, 8, 16, 32} and np.all(per_cu >= 1) and np.all(per_cu <= 16)
    # no two persistent candidates launch the same grid on the sample
    grids = [(a, b, min(c, 256 * d)) for a, b, c, d, e in zip(wide, got, need, per_cu, sched) if e == 0]
    assert len(set(grids)) == len(grids)
