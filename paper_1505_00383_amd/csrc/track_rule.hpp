// track_rule.hpp -- host-side choice of the tracker kernel and its lanes per path.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include "../../include/ph.h"
#include "ph_internal.hpp"

namespace ph {

// Bytes of LDS of one workgroup.  A wave per path: the arrays of run_wide
// (ph_track_wide.hpp), partials for kmax factors a term.
inline size_t track_wide_lds_bytes(int prec, int mixed, int np_max, int kmax)
{
    const size_t l2 = 2 * (size_t)prec, ls2 = 2 * (size_t)(mixed ? 1 : prec), np = np_max;
    return (np * l2 + (np + 1) * np * ls2 + np * ls2 + 64 * (size_t)WIDE_ROUNDS * (l2 + kmax * ls2)) * sizeof(double);
}

inline size_t track_lds_bytes(int prec, int mixed, int np_max)
{
    const int ls = mixed ? 1 : prec;
    const size_t w = (size_t)(64 / np_max) * (np_max + 1) * np_max * 2 * ls;
    return (64 * 2 * (size_t)prec + w) * sizeof(double);
}

// Workgroups of either kernel that fit a CU by their LDS (gfx950: 160 KB).
inline int track_fit(size_t lds) { return (int)std::max<size_t>(1, (160 * 1024) / lds); }

// Lanes per path of a natural count: the next power of two >= n, at least 4.
inline int natural_lanes(int n)
{
    int np = 4;
    while (np < n) np *= 2;
    return np;
}

// wide: a whole wave per path (track_wide_kernel); else `lanes` at least (0: the
// natural count of each system).
struct LaneRule {
    bool wide = false;
    int lanes = 0;
};

// Lanes per path: as asked; else a whole wave while the paths are few (a run
// lasts as long as its longest path, and a wave takes a path's Newton iteration
// in a quarter to two thirds of the time); else the natural count, where a wave's
// lanes do less in vain.  The line lies at f paths per resident wave times the
// ratio of the workgroups that the two kernels have resident: f = 1 up to n = 4, 8
// up to n = 8, 11 up to n = 16, 22 beyond.  Both kernels have eight workgroups of a
// wave per CU with FP64 solves and short terms, and as few as one or two where
// double-double or quad-double matrices, or the partials of long terms, fill the
// LDS.  Measured, natural / wave per path in ms, by workgroups per CU (w: wave per
// path, l: natural).  w 8, l 8: n = 3, 512 paths 1.15 / 0.80 and 4096 1.09 / 1.70; n =
// 8 in double double, 6561 paths 91 / 43 and 52488 132 / 185; n = 16 in quad double,
// 24576 paths 515 / 483.  Quad-double solves, 8 factors: n = 8 (w 2, l 4) 2048 paths
// 302 / 242, 4096 349 / 438, 8192 360 / 833; n = 16 (w 1, l 2) 1408 paths 860 / 790,
// 2816 1423 / 1452, 5632 1474 / 2783.  Double-double solves, 8 factors: n = 8 (w 4, l
// 8) 4096 paths 62 / 53, 8192 66 / 90; n = 16 (w 3, l 4) 5632 paths 244 / 229, 11264
// 335 / 434; n = 24 with 2 factors (w 3, l 2) 4224 paths 2304 / 1549, 16896 7714 /
// 5440.  In double at n = 24 (w 6, l 4) 22528 paths 1091 / 1033.  How far the paths
// of a run differ in length moves the line: 8192 paths of like lengths at n = 8 with
// FP64 solves (w 7, l 8) took 30 / 35.
//
// kmax: most factors of a term; blocks: a bound on all workgroups (0: none);
// bounded_history: the predictor history must fit a buffer made for the other
// kernel's lanes.
inline LaneRule track_lane_rule(int nsys, const int *n_var, const int64_t *path_off, int kmax, const ph_track_opts &o,
                                int cus, int blocks, bool bounded_history)
{
    LaneRule r;
    r.lanes = o.lanes_per_path;
    if (r.lanes != 0) return r;
    int nat_max = 4;
    for (int s = 0; s < nsys; ++s) nat_max = std::max(nat_max, natural_lanes(n_var[s]));
    auto resident = [&](size_t lds) {
        int per_cu = std::min(8, track_fit(lds));
        if (o.blocks_per_cu > 0) per_cu = std::min(per_cu, (int)o.blocks_per_cu);
        const double w = (double)cus * per_cu;
        return blocks > 0 ? std::min(w, (double)blocks) : w;
    };
    const double waves = resident(track_wide_lds_bytes(o.prec, o.mixed, nat_max, kmax));
    const double other = resident(track_lds_bytes(o.prec, o.mixed, nat_max));
    double lanes = 0, share = 0;
    for (int s = 0; s < nsys; ++s) {
        const int nat = natural_lanes(n_var[s]);
        const double np = (double)(path_off[s + 1] - path_off[s]);
        const int f = nat <= 4 ? 1 : (nat <= 8 ? 8 : (nat <= 16 ? 11 : 22));
        lanes += np * nat;
        share += np * other / (f * waves * waves);
    }
    r.wide = share <= 1.0 && !bounded_history;
    // where a wave per path is ruled out: twice the natural count when the paths
    // fill less than one wave per SIMD, and all of them are resident with it (n = 8
    // with 8 factors and quad-double solves, 6000 paths of which 2048 are: 597 ms,
    // 355 with the natural count)
    if (!r.wide && lanes < 64.0 * 4 * cus && 2 * nat_max <= 32 &&
        2 * lanes <= 64.0 * resident(track_lds_bytes(o.prec, o.mixed, 2 * nat_max)))
        r.lanes = 2 * nat_max;
    return r;
}

// Workgroups that the paths keep busy: one path per wave, or 64 / lanes of each
// lane-count class.
inline int64_t track_workgroups(int nsys, const int *n_var, const int64_t *path_off, const LaneRule &r)
{
    int64_t cls[7] = {0};  // paths by log2 of the lanes
    int64_t need = 0;
    for (int s = 0; s < nsys; ++s) {
        const int lanes = std::max(natural_lanes(n_var[s]), r.lanes);
        cls[std::min(6, __builtin_ctz(lanes))] += path_off[s + 1] - path_off[s];
    }
    for (int c = 2; c < 7; ++c) {
        const int per_wave = r.wide ? 1 : 64 >> c;
        need += (cls[c] + per_wave - 1) / per_wave;
    }
    return need;
}

// A launch shape to time: options, and the kernel that the whole run takes
// with them (a sample has fewer paths, and the automatic choice would take another).
struct TuneCand {
    ph_track_opts o;
    LaneRule rule;
};

// The launch shapes of a run with path counts full_off, timed on a sample with path
// counts off: the automatic lane count, the natural one (4) where that is another,
// twice and four times the natural count; residency-limited workgroups per CU in the
// persistent schedule (of those that launch the same grid on the sample, the
// largest), and round counts and time budgets per launch in the graph schedule.
inline std::vector<TuneCand> tune_candidates(int nsys, const int *n_var, const int64_t *full_off, const int64_t *off,
                                             int kmax, const ph_track_opts &opts, int cus, int blocks)
{
    int np_max = 4;
    for (int s = 0; s < nsys; ++s) np_max = std::max(np_max, natural_lanes(n_var[s]));
    std::vector<TuneCand> cands;
    auto make = [&](int lanes, int sch, int rnd, int bpc, double lms) {
        TuneCand c{opts, {}};
        c.o.schedule = sch;
        c.o.rounds_per_launch = rnd;
        c.o.blocks_per_cu = bpc;
        c.o.lanes_per_path = lanes;
        c.o.launch_ms = lms;
        c.rule = track_lane_rule(nsys, n_var, full_off, kmax, c.o, cus, blocks, false);
        return c;
    };
    auto fit = [&](const LaneRule &r) {
        const int np = std::max(np_max, r.lanes);
        return r.wide ? std::min(8, track_fit(track_wide_lds_bytes(opts.prec, opts.mixed, np, kmax)))
                      : track_fit(track_lds_bytes(opts.prec, opts.mixed, np));
    };
    const LaneRule first = make(0, PH_SCHED_PERSISTENT, opts.rounds_per_launch, 8, opts.launch_ms).rule;
    for (int lanes : {0, 4, 2 * np_max, 4 * np_max}) {
        if (lanes > 32 || (lanes == 4 && !first.wide && first.lanes == 0)) continue;
        if (lanes > 4 && !first.wide && first.lanes == lanes) continue;  // what 0 chooses
        std::vector<TuneCand> shapes;
        for (int bpc : {16, 12, 8, 4, 2}) {
            const TuneCand c = make(lanes, PH_SCHED_PERSISTENT, opts.rounds_per_launch, bpc, opts.launch_ms);
            if (bpc > fit(c.rule) && bpc != 2) continue;
            if (!shapes.empty()) {
                const TuneCand &b = shapes.back();
                const int64_t need = track_workgroups(nsys, n_var, off, c.rule);
                if (b.rule.wide == c.rule.wide && b.rule.lanes == c.rule.lanes && need <= (int64_t)cus * bpc) continue;
            }
            shapes.push_back(c);
        }
        cands.insert(cands.end(), shapes.rbegin(), shapes.rend());
        const int bpc = std::min(8, fit(make(lanes, PH_SCHED_GRAPH, 32, 8, 0.0).rule));
        for (int rnd : {8, 32, 128}) cands.push_back(make(lanes, PH_SCHED_GRAPH, rnd, bpc, 0.0));
        for (double lms : {1.0, 2.0, 4.0}) cands.push_back(make(lanes, PH_SCHED_GRAPH, 32, bpc, lms));
    }
    return cands;
}

}  // namespace ph
