// ph_track_wide.hpp -- the tracker kernel that gives a whole wave to one path.
//
// What bounds it: a run with few paths lasts as long as its longest path, and a
// path is a serial chain of Newton iterations, so the time of one iteration
// on one wave is what counts, not the work of the lanes.  With one lane per
// equation (ph_track_dev.hpp) two thirds of an iteration were the term
// sweeps, one after the other, and a quarter the projections of the MGS.
// Here
//   * the terms of all equations are dealt to the 64 lanes (wide_table.cpp):
//     n = 8 with 22 terms per equation takes three rounds of sweeps instead of
//     eleven, and the lanes of a round sweep terms of the same shape;
//   * partials and values are handed over in LDS slots, and each matrix entry
//     is summed by one lane from a list, in term order;
//   * the 64 / NP groups of NP lanes (lane i of a group owns row i) each
//     project their own columns of [J | -H], which stay in registers;
//   * every group carries the same path state, so nothing about a path is
//     exchanged, and every path decision is uniform over the wave.
// The sums are the additions of ph_track_dev.hpp in the same order and the
// projections the same operations, so the results are the same bit for bit.
#pragma once

#include "ph_track_dev.hpp"

namespace ph {

// LDS of one wave in doubles, in the order of the arrays below.
template <int L, int NP, int LS>
__host__ __device__ constexpr size_t wide_lds_doubles(int kmax)
{
    return (size_t)NP * 2 * L + (size_t)(NP + 1) * NP * 2 * LS + (size_t)NP * 2 * LS +
           (size_t)64 * WIDE_ROUNDS * (2 * L + kmax * 2 * LS);
}

template <int L>
__device__ __forceinline__ R<L> lds_getr(const double *p)
{
    R<L> r;
#pragma unroll
    for (int l = 0; l < L; ++l) r.v[l] = p[l];
    return r;
}

__device__ __forceinline__ double wave_read(double v, int lane)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), lane);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

__device__ __forceinline__ void wave_handover()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// Run at most max_rounds rounds of the tracker on this wave's path, or until
// the queue of the class is empty (returns true).
template <int L, int NP, int KMAX, bool MIXED>
__device__ __forceinline__ bool run_wide(const TrackArgs &a, const TrackClass &cl, Slot<L> &S, int max_rounds,
                                         double *__restrict__ lds)
{
    constexpr int LS = MIXED ? 1 : L;
    constexpr int CW = 64 / NP;                // lane groups, each with its own columns
    constexpr int NC = (NP + CW - 1) / CW;     // columns per group
    // columns in registers where they are few; else in LDS with rolled loops
    // (a plain quad-double projection is 2000 instructions)
    constexpr bool REG = LS == 1 ? NC <= 4 : NC == 1;
    constexpr int SL = 64 * WIDE_ROUNDS;       // slots of a chunk
    constexpr bool AHEAD = L <= 2;             // read the next round's terms during the current sweep
    const int lane = threadIdx.x;
    const int i = lane % NP, c = lane / NP;
    const PathLane<L> pl{i, c == 0, (int64_t)blockIdx.x * a.wide_cols + i};
    const R<L> h3 = half_sqrt3_t<L>();
    double *xg = lds;                          // the iterate
    double *wsh = xg + NP * 2 * L;             // [J | -H], column major
    double *ash = wsh + (NP + 1) * NP * 2 * LS;  // projected right-hand side (LDS columns)
    double *vs = ash + NP * 2 * LS;            // term values: [re, im][slot][limb]
    double *ps = vs + SL * 2 * L;              // partials: [factor][slot][re, im][limb]
    auto W = [&](int j, int row) -> double * { return wsh + ((size_t)j * NP + row) * 2 * LS; };

    bool retired = false;
    const long long t_start = a.budget ? wall_clock64() : 0;  // time-budgeted launches
    for (int round = 0; round < max_rounds; ++round) {
        // ---- refill -------------------------------------------------------
        if (__builtin_amdgcn_readfirstlane(S.phase) == PH_EMPTY) {
            unsigned long long id = 0;
            if (lane == 0) id = queue_pop(cl.queue);
            id = __shfl(id, 0);
            path_start<L>(a, cl, S, pl, (int64_t)id, h3);
        }
        if (__builtin_amdgcn_readfirstlane(S.phase) == PH_STEP && __builtin_amdgcn_readfirstlane(S.steps) == 0) {
            const bool any_bad = gmax_d<NP>(c_bad<L>(S.x) ? 1.0 : 0.0) > 0.0;
            if (a.o.h_min > a.o.h_init) path_finish<L>(a, S, pl, PH_R_STEP_UNDERFLOW);
            else if (any_bad) path_finish<L>(a, S, pl, PH_R_NAN);
        }
        if (__builtin_amdgcn_readfirstlane(S.phase) == PH_RETIRED) {
            retired = true;
            break;
        }
        // the first round's terms are read before the predictor runs
        const SysDesc &sd = a.sys[__builtin_amdgcn_readfirstlane(S.sidx)];
        const WideDev wd = sd.wide;
        auto fetch = [&](int r, uint32_t &m, C<L> &cf, uint32_t (&fw)[KMAX]) {
            m = tab_read(wd.meta, r * 64 + lane);
#pragma unroll
            for (int l = 0; l < L; ++l) {
                cf.re.v[l] = tab_read(wd.coef, (r * 8 + l) * 64 + lane);
                cf.im.v[l] = tab_read(wd.coef, (r * 8 + 4 + l) * 64 + lane);
            }
#pragma unroll
            for (int l = 0; l < KMAX; ++l) fw[l] = tab_read(wd.fac, (r * 8 + l) * 64 + lane);
        };
        uint32_t mn = WIDE_NONE, fn[KMAX];
        C<L> cn = c_zero<L>();
#pragma unroll
        for (int l = 0; l < KMAX; ++l) fn[l] = 0u;
        if (AHEAD && wd.rounds > 0) fetch(0, mn, cn, fn);
        if (__builtin_amdgcn_readfirstlane(S.phase) == PH_STEP) path_predict<L>(a, S, pl);
        const int phase = __builtin_amdgcn_readfirstlane(S.phase);
        if (phase == PH_CORRECT || phase == PH_POLISH) {
            const int n = __builtin_amdgcn_readfirstlane(S.n);
            const double tt = phase == PH_POLISH ? 1.0 : S.t1;

            // ---- evaluate H and J at (xh, tt) -------------------------------
            if (c == 0) {
#pragma unroll
                for (int l = 0; l < L; ++l) {
                    xg[i * 2 * L + l] = S.xh.re.v[l];
                    xg[i * 2 * L + L + l] = S.xh.im.v[l];
                }
            }
            for (int e = lane; e < (NP + 1) * NP; e += 64) lds_put<LS>(wsh + (size_t)e * 2 * LS, c_zero<LS>());
            wave_handover();
            C<L> gs;
            {
                double o1, oe;
                two_sum(1.0, -tt, o1, oe);
                R<L> omt = r_zero<L>();
                omt.v[0] = o1;
                if constexpr (L > 1) omt.v[1] = oe;
                gs = c_mul_r<L>(c_from<L>(sd.gre, sd.gim), omt);
            }
            auto X = [&](int var) -> C<L> {
                C<L> z;
#pragma unroll
                for (int l = 0; l < L; ++l) {
                    z.re.v[l] = xg[var * 2 * L + l];
                    z.im.v[l] = xg[var * 2 * L + L + l];
                }
                return z;
            };
            Acc<L> v = acc_zero<L>();  // lane 2 e + c: component c of H_e
            for (int ch = 0; ch < wd.chunks; ++ch) {
                const vec4i cd = tab_read(reinterpret_cast<const vec4i *>(wd.chunk), ch);
                auto list4 = [&](int s, vec2u (&g)[4]) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        g[q] = tab_read(reinterpret_cast<const vec2u *>(wd.list), (cd.x + s + q) * 64 + lane);
                };
                vec2u gn[4];
                if (AHEAD) list4(0, gn);
                for (int r = ch * WIDE_ROUNDS; r < (ch + 1) * WIDE_ROUNDS && r < wd.rounds; ++r) {
                    uint32_t m = mn, fw[KMAX];
                    C<L> cf = cn;
#pragma unroll
                    for (int l = 0; l < KMAX; ++l) fw[l] = fn[l];
                    if (AHEAD) {
                        if (r + 1 < wd.rounds) fetch(r + 1, mn, cn, fn);
                    } else {
                        fetch(r, m, cf, fw);
                    }
                    if (m != WIDE_NONE) {
                        const int slot = (r - ch * WIDE_ROUNDS) * 64 + lane;
                        const bool start = (m & 0x100u) != 0;
                        const C<L> ct = coef_t<L>(cf, tt, a.coef_single != 0);
                        cf = __any(start) ? c_sel<L>(start, c_mul<L>(cf, gs), ct) : ct;
                        const C<L> tv = wave_sweep<KMAX, L>(
                            (int)(m & 0xffu), fw, cf, X, [&](int l, uint32_t, const C<L> &part) {
                                lds_put<LS>(ps + (size_t)(l * SL + slot) * 2 * LS, narrow<LS, L>(part));
                            });
#pragma unroll
                        for (int q = 0; q < L; ++q) {
                            vs[slot * L + q] = tv.re.v[q];
                            vs[(SL + slot) * L + q] = tv.im.v[q];
                        }
                    }
                }
                wave_handover();
                // add the chunk's partials and values, every entry by one lane
                // in term order: four list words of each kind at a time, the
                // next ones read meanwhile
                if (!AHEAD) list4(0, gn);
                C<LS> run = c_zero<LS>();
#pragma unroll 1
                for (int s = 0; s < cd.y; s += 4) {
                    vec2u g[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) g[q] = gn[q];
                    if (s + 4 < cd.y) list4(s + 4, gn);
                    R<L> u[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        u[q] = lds_getr<L>(vs + ((lane & 1) * SL + (g[q].y & (SL - 1))) * L);
                    if (s < cd.z) {
                        // an entry's partials follow each other in its lane's
                        // list: it is read before the first and written
                        // after the last of them
                        C<LS> part[4], old[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            part[q] = lds_get<LS>(ps + (size_t)(g[q].x & 0xffffu) * 2 * LS);
                            old[q] = lds_get<LS>(wsh + (size_t)((g[q].x >> 16) & WIDE_ENTRY) * 2 * LS);
                        }
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            run = c_add<LS>(c_sel<LS>((g[q].x & WIDE_FIRST) != 0, old[q], run), part[q]);
                            if (g[q].x & WIDE_LAST) lds_put<LS>(wsh + (size_t)((g[q].x >> 16) & WIDE_ENTRY) * 2 * LS, run);
                        }
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
#pragma unroll
                        for (int l = 0; l < L; ++l) u[q].v[l] = g[q].y == WIDE_NONE ? 0.0 : u[q].v[l];
                        acc_add<L>(v, u[q]);
                    }
                }
                wave_handover();
            }
            if (lane < 2 * n) {
                const R<L> nv = r_neg<L>(acc_value<L>(v));
                double *en = W(NP, lane >> 1) + (lane & 1) * LS;
#pragma unroll
                for (int l = 0; l < LS; ++l) en[l] = nv.v[l];
            }
            wave_handover();

            // ---- correct: MGS least squares on [J | -H] ----------------------
            C<LS> rhs = lds_get<LS>(W(NP, i));
            const C<LS> res = rhs;
            double fro = 0.0;
#pragma unroll 4
            for (int j = 0; j < n; ++j) {
                const C<LS> w = lds_get<LS>(W(j, i));
                fro += w.re.v[0] * w.re.v[0] + w.im.v[0] * w.im.v[0];
            }
            fro = gsum_d<NP>(fro);
            double lim2 = a.eps_sing * a.eps_sing * fro;
            // rare: out of the loop's way (in line, n = 24 in double double 440
            // ms instead of 403)
            if (__builtin_expect(mgs_far(__builtin_amdgcn_readfirstlane(mgs_high(fro))), 0)) {
                const int sc = mgs_exponent(fro);
                for (int j = c; j <= NP; j += CW) mgs_scale<LS>(W(j, i), sc);
                wave_handover();
                rhs = lds_get<LS>(W(NP, i));
                lim2 = a.eps_sing * a.eps_sing * __builtin_amdgcn_ldexp(fro, 2 * sc);
            }
            bool sing = false;
            C<LS> acc = c_zero<LS>();       // r_{i,rhs}, then the back-substitution value
            if constexpr (REG) {
                C<LS> col[NC];
#pragma unroll
                for (int jj = 0; jj < NC; ++jj)
                    col[jj] = jj * CW + c < NP ? lds_get<LS>(W(jj * CW + c, i)) : c_zero<LS>();
                // the right-hand side takes the place of the first group's
                // column once that column is the pivot: no lane projects it
                // beside a column of its own
#pragma unroll
                for (int kk = 0; kk < NC; ++kk) {
#pragma unroll 1
                    for (int ck = 0; ck < CW; ++ck) {
                        const int k = kk * CW + ck;
                        if (k >= n || sing) break;
                        const C<LS> wk = shfl_c<LS>(col[kk], ck * NP + i);
                        if (ck == 0) {
                            if (c == 0) col[kk] = rhs;
                        }
                        // all group sums of the step side by side
                        const R<LS> nu = gsum_r<NP, LS>(c_abs2<LS>(wk));
                        C<LS> r[NC];
#pragma unroll
                        for (int jj = kk; jj < NC; ++jj) r[jj] = gsum_c<NP, LS>(c_cmul<LS>(wk, col[jj]));
                        R<LS> inv;
                        if (!mgs_pivot<LS>(nu, lim2, inv)) {
                            sing = true;
                            break;
                        }
                        // columns up to k are finished: what these lanes
                        // compute of them is never read
#pragma unroll
                        for (int jj = kk; jj < NC; ++jj) {
                            r[jj] = c_mul_r<LS>(r[jj], inv);
                            col[jj] = c_submul<LS>(col[jj], r[jj], wk);
                            // R'(k, j) to column j, row k of the matrix in LDS
                            if (i == jj && jj * CW + c < NP) lds_put<LS>(W(jj * CW + c, k), r[jj]);
                        }
                        if (i == k) acc = r[kk];  // the first group's
                    }
                    rhs = col[kk];
                }
            } else {
#pragma unroll 1
                for (int k = 0; k < n; ++k) {
                    const C<LS> wk = lds_get<LS>(W(k, i));
                    R<LS> inv;
                    if (!mgs_pivot<LS>(gsum_r<NP, LS>(c_abs2<LS>(wk)), lim2, inv)) {
                        sing = true;
                        break;
                    }
                    // column k is dead: R'(k, j) goes to row j of it; jv = n
                    // stands for the right-hand side
#pragma unroll 1
                    for (int jv = k + 1 + c; jv <= n; jv += CW) {
                        double *ej = W(jv == n ? NP : jv, i);
                        const C<LS> wj = lds_get<LS>(ej);
                        const C<LS> r = c_mul_r<LS>(gsum_c<NP, LS>(c_cmul<LS>(wk, wj)), inv);
                        lds_put<LS>(ej, c_submul<LS>(wj, r, wk));
                        if (i == 0) lds_put<LS>(jv == n ? ash + k * 2 * LS : W(k, jv), r);
                    }
                    wave_handover();
                }
            }
            wave_handover();
            if constexpr (!REG) acc = lds_get<LS>(ash + i * 2 * LS);
            // back substitution R' dx = r_rhs (unit diagonal), column oriented:
            // lane i of the first group carries acc_i
            C<LS> dxi = c_zero<LS>();
            if (!sing) {
#pragma unroll 1
                for (int k = n - 1; k >= 0; --k) {
                    const C<LS> rik = lds_get<LS>(REG ? W(k, i) : W(i, k));  // R'(i, k)
                    C<LS> dk;
#pragma unroll
                    for (int l = 0; l < LS; ++l) {
                        dk.re.v[l] = wave_read(acc.re.v[l], k);
                        dk.im.v[l] = wave_read(acc.im.v[l], k);
                    }
                    if (i == k) dxi = dk;
                    if (i < k) acc = c_submul<LS>(acc, rik, dk);
                }
            }
            if (i >= n) dxi = c_zero<LS>();
            path_decide<L, NP, LS>(a, S, pl, dxi, sing, res, fro);
            // the first group's history writes reach the others
            if (a.o.predictor_order >= 2) wave_handover();
        }
        if (a.budget && (unsigned long long)(wall_clock64() - t_start) >= a.budget) break;
    }
    return retired;
}

// As run_class and track_kernel of ph_track_dev.hpp.
template <int L, int KMAX, bool MIXED, int NPSEL>
__device__ __forceinline__ bool run_wide_class(const TrackArgs &a, Slot<L> &S, int max_rounds, double *lds)
{
    const int b = blockIdx.x;
    int c = 0;
    while (c < 3 && b >= a.cls[c].block_end) ++c;
    const TrackClass &cl = a.cls[c];
    if constexpr (NPSEL < 0) {
        return run_wide<L, -NPSEL, KMAX, MIXED>(a, cl, S, max_rounds, lds);
    } else {
        if (cl.np == 4) return run_wide<L, 4, KMAX, MIXED>(a, cl, S, max_rounds, lds);
        if (cl.np == 8) return run_wide<L, 8, KMAX, MIXED>(a, cl, S, max_rounds, lds);
        if (cl.np == 16 || NPSEL == 16) return run_wide<L, 16, KMAX, MIXED>(a, cl, S, max_rounds, lds);
        if constexpr (NPSEL >= 32) return run_wide<L, 32, KMAX, MIXED>(a, cl, S, max_rounds, lds);
        return true;
    }
}

template <int L, int KMAX, bool MIXED, int NPSEL>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) track_wide_kernel(TrackArgs a)
{
    extern __shared__ double lds[];
    Slot<L> *st = a.state ? reinterpret_cast<Slot<L> *>(a.state) + (size_t)blockIdx.x * 64 + threadIdx.x
                          : nullptr;
    Slot<L> S;
    if (st)
        S = *st;
    else
        slot_init<L>(S);
    if (__all(S.phase == PH_RETIRED)) return;
    const bool retired = run_wide_class<L, KMAX, MIXED, NPSEL>(a, S, st ? a.rounds : 0x7fffffff, lds);
    if (st) {
        *st = S;
        if (!retired && threadIdx.x == 0) atomicAdd(a.active, 1u);
    }
}

}  // namespace ph
