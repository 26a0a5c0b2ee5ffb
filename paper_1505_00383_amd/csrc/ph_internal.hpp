// ph_internal.hpp -- internal structures shared by the system compiler, the
// evaluation kernels and the tracker.  Not part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/ph.h"
#include "ph_sweep.hpp"

namespace ph {

// Error reporting: the message of the last failure on this thread.
void set_error(const std::string &msg);
int fail(int code, const std::string &msg);
int hip_fail(hipError_t e, const char *what);

#define PH_HIP(call)                                     \
    do {                                                 \
        hipError_t e_ = (call);                          \
        if (e_ != hipSuccess) return ph::hip_fail(e_, #call); \
    } while (0)


// Term descriptor: {k = number of factors, offset of the first factor word,
// sel = 0 for a target term (coefficient scaled by t) or 1 for a start-system
// term (scaled by gamma (1 - t)), unused}.
//
// One "homotopy table" is the merged term stream of target and start system,
// equation by equation: the instruction stream that every lane of a wave runs
// on its own point (Section 3: all threads of a block evaluate the same
// monomial at different points).
// Term record of the complex-double fast path: everything one term needs in
// one 192-byte block read through scalar loads, each field ready to use so
// that the kernel spends no scalar instructions decoding it: per factor l the
// LDS byte offsets of x_{j_l} and of x_{j_l}^{a_l - 1} (powers x, x^2, x^3
// and a row of ones are staged per point), the register index 2 j_l of its
// Jacobian column, and the exponent a_l as a double (folded into the FMA that
// accumulates the partial).
// Fast-path record groups: (k, m) with 0 <= m <= k <= 8, numbered k(k+1)/2 + m;
// DRUN offsets per equation (45 groups and the end).
constexpr int DRUN = 46;
inline constexpr int drun_group(int k, int m) { return k * (k + 1) / 2 + m; }

// A term of 9 to 16 factors of exponent 1 is two records of half the factors
// each, the other half's factors in the place of the powers; the second adds
// no value.  A quarter more products than one sweep, with the row on chip: n =
// 10, terms of up to 10 factors, 34940 points, general or register-row kernel and
// this: 154 and 34 us in double, 393 and 150 us in double double, 1.95 and 1.05
// ms in quad double.
constexpr int32_t DSEL_NOVALUE = 2;
// The record's first factor belongs to the other half: no partial of it.
constexpr int32_t DSEL_DROP = 4;
// DSEL_TWO << l: factor l < m has no x^a in the power table, its value takes
// the products by x^(a-1) (or the other half's factor) and by x.
constexpr int32_t DSEL_TWO = 1 << 8;
struct DTerm {
    double cre, cim;
    int32_t k;
    int32_t sel;     // bit 0: start term; DSEL_NOVALUE, DSEL_DROP, DSEL_TWO; bits 16..19: m
    uint32_t xo[8];  // LDS byte offset of the factor's coordinate x_v (v * 1024)
    uint32_t po[8];  // LDS byte offset of x_v^(a-1), or of the ones row for a = 1
    uint32_t j2[8];  // 2 * v: register index of column v in the pinned row
    double a[8];     // exponents
    int32_t pad[2];
};

// Term record of the double-double and quad-double fast paths, in the same
// order as the DTerm records (the same d_run groups index both): the
// coefficient in all its limbs, per factor the LDS byte offsets of x_{j_l}
// and x_{j_l}^{a_l - 1} (both staging layouts give a (plane, variable) block
// 2048 bytes: DD four rows of 64 points, QD eight rows of 32 points), the
// accumulation-register index 8 j_l of its Jacobian column, and the exponent
// as a double.
struct MTerm {
    double c[8];     // [re, im][4 limbs]
    int32_t k, sel;  // as in DTerm
    uint32_t xo[8];
    uint32_t po[8];
    uint32_t jo[8];
    double a[8];
    int32_t pad[6];
};
static_assert(sizeof(MTerm) == 256, "MTerm is one 256-byte record");

// Term schedule of the tracker kernel that gives a wave to one path (built by
// build_wide, see wide_table.cpp): per round of 64 terms and lane the term's
// shape (factors in bits 0..7, start term in bit 8; WIDE_NONE: no term), its
// factor words and coefficient limbs; per chunk of WIDE_ROUNDS rounds {first
// list step, list steps, a multiple of four, steps with partials}; per list
// step and lane {a partial's slot, the matrix entry it is added to in bits 16.. and whether it is
// the entry's first and last one of the chunk (zero: nothing to add); the slot
// of a term's value, WIDE_NONE for nothing}.
constexpr int WIDE_ROUNDS = 2;
constexpr uint32_t WIDE_NONE = 0xffffffffu;
constexpr uint32_t WIDE_FIRST = 0x80000000u, WIDE_LAST = 0x40000000u, WIDE_ENTRY = 0x7ffu;
struct WideTable {
    int rounds = 0;
    std::vector<uint32_t> meta, fac;
    std::vector<uint2> list;
    std::vector<double> coef;
    std::vector<int4> chunk;
};

// The device copy of a WideTable.
struct WideDev {
    const uint32_t *meta, *fac;
    const uint2 *list;
    const double *coef;
    const int4 *chunk;
    int32_t rounds, chunks;
};

struct DevTable {
    int n_eq = 0, n_var = 0, kmax = 0;
    int emax = 0;                // largest exponent of a target/start term
    bool dfast = false;          // the fast-path records below are valid
    bool dlong = false;          // records of terms with more than 8 factors among them
    int dfast_planes = 0;        // power planes staged in LDS (x, x^2, x^3)
    int32_t *d_eq_off = nullptr; // [n_eq + 1] offsets into dterm
    DTerm *dterm = nullptr;      // fast-path records (target terms, custom start terms)
    int32_t *d_deg = nullptr;    // [n_eq] total-degree start exponents (0: explicit start)
    bool mfast = false;          // the DD / QD records below are valid (LDS fits)
    MTerm *mterm = nullptr;      // DD / QD fast-path records, parallel to dterm
    int32_t *d_run = nullptr;    // [n_eq][DRUN]: records of equation i in group g (k
                                 // factors, m of them with a >= 2; g = drun_group(k, m))
                                 // are d_run[i*DRUN+g] .. d_run[i*DRUN+g+1]-1
    int64_t n_terms = 0, n_fac = 0;
    int32_t *eq_off = nullptr;   // [n_eq + 1]
    int4 *tdesc = nullptr;       // [n_terms]
    uint32_t *fac = nullptr;     // [n_fac]
    uint32_t *fac8 = nullptr;    // [n_terms][8]: each term's factor words, zero padded (tracker)
    double *coef = nullptr;      // [n_terms][2][4] limbs
    bool coef_single = false;    // every coefficient is an FP64 number
    int cus = 256;               // compute units of the device
    // fast path: mean over the G groups of the work of a workgroup's slowest
    // wave with min(2^c, n_eq) waves, at [c][G - 1]
    std::vector<float> fit[4], fit_max[4];  // (and the slowest of the groups)
    WideDev wide{};              // square systems of n <= 32, k <= 8 (rounds 0: none)
    int32_t *zc_off = nullptr;   // [n_eq + 1] columns of each row no term touches
    int32_t *zc = nullptr;
    // the paper's unfused three-kernel design (coeff, mon, sum; an ablation):
    int64_t u_slots = 0;         // monomial slots: value and k partials per term
    int32_t *u_slot = nullptr;   // [n_terms] first slot of each term
    int32_t *u_off = nullptr;    // [n_eq * (1 + n_var) + 1] slots summed into each output
    int32_t *u_list = nullptr;   //   entry: H_i (entries 0..n_eq-1), then J_ij row-major
    void *block = nullptr;       // single device allocation holding all of the above
    void *u_scratch = nullptr;   // grow-only intermediate arrays of the unfused design,
    size_t u_scratch_bytes = 0;  //   sized by ph_eval_prepare (never by an evaluation)
};

// Waves per workgroup and equation groups of a fast-path launch where the
// configuration names none.  A workgroup of W waves stages a tile of points and
// takes every G-th run of W equations; a CU holds `waves` waves of the kernel
// and as many workgroups as their LDS allows.  The launch takes the number of
// rounds of workgroups times the work of one, which is that of its slowest wave
// (DevTable::fit, in complex products) and the staging; the choice begins with
// the largest W and one group, and another must win 3 %.  Measured against the
// largest W and one group (double: enough groups for 1024 workgroups), n = 32
// with 64 terms of 8 factors: 1000 points 1.53 -> 0.20 ms in double double, 7.97
// -> 1.04 ms in quad double; 4999 points 1.55 -> 0.60 and 8.0 -> 5.2; 50000
// points 0.751 -> 0.669 in double, 6.5 -> 5.0 in double double.
struct EvalFit {
    int W, G;
};
inline EvalFit eval_fit(const DevTable &tab, int64_t tiles, int max_w, int fixed_w, int waves, size_t lds,
                        double stage, double even)
{
    EvalFit best{1, 1};
    double best_t = -1;
    for (int c = 3; c >= 0; --c) {
        const int W = std::min(1 << c, tab.n_eq);
        if ((1 << c) > max_w || (fixed_w > 0 && (1 << c) > fixed_w) || (c > 0 && W <= 1 << (c - 1))) continue;
        const int64_t fit = std::min<int64_t>(std::max(1, waves / W), std::max<int64_t>(1, (160 * 1024) / lds));
        const int64_t slots = tab.cus * fit;
        const double st = stage + double(tab.dfast_planes) * tab.n_var / W;
        for (int G = 1; G <= (int)tab.fit[c].size(); ++G) {
            const double rounds = double((tiles * G + slots - 1) / slots);
            const double t = rounds > 1 ? rounds * (tab.fit[c][G - 1] + st) : tab.fit_max[c][G - 1] + st;
            if (best_t < 0 || t < 0.97 * best_t) {
                best = EvalFit{W, G};
                // a single round of workgroups evens nothing out
                best_t = G == 1 && tiles <= slots ? even * t : t;
            }
        }
        if (fixed_w > 0) break;
    }
    return best;
}

// Waves and groups of a launch for a configuration that may name either: waves
// alone, the groups are chosen for them (fit(W)); groups alone, the waves are
// the default def_w and the groups are halved until every one has W equations,
// as when both are named.  No workgroup is left without an equation.
template <class Fit>
EvalFit named_tiling(int n_eq, int cfg_w, int cfg_g, int def_w, int max_w, Fit &&fit)
{
    int W = std::min({cfg_w > 0 ? cfg_w : (cfg_g > 0 ? def_w : 0), max_w, n_eq}), G = cfg_g;
    if (cfg_g > 0) {
        while (G > 1 && G * W > n_eq) G >>= 1;
    } else {
        const EvalFit ft = fit(W);
        if (W <= 0) W = ft.W;
        for (G = ft.G; G > 1 && (G - 1) * W >= n_eq;) --G;
    }
    return EvalFit{W, G};
}
inline EvalFit fast_tiling(const DevTable &tab, int64_t tiles, int cfg_w, int cfg_g, int def_w, int max_w, int waves,
                           size_t lds, double stage, double even)
{
    return named_tiling(tab.n_eq, cfg_w, cfg_g, def_w, max_w,
                        [&](int W) { return eval_fit(tab, tiles, max_w, W, waves, lds, stage, even); });
}

// The same for the double-double values kernel: `waves` waves per CU hide each other's
// chains, in as small workgroups as their LDS lets a CU hold them (or of fixed_w
// waves), and the work of a CU is the equations of its workgroups.
inline EvalFit values_fit(const DevTable &tab, int64_t tiles, int fixed_w, int waves, size_t lds, double stage)
{
    const int fit = std::max<int>(1, (int)((160 * 1024) / lds));
    EvalFit best{1, 1};
    while (best.W < waves && best.W * fit < waves) best.W *= 2;
    if (fixed_w > 0) best.W = fixed_w;
    if (best.W > tab.n_eq) best.W = tab.n_eq;
    const int W = best.W;
    double best_t = -1;
    for (int G = 1; (G - 1) * W < tab.n_eq; ++G) {
        const double t = double((tiles * G + tab.cus - 1) / tab.cus) * (W * ((tab.n_eq + G * W - 1) / (G * W)) + stage);
        if (best_t < 0 || t < 0.97 * best_t) {
            best_t = t;
            best.G = G;
        }
    }
    return best;
}

// Kernel choice and tiling of one evaluation: kernel 0 automatic, 1 general
// (Jacobian row accumulated in the output), 2 register row (double, n <= 32),
// 3 fast path with the row pinned in registers (double: upper architectural
// registers; double double and quad double: accumulation registers), 4 the double fast path
// with a compiler-held row, 5 the unfused coeff / mon / sum kernels; W waves
// per workgroup, G equation groups (0: default).  tuned: timed on calls with a
// Jacobian, so its tiling says nothing about the values kernels.
struct EvalCfg {
    int kernel = 0, W = 0, G = 0;
    bool tuned = false;
};

struct HostSystem {
    uint64_t fingerprint = 0;  // FNV-1a of the defining arrays
    int n_eq = 0, n_var = 0, max_k = 0;
    std::vector<int32_t> eq_term_off, term_fac_off, fac_var, fac_exp, deg;
    std::vector<double> coef;  // [T][2][4]
};

struct ph_system_impl;

}  // namespace ph

struct ph_system {
    ph::HostSystem h;
    ph::DevTable total;  // target merged with the total-degree start system
    std::mutex mu;
    std::map<const ph_system *, ph::DevTable> with_start;  // custom start systems
    std::map<std::pair<const ph_system *, int>, ph::EvalCfg> eval_cfg;  // (start, prec) -> config
    // entries of the PH_AUTOTUNE_CACHE file for this target, read once when
    // the handle is created: (start fingerprint or 0, prec) -> config
    std::map<std::pair<uint64_t, int>, ph::EvalCfg> file_cfg;
    // the choices autotuned for calls without a Jacobian, which other calls
    // must not take (a values kernel says nothing about the Jacobian's)
    std::map<std::pair<const ph_system *, int>, ph::EvalCfg> values_cfg;
    std::map<std::pair<uint64_t, int>, ph::EvalCfg> file_values;
    int device = 0;
};

namespace ph {
// Build and upload the merged table of (f, g); g == nullptr selects the
// total-degree start system g_i = x_i^{d_i} - 1.
int build_table(const HostSystem &f, const HostSystem *g, DevTable &out);
void build_wide(int n, const std::vector<int32_t> &eq_off, const std::vector<int4> &tdesc,
                const std::vector<uint32_t> &fac, const std::vector<double> &coef, WideTable &w);
void free_table(DevTable &t);
// Table for (target, start), built on first use and cached in the target
// (allocates and synchronises when it builds).
int get_table(const ph_system *target, const ph_system *start, const DevTable **out);
// The same without building: PH_EINVAL when (target, start) was not prepared.
int find_table(const ph_system *target, const ph_system *start, const DevTable **out);
// Size the unfused design's intermediate arrays for npts points of prec limbs
// (grow-only; synchronises the device before releasing a smaller buffer).
int prepare_unfused(const ph_system *target, DevTable &tab, int prec, int64_t npts);
// Entries of the PH_AUTOTUNE_CACHE file for this target (called at creation).
void load_eval_cache(ph_system *s);
// Values alone of a system with records, in double double and quad double.
// W and G as configured, 0: chosen by the launch.
int dd_values_launch(const DevTable &tab, const double gamma[2], int64_t npts, const double *t, const double *x,
                     int64_t ld, double *val, int W, int G, hipStream_t st);
int qd_values_launch(const DevTable &tab, const double gamma[2], int64_t npts, const double *t, const double *x,
                     int64_t ld, double *val, int W, int G, hipStream_t st);
// The unfused three-kernel evaluation (kernel choice 5).
int unfused_launch(const DevTable &tab, const double gamma[2], int prec, int64_t npts,
                   const double *t, const double *x, int64_t ld, double *val, double *jac,
                   hipStream_t st);
// Double-double fast path (kernel choice 3 at prec 2): Jacobian row in the
// accumulation registers, W <= 4 waves per workgroup, G equation groups.
int dd_fast_launch(const DevTable &tab, const double gamma[2], int64_t npts, const double *t,
                   const double *x, int64_t ld, double *val, double *jac, int W, int G,
                   hipStream_t st);
// Quad-double fast path (kernel choice 3 at prec 4): two lanes per point, each
// lane's component of the Jacobian row in the accumulation registers.
int qd_fast_launch(const DevTable &tab, const double gamma[2], int64_t npts, const double *t,
                   const double *x, int64_t ld, double *val, double *jac, int W, int G,
                   hipStream_t st);
// Evaluation launch with an explicit configuration (cfg == NULL: defaults).
int eval_launch(const DevTable &tab, const double gamma[2], int prec, int64_t npts,
                const double *t, const double *x, int64_t ld, double *val, double *jac,
                hipStream_t st, const EvalCfg *cfg);
}  // namespace ph
