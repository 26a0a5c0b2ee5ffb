// eval_values.hip -- values alone of gamma (1-t) g + t f (Eq. (1)) in double
// double, for the systems of the fast-path records (n <= 32, exponents up to 4;
// quad double: eval_qd.hip).
//
// Without derivatives a term is one chain of products.  The points' powers x,
// x^2, x^3 are staged in LDS as for the Jacobian kernels, so a factor x^a is one
// product where the table holds it (the sweep of the general kernel multiplied
// a times); records, mapping (lane = point, wave = equation) and the start part
// are the fast path's.  Nothing is held per column, so the kernel needs few
// registers, and the waves of a SIMD hide the chain of each other's products.
// Bound by the FP64 products: n = 32, 64 terms of 8 factors, exponents 1..3,
// 6561 points 431 us in the general kernel, 256 us here; n = 10, up to 10
// factors, 34940 points 158 us, 51 us.  (In complex double a product is four
// instructions, the operands from LDS bound both kernels, and the general one
// was the faster: 214 us against 286 us for 60000 points of n = 25.)
#include <hip/hip_runtime.h>

#include "ph_arith.hpp"
#include "ph_internal.hpp"

namespace ph {

struct ValArgs {
    const double *t;
    const double *x;
    double *val;
    int64_t npts, ld;
    double gre, gim;
    int n_eq, n_var, eq_stride, planes;
};

// a staged number: 2 L rows of 64 points at byte offset off
template <int L>
__device__ __forceinline__ C<L> val_lds(const char *__restrict__ xb, uint32_t off, int lane)
{
    const double *p = reinterpret_cast<const double *>(xb + off) + lane;
    C<L> z;
#pragma unroll
    for (int l = 0; l < L; ++l) {
        z.re.v[l] = p[l * 64];
        z.im.v[l] = p[(L + l) * 64];
    }
    return z;
}

// Scalar copy of a record, read one term ahead.
struct ValHead {
    double c[4];
    int sel, k;
    uint32_t xo[8], po[8];
};
__device__ __forceinline__ ValHead val_head(const MTerm *__restrict__ r)
{
    ValHead h;
    h.c[0] = r->c[0];
    h.c[1] = r->c[1];
    h.c[2] = r->c[4];
    h.c[3] = r->c[5];
    h.sel = r->sel;
    h.k = r->k;
#pragma unroll
    for (int l = 0; l < 8; ++l) {
        h.xo[l] = r->xo[l];
        h.po[l] = r->po[l];
    }
    return h;
}

__global__ void __launch_bounds__(1024)
eval_dd_values_kernel(ValArgs a, const int32_t *__restrict__ d_run, const MTerm *__restrict__ recs,
                      const int32_t *__restrict__ d_deg)
{
    constexpr int L = 2;
    extern __shared__ double xl[];
    const char *xb = reinterpret_cast<const char *>(xl);
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int W = blockDim.x >> 6;
    const int64_t p = (int64_t)blockIdx.x * 64 + lane;
    const bool act = p < a.npts;
    const int nv = a.n_var;
    // plane q holds x^(q+1), then a row of ones, as in the Jacobian kernels
    auto put = [&](int row, const C<L> &z) {
        double *r = xl + (size_t)row * 2 * L * 64 + lane;
#pragma unroll
        for (int l = 0; l < L; ++l) {
            r[l * 64] = z.re.v[l];
            r[(L + l) * 64] = z.im.v[l];
        }
    };
    for (int var = w; var < nv; var += W) {
        C<L> x1 = c_zero<L>();
        if (act) {
#pragma unroll
            for (int l = 0; l < L; ++l) {
                x1.re.v[l] = a.x[(int64_t)(var * 2 * L + l) * a.ld + p];
                x1.im.v[l] = a.x[(int64_t)(var * 2 * L + L + l) * a.ld + p];
            }
        }
        C<L> z = x1;
        for (int q = 0; q < a.planes; ++q) {
            put(q * nv + var, z);
            if (q + 1 < a.planes) z = c_mul<L>(z, x1);
        }
    }
    if (w == 0) put(a.planes * nv, c_from<L>(1.0, 0.0));
    __syncthreads();

    // c(t): t for target terms, gamma (1 - t) for start terms, (1 - t) exact
    double tv = 1.0;
    if (a.t) tv = act ? a.t[p] : 0.0;
    C<L> gs = c_zero<L>();
    if (a.t) {
        R<L> omt;
        two_sum(1.0, -tv, omt.v[0], omt.v[1]);
        gs = c_mul_r<L>(c_from<L>(a.gre, a.gim), omt);
    }
    const uint32_t plane = (uint32_t)nv * 2 * L * 512;  // bytes

    for (int i = blockIdx.y * W + w; i < a.n_eq; i += a.eq_stride) {
        C<L> v = c_zero<L>();
        const int s0 = d_run[i * DRUN], s1 = d_run[i * DRUN + DRUN - 1];
        ValHead h = val_head(recs + (s0 < s1 ? s0 : 0));
        for (int s = s0; s < s1; ++s) {
            // every operand from LDS, the next record by scalar loads, then
            // the products
            const int sel = h.sel, k = h.k, m = (sel >> 16) & 15;
            const C<2> c0 = {{{h.c[0], h.c[1]}}, {{h.c[2], h.c[3]}}};
            C<L> f[8];
            uint32_t xo[8];
#pragma unroll
            for (int l = 0; l < 8; ++l) {
                // x^(a-1) is at po: x^a one plane further, unless the factor
                // takes two products
                xo[l] = h.xo[l];
                const uint32_t off = l < m ? h.po[l] + (sel & (DSEL_TWO << l) ? 0u : plane) : xo[l];
                if (l < k) f[l] = val_lds<L>(xb, off, lane);
            }
            h = val_head(recs + (s + 1 < s1 ? s + 1 : s));
            if (sel & DSEL_NOVALUE) continue;
            C<L> q = (sel & 1) ? c_mul<L>(c0, gs) : c_mul_d<L>(c0, tv);
#pragma unroll
            for (int l = 0; l < 8; ++l)
                if (l < k) q = c_mul<L>(q, f[l]);
#pragma unroll
            for (int l = 0; l < 8; ++l)
                if (sel & (DSEL_TWO << l)) q = c_mul<L>(q, val_lds<L>(xb, xo[l], lane));
            v = c_add<L>(v, q);
        }
        // total-degree start part gamma (1-t) (x_i^d - 1)
        const int d = d_deg[i];
        if (d > 0 && a.t) {
            C<L> base = val_lds<L>(xb, (uint32_t)(i * 2 * L * 512), lane), pw = c_from<L>(1.0, 0.0);
            for (int e = d; e > 0; e >>= 1) {
                if (e & 1) pw = c_mul<L>(pw, base);
                if (e > 1) base = c_mul<L>(base, base);
            }
            v = c_add<L>(v, c_mul<L>(gs, c_sub<L>(pw, c_from<L>(1.0, 0.0))));
        }
        if (act) {
            double *hv = a.val + (int64_t)i * 2 * L * a.ld + p;
#pragma unroll
            for (int l = 0; l < L; ++l) {
                __builtin_nontemporal_store(v.re.v[l], hv + l * a.ld);
                __builtin_nontemporal_store(v.im.v[l], hv + (L + l) * a.ld);
            }
        }
    }
}

int dd_values_launch(const DevTable &tab, const double gamma[2], int64_t npts, const double *t, const double *x,
                     int64_t ld, double *val, int W, int G, hipStream_t st)
{
    ValArgs a;
    a.t = t;
    a.x = x;
    a.val = val;
    a.npts = npts;
    a.ld = ld;
    a.gre = gamma ? gamma[0] : 1.0;
    a.gim = gamma ? gamma[1] : 0.0;
    a.n_eq = tab.n_eq;
    a.n_var = tab.n_var;
    a.planes = tab.dfast_planes;
    const size_t lds = ((size_t)tab.dfast_planes * tab.n_var + 1) * 4 * 512;
    const int64_t tiles = (npts + 63) / 64;
    // four waves per SIMD; staging: about half an equation
    const EvalFit ft = named_tiling(tab.n_eq, W, G, 8, 8, [&](int w) { return values_fit(tab, tiles, w, 16, lds, 0.5); });
    W = ft.W;
    G = ft.G;
    a.eq_stride = G * W;
    hipLaunchKernelGGL(eval_dd_values_kernel, dim3((unsigned)tiles, (unsigned)G), dim3(64 * W), lds, st, a, tab.d_run,
                       tab.mterm, tab.d_deg);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "eval_dd_values_kernel launch");
    return PH_OK;
}

}  // namespace ph
