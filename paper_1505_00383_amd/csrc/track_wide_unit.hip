// track_wide_unit.hip -- launchers of the tracker kernel that gives a wave to
// one path, for one residual precision L and one solve precision (compiled once
// per pair, like track_unit.hip).
#include "ph_track_wide.hpp"

namespace ph {

template <int L, bool MIXED, int KMAX, int NPSEL>
static int launch_w(const TrackArgs &a, int blocks, size_t lds, hipStream_t st, int *occ)
{
    if (occ) {
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(occ, track_wide_kernel<L, KMAX, MIXED, NPSEL>, 64, lds);
        if (e != hipSuccess) return hip_fail(e, "wide track kernel occupancy");
        return PH_OK;
    }
    hipLaunchKernelGGL((track_wide_kernel<L, KMAX, MIXED, NPSEL>), dim3(blocks), dim3(64), lds, st, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "wide track kernel launch");
    return PH_OK;
}

template <int L, bool MIXED, int NPSEL>
static int launch_wk(const TrackArgs &a, int kmax, int blocks, size_t lds, hipStream_t st, int *occ)
{
    if constexpr (NPSEL < 0)
        if (kmax <= 2) return launch_w<L, MIXED, 2, NPSEL>(a, blocks, lds, st, occ);
    if (kmax <= 4) return launch_w<L, MIXED, 4, NPSEL>(a, blocks, lds, st, occ);
    return launch_w<L, MIXED, 8, NPSEL>(a, blocks, lds, st, occ);
}

template <int L, bool MIXED>
int track_wide_launch_t(const TrackArgs &a, int kmax, int blocks, size_t lds, hipStream_t st, int *occ)
{
    int npmax = 4, classes = 0;
    for (int c = 0; c < 4; ++c)
        if (a.cls[c].total > 0) {
            npmax = a.cls[c].np;
            ++classes;
        }
    if (classes == 1) {
        switch (npmax) {
        case 4: return launch_wk<L, MIXED, -4>(a, kmax, blocks, lds, st, occ);
        case 8: return launch_wk<L, MIXED, -8>(a, kmax, blocks, lds, st, occ);
        case 16: return launch_wk<L, MIXED, -16>(a, kmax, blocks, lds, st, occ);
        default: return launch_wk<L, MIXED, -32>(a, kmax, blocks, lds, st, occ);
        }
    }
    if (npmax <= 16) return launch_wk<L, MIXED, 16>(a, kmax, blocks, lds, st, occ);
    return launch_wk<L, MIXED, 32>(a, kmax, blocks, lds, st, occ);
}

#define PH_WIDE_INSTANTIATE(L_, M_)                                                                   \
    template int track_wide_launch_t<L_, M_>(const TrackArgs &, int, int, size_t, hipStream_t, int *);

#if defined(PH_TRACK_L) && defined(PH_TRACK_MIXED)
PH_WIDE_INSTANTIATE(PH_TRACK_L, (PH_TRACK_MIXED != 0))
#else
PH_WIDE_INSTANTIATE(1, true)
PH_WIDE_INSTANTIATE(2, true)
PH_WIDE_INSTANTIATE(4, true)
PH_WIDE_INSTANTIATE(1, false)
PH_WIDE_INSTANTIATE(2, false)
PH_WIDE_INSTANTIATE(4, false)
#endif

}  // namespace ph
