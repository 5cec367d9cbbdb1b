// ecc_kernels.hip -- the launchers of the single-image histogram kernels (compiled
// per data type, ecc_kernels_dt.h) and what the host needs to know about them.
#include <map>
#include <mutex>
#include <tuple>

#include "ecc_internal.h"

namespace ecc {

int64_t wg_bricks(int ndim, int construction, const Geom& g, int waves, int64_t depth)
{
    if (ndim == 2) return ((int64_t)units_2d(g, construction, depth).tasks + waves - 1) / waves;
    return ((int64_t)units_3d(g, construction).tasks + waves - 1) / waves * ((g.n0 + depth - 1) / depth);
}

hipError_t launch_ecc(const EccLaunch& L, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    switch (L.dtype) {
    case DT_U8: return launch_ecc_dt<DT_U8>(L, s, t0, t1);
    case DT_U16: return launch_ecc_dt<DT_U16>(L, s, t0, t1);
    default: return launch_ecc_dt<DT_F32>(L, s, t0, t1);
    }
}

int resident_wgs_per_cu(int ndim, int dtype, int construction, bool windowed, int waves, uint32_t lds_bytes)
{
    // the answer only depends on the LDS in steps of the allocation granule
    static std::mutex mu;
    static std::map<std::tuple<int, int, int, int, int, uint32_t>, int> cache;
    const uint32_t lds = (lds_bytes + 511u) / 512u * 512u;
    const auto key = std::make_tuple(ndim == 3, dtype, construction == CONS_TOP, windowed ? 1 : 0, waves, lds);
    std::lock_guard<std::mutex> lock(mu);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    const void* k = dtype == DT_U8    ? kernel_dt<DT_U8>(ndim, construction, windowed)
                    : dtype == DT_U16 ? kernel_dt<DT_U16>(ndim, construction, windowed)
                                      : kernel_dt<DT_F32>(ndim, construction, windowed);
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, waves * 64, lds) != hipSuccess || n < 1) n = 1;
    cache[key] = n;
    return n;
}


}  // namespace ecc
