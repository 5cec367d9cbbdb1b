// ecc_kernels.hip -- the histogram kernels of the ECC library for one image (2D
// and 3D) and their launchers.  The method and its mapping to the hardware are
// described in ecc_device.h; the min/max pass and the merge are in
// ecc_reduce.hip.
#include <map>
#include <mutex>
#include <tuple>

#include <hip/hip_ext.h>

#include "ecc_march.h"

namespace ecc {

namespace {

using namespace dev;

// 3D images.  A workgroup brick is as many consecutive wave tasks (Units: 2 x 63
// slots of kStripRows rows each) as it has waves x L.depth planes.  Its waves read
// neighbouring parts of the same rows at about the same time.
template <int DT, int CONS, bool WIN, bool PAIR>
__global__ __launch_bounds__(kMaxWaves * 64) __attribute__((amdgpu_waves_per_eu(ECC_WAVES_PER_EU_3D))) void k_ecc_3d(EccLaunch L)
{
    extern __shared__ __align__(16) int32_t hist[];
    const BinParams P = load_params<DT>(L);
    const HistRef H = march_hist<WIN>(hist, L.width, L.hist_stride, L.hist_copies);
    zero_hist(H, L.width);
    const uint32_t waves = blockDim.x >> 6;
    const uint32_t per_z = (L.units.tasks + waves - 1u) / waves;
    const uint32_t nbricks = per_z * (uint32_t)((L.z_own + L.depth - 1) / L.depth);
    for (uint32_t brick = blockIdx.x; brick < nbricks; brick += gridDim.x) {
        const uint32_t zb = uniform_u32(brick / per_z), r = uniform_u32(brick - zb * per_z);
        const uint32_t z0 = zb * (uint32_t)L.depth;
        const uint32_t ze = (int64_t)z0 + L.depth < L.z_own ? z0 + (uint32_t)L.depth : (uint32_t)L.z_own;
        const Task3 K = strip_task<DT, CONS, kStripRows>(L.g, L.units, H.sm, r * waves + (uint32_t)wave_id());
        run_march_3d<DT, CONS, kStripRows, WIN, PAIR>(L, P, H, K, z0, ze);
    }
    const size_t row = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
    flush_hist(H, L.partials + row * (size_t)L.width, L.width, L.flush_add != 0, L.flush_sign, WIN ? L.carry + row : nullptr,
               L.bin_lo == 0);
    if (L.fused) fused_merge(hist, L.partials, L.width, L.out, L.counter);
}

// 2D images.  A workgroup brick is as many consecutive wave tasks (Units: 2 x 63
// slots x L.depth rows each) as it has waves.
template <int DT, int CONS, bool WIN>
__global__ __launch_bounds__(kMaxWaves * 64) __attribute__((amdgpu_waves_per_eu(ECC_WAVES_PER_EU_2D))) void k_ecc_2d(EccLaunch L)
{
    extern __shared__ __align__(16) int32_t hist[];
    const BinParams P = load_params<DT>(L);
    const HistRef H = march_hist<WIN>(hist, L.width, L.hist_stride, L.hist_copies);
    zero_hist(H, L.width);
    const uint32_t waves = blockDim.x >> 6;
    const WinKeys W = win_keys<WIN>(L.bin_lo, L.width);
    for (uint32_t task = blockIdx.x * waves + (uint32_t)wave_id(); task < L.units.tasks; task += gridDim.x * waves)
        run_march_2d<DT, CONS, WIN>(L.data, L.g, L.depth, P, W, H,
                                    block_task<DT, CONS>(L.g, L.units, L.depth, H.sm, task));
    flush_hist(H, L.partials + (size_t)blockIdx.x * (size_t)L.width, L.width, L.flush_add != 0, L.flush_sign,
               WIN ? L.carry + blockIdx.x : nullptr, L.bin_lo == 0);
    if (L.fused) fused_merge(hist, L.partials, L.width, L.out, L.counter);
}

}  // namespace

// ----------------------------------------------------------------- launchers


int64_t wg_bricks(int ndim, int construction, const Geom& g, int waves, int64_t depth)
{
    if (ndim == 2) return ((int64_t)units_2d(g, construction, depth).tasks + waves - 1) / waves;
    return ((int64_t)units_3d(g, construction).tasks + waves - 1) / waves * ((g.n0 + depth - 1) / depth);
}

template <class K>
static hipError_t launch_k(K kernel, const EccLaunch& L, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    const dim3 grid((unsigned)L.grid, (unsigned)(L.npass > 1 ? L.npass : 1));
    if (t0 || t1)
        hipExtLaunchKernelGGL(kernel, grid, dim3(L.waves * 64), L.lds_bytes, s, t0, t1, 0, L);
    else
        hipLaunchKernelGGL(kernel, grid, dim3(L.waves * 64), L.lds_bytes, s, L);
    return hipGetLastError();
}

template <int NDIM, int DT, int CONS, bool WIN>
static hipError_t launch_t(const EccLaunch& L, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    if constexpr (NDIM == 2) return launch_k(k_ecc_2d<DT, CONS, WIN>, L, s, t0, t1);
    else if (L.data2) return launch_k(k_ecc_3d<DT, CONS, WIN, true>, L, s, t0, t1);
    else return launch_k(k_ecc_3d<DT, CONS, WIN, false>, L, s, t0, t1);
}

template <int NDIM, int DT, int CONS>
static hipError_t launch_w(const EccLaunch& L, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    return L.windowed ? launch_t<NDIM, DT, CONS, true>(L, s, t0, t1) : launch_t<NDIM, DT, CONS, false>(L, s, t0, t1);
}

template <int NDIM, int DT>
static hipError_t launch_c(const EccLaunch& L, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    return L.construction == CONS_TOP ? launch_w<NDIM, DT, CONS_TOP>(L, s, t0, t1)
                                      : launch_w<NDIM, DT, CONS_VERTEX>(L, s, t0, t1);
}

template <int NDIM>
static hipError_t launch_d(const EccLaunch& L, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    switch (L.dtype) {
    case DT_U8: return launch_c<NDIM, DT_U8>(L, s, t0, t1);
    case DT_U16: return launch_c<NDIM, DT_U16>(L, s, t0, t1);
    default: return launch_c<NDIM, DT_F32>(L, s, t0, t1);
    }
}

hipError_t launch_ecc(const EccLaunch& L, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    return L.ndim == 2 ? launch_d<2>(L, s, t0, t1) : launch_d<3>(L, s, t0, t1);
}

template <int NDIM, int DT, int CONS, bool WIN>
static const void* kernel_of()
{
    if constexpr (NDIM == 2) return (const void*)k_ecc_2d<DT, CONS, WIN>;
    else return (const void*)k_ecc_3d<DT, CONS, WIN, false>;
}

template <int NDIM, int DT, int CONS>
static const void* kernel_w(bool win)
{
    return win ? kernel_of<NDIM, DT, CONS, true>() : kernel_of<NDIM, DT, CONS, false>();
}

template <int NDIM, int DT>
static const void* kernel_c(int cons, bool win)
{
    return cons == CONS_TOP ? kernel_w<NDIM, DT, CONS_TOP>(win) : kernel_w<NDIM, DT, CONS_VERTEX>(win);
}

template <int NDIM>
static const void* kernel_d(int dtype, int cons, bool win)
{
    switch (dtype) {
    case DT_U8: return kernel_c<NDIM, DT_U8>(cons, win);
    case DT_U16: return kernel_c<NDIM, DT_U16>(cons, win);
    default: return kernel_c<NDIM, DT_F32>(cons, win);
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
    const void* k = ndim == 2 ? kernel_d<2>(dtype, construction, windowed) : kernel_d<3>(dtype, construction, windowed);
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, waves * 64, lds) != hipSuccess || n < 1) n = 1;
    cache[key] = n;
    return n;
}


}  // namespace ecc
