// ecc_kernels_dt.h -- the histogram kernels of one data type, for one image (2D and
// 3D) and for batches, and their launchers.  A source per data type includes it with
// ECC_KERNEL_DT defined (they compile side by side).  The method and its mapping to
// the hardware are described in ecc_device.h and ecc_march.h.
#pragma once

#include <hip/hip_ext.h>

#include "ecc_march.h"

namespace ecc {

namespace {

using namespace dev;

// The kernels take the workgroup's size and the brick counts from the launch arguments:
// the hidden argument that holds the size is a load of its own at every use, the counts
// a 64-bit division, and both stand in the serial chain of a small image (with them and
// with the copies cleared word by word one after the other: 20^3 uint16, 16 bins, 9.6 us
// a call and 8.4 without, 64^2 uint8, 64 bins, 7.8 and 6.9; 256^3 uint8 25.1 and 24.2).

// 3D images.  A workgroup brick is as many consecutive wave tasks (Units: 2 x 63
// slots of kStripRows rows each) as it has waves x L.depth planes.  Its waves read
// neighbouring parts of the same rows at about the same time.
template <int DT, int CONS, bool WIN, bool PAIR>
__global__ __launch_bounds__(kMaxWaves * 64) __attribute__((amdgpu_waves_per_eu(ECC_WAVES_PER_EU_3D))) void k_ecc_3d(EccLaunch L)
{
    extern __shared__ __align__(16) int32_t hist[];
    const uint32_t waves = (uint32_t)L.waves;
    const BinParams P = load_params<DT>(L, waves);
    const HistRef H = march_hist<WIN>(hist, L.width, L.hist_stride, L.hist_copies);
    zero_hist(H, waves);
    const uint32_t per_z = L.per_z;
    for (uint32_t brick = blockIdx.x; brick < L.nbricks; brick += gridDim.x) {
        const uint32_t zb = uniform_u32(brick / per_z), r = uniform_u32(brick - zb * per_z);
        const uint32_t z0 = zb * (uint32_t)L.depth;
        const uint32_t ze = (int64_t)z0 + L.depth < L.z_own ? z0 + (uint32_t)L.depth : (uint32_t)L.z_own;
        const Task3 K = strip_task<DT, CONS, kStripRows>(L.g, L.units, H.sm, r * waves + (uint32_t)wave_id());
        run_march_3d<DT, CONS, kStripRows, WIN, PAIR, !PAIR>(L, P, H, K, z0, ze);
    }
    const size_t row = (size_t)blockIdx.y * gridDim.x + blockIdx.x;
    int32_t* dst = L.partials + row * (size_t)(WIN ? L.row_stride : L.width);
    flush_hist(H, dst, L.width, L.flush_add != 0, L.flush_sign, waves,
               WIN && L.bin_lo > 0 ? dst + L.row_stride - 1 : nullptr);
    if (L.fused) fused_merge(hist, L.partials, L.width, L.out, L.counter, waves);
}

// 2D images.  A workgroup brick is as many consecutive wave tasks (Units: 2 x 63
// slots x L.depth rows each) as it has waves.
template <int DT, int CONS, bool WIN>
__global__ __launch_bounds__(kMaxWaves * 64) __attribute__((amdgpu_waves_per_eu(ECC_WAVES_PER_EU_2D))) void k_ecc_2d(EccLaunch L)
{
    extern __shared__ __align__(16) int32_t hist[];
    const uint32_t waves = (uint32_t)L.waves;
    const BinParams P = load_params<DT>(L, waves);
    const HistRef H = march_hist<WIN>(hist, L.width, L.hist_stride, L.hist_copies);
    zero_hist(H, waves);
    const WinKeys W = win_keys<WIN>(L.bin_lo, L.width);
    for (uint32_t task = blockIdx.x * waves + (uint32_t)wave_id(); task < L.units.tasks; task += gridDim.x * waves)
        run_march_2d<DT, CONS, WIN>(L.data, L.g, L.depth, P, W, H,
                                    block_task<DT, CONS>(L.g, L.units, L.depth, H.sm, task));
    int32_t* dst = L.partials + (size_t)blockIdx.x * (size_t)(WIN ? L.row_stride : L.width);
    flush_hist(H, dst, L.width, L.flush_add != 0, L.flush_sign, waves,
               WIN && L.bin_lo > 0 ? dst + L.row_stride - 1 : nullptr);
    if (L.fused) fused_merge(hist, L.partials, L.width, L.out, L.counter, waves);
}

// Every workgroup takes its segments in turn, their counts to one histogram.  A
// segment is a run of steps (planes, or groups of kChunk2 rows) of the volume's wave
// tasks, numbered task by task; each wave takes an equal part of it.  With whole tasks
// of 8 planes or 128 rows per wave the last round left waves idle and the start-up of
// a task (2.5 planes) was a quarter of its work: 512 uint8 images took 376 us and 338
// with equal parts, 71 float32 images of 4096 bins 146 and 123, 11 uint8 images 31
// and 26.  PAIRS: the launch
// holds pair volumes (their tasks load two hyperplanes).  WAVES per workgroup, as a
// constant (read from the launch it costs the 512-image batch 5%).
template <int DT, int CONS, bool WIN, bool PAIRS, int WAVES>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(ECC_WAVES_PER_EU_BATCH)))
void k_ecc_batch(BatchLaunch B)
{
    extern __shared__ __align__(16) int32_t hist[];
    const HistRef H = march_hist<WIN>(hist, B.width, B.hist_stride, B.hist_copies);
    const WinKeys W = win_keys<WIN>(B.bin_lo, B.width);
    const int s_end = B.wg_seg[blockIdx.x + 1];
    for (int si = B.wg_seg[blockIdx.x]; si < s_end; ++si) {
        // The tables are read with vector loads (the kernel also writes global
        // memory, so the scalar cache is not used for them): every value the
        // marching bodies depend on is read back from the first lane, so that
        // sizes, offsets and pointers stay in scalar registers there.
        const BatchSeg S = B.segs[si];
        const int vol = (int)uniform_u32((uint32_t)S.image);
        const BatchImage& I = B.images[vol];
        const BinParams P = uniform_params<DT>(
            I.auto_range ? params_from_keys(B.mm[2 * I.owner], B.mm[2 * I.owner + 1], DT, B.nbins) : I.params);
        EccLaunch L;   // the fields the marching bodies read
        L.data = uniform_ptr(I.data);
        L.data2 = PAIRS ? uniform_ptr(I.data2) : nullptr;
        L.g = Geom{uniform_i64(I.g.n0), uniform_i64(I.g.n1), uniform_i64(I.g.n2)};
        L.depth = uniform_i64(I.depth);
        L.z_base = 0;
        L.pass_stride = 0;
        L.n0_global = L.g.n0;
        L.bin_lo = B.bin_lo;
        L.width = B.width;
        const Units Y = {uniform_u32(I.units.slots), uniform_u32(I.units.sa), uniform_u32(I.units.sb),
                         uniform_u32(I.units.pairs_full), uniform_u32(I.units.pairs_edge),
                         uniform_u32(I.units.tasks)};
        const int ndim = (int)uniform_u32((uint32_t)I.ndim);
        zero_hist_words(H, B.width);
        // steps of a wave task: groups of rows (2D), planes (3D)
        const int64_t len = ndim == 2 ? L.depth / kChunk2 : L.depth;
        const int64_t b0 = uniform_i64(S.b0), steps = uniform_i64(S.b1) - b0;
        int64_t a = b0 + steps * wave_id() / WAVES;
        const int64_t e = b0 + steps * (wave_id() + 1) / WAVES;
        while (a < e) {
            const int64_t task = uniform_i64((a >> 32) == 0 ? (int64_t)((uint32_t)a / (uint32_t)len) : a / len);
            const uint32_t s0 = uniform_u32((uint32_t)(a - task * len));
            const uint32_t s1 = (int64_t)s0 + (e - a) < len ? s0 + (uint32_t)(e - a) : (uint32_t)len;
            if (ndim == 2) {
                const uint32_t row_bytes = (uint32_t)L.g.n2 * (uint32_t)sizeof(typename ValT<DT>::T);
                const Task2 K = block_part(block_task<DT, CONS>(L.g, Y, L.depth, H.sm, (uint32_t)task), L.g, L.depth,
                                           row_bytes, s0 * kChunk2, s1 * kChunk2);
                run_march_2d<DT, CONS, WIN>(L.data, L.g, (int64_t)(s1 - s0) * kChunk2, P, W, H, K);
            } else {
                // tasks are numbered plane block by plane block
                const uint32_t zb = uniform_u32((uint32_t)task / Y.tasks);
                const Task3 K = strip_task<DT, CONS, kStripRows>(L.g, Y, H.sm, (uint32_t)task - zb * Y.tasks);
                const int64_t z0 = (int64_t)zb * L.depth + s0, z1 = (int64_t)zb * L.depth + s1;
                const uint32_t ze = (uint32_t)(z1 < L.g.n0 ? z1 : L.g.n0);
                // (the last block may have fewer planes)
                if (z0 < L.g.n0) {
                    if (PAIRS && L.data2) run_march_3d<DT, CONS, kStripRows, WIN, true>(L, P, H, K, (uint32_t)z0, ze);
                    else run_march_3d<DT, CONS, kStripRows, WIN, false>(L, P, H, K, (uint32_t)z0, ze);
                }
            }
            a += s1 - s0;
        }
        const size_t slot = (size_t)uniform_u32((uint32_t)S.slot);
        int32_t* dst = B.partials + slot * (size_t)(WIN ? B.row_stride : B.width);
        flush_hist(H, dst, B.width, false, (int)uniform_u32((uint32_t)I.sign), blockDim.x >> 6,
                   WIN && B.bin_lo > 0 ? dst + B.row_stride - 1 : nullptr);
        __syncthreads();   // the histogram is read before the next segment clears it
    }
}

// ----------------------------------------------------------------- launchers

template <class K>
inline hipError_t launch_k(K kernel, const EccLaunch& L, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    const dim3 grid((unsigned)L.grid, (unsigned)(L.npass > 1 ? L.npass : 1));
    if (t0 || t1)
        hipExtLaunchKernelGGL(kernel, grid, dim3(L.waves * 64), L.lds_bytes, s, t0, t1, 0, L);
    else
        hipLaunchKernelGGL(kernel, grid, dim3(L.waves * 64), L.lds_bytes, s, L);
    return hipGetLastError();
}

template <int NDIM, int DT, int CONS, bool WIN>
inline hipError_t launch_t(const EccLaunch& L, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    if constexpr (NDIM == 2) return launch_k(k_ecc_2d<DT, CONS, WIN>, L, s, t0, t1);
    else if (L.data2) return launch_k(k_ecc_3d<DT, CONS, WIN, true>, L, s, t0, t1);
    else return launch_k(k_ecc_3d<DT, CONS, WIN, false>, L, s, t0, t1);
}

template <int NDIM, int DT, int CONS>
inline hipError_t launch_w(const EccLaunch& L, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    return L.windowed ? launch_t<NDIM, DT, CONS, true>(L, s, t0, t1) : launch_t<NDIM, DT, CONS, false>(L, s, t0, t1);
}

template <int NDIM, int DT>
inline hipError_t launch_c(const EccLaunch& L, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    return L.construction == CONS_TOP ? launch_w<NDIM, DT, CONS_TOP>(L, s, t0, t1)
                                      : launch_w<NDIM, DT, CONS_VERTEX>(L, s, t0, t1);
}

template <int NDIM, int DT, int CONS, bool WIN>
inline const void* kernel_of()
{
    if constexpr (NDIM == 2) return (const void*)k_ecc_2d<DT, CONS, WIN>;
    else return (const void*)k_ecc_3d<DT, CONS, WIN, false>;
}

template <int NDIM, int DT, int CONS>
inline const void* kernel_w(bool win)
{
    return win ? kernel_of<NDIM, DT, CONS, true>() : kernel_of<NDIM, DT, CONS, false>();
}

template <int NDIM, int DT>
inline const void* kernel_c(int cons, bool win)
{
    return cons == CONS_TOP ? kernel_w<NDIM, DT, CONS_TOP>(win) : kernel_w<NDIM, DT, CONS_VERTEX>(win);
}

template <class K>
hipError_t launch_batch_k(K kernel, const BatchLaunch& B, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    if (t0 || t1)
        hipExtLaunchKernelGGL(kernel, dim3(B.grid), dim3(B.waves * 64), B.lds_bytes, s, t0, t1, 0, B);
    else
        hipLaunchKernelGGL(kernel, dim3(B.grid), dim3(B.waves * 64), B.lds_bytes, s, B);
    return hipGetLastError();
}

template <int DT, int CONS, bool PAIRS>
hipError_t launch_batch_p(const BatchLaunch& B, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    constexpr int N = kBatchWaves;
    if constexpr (!PAIRS)   // 16 waves only there (build_batch_tables)
        if (!B.windowed && B.waves > N)
            return launch_batch_k(k_ecc_batch<DT, CONS, false, false, kMaxWaves>, B, s, t0, t1);
    return B.windowed ? launch_batch_k(k_ecc_batch<DT, CONS, true, PAIRS, N>, B, s, t0, t1)
                      : launch_batch_k(k_ecc_batch<DT, CONS, false, PAIRS, N>, B, s, t0, t1);
}

template <int DT, int CONS>
hipError_t launch_batch_w(const BatchLaunch& B, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    return B.pairs ? launch_batch_p<DT, CONS, true>(B, s, t0, t1) : launch_batch_p<DT, CONS, false>(B, s, t0, t1);
}

}  // namespace

template <>
hipError_t launch_ecc_dt<ECC_KERNEL_DT>(const EccLaunch& L, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    return L.ndim == 2 ? launch_c<2, ECC_KERNEL_DT>(L, s, t0, t1) : launch_c<3, ECC_KERNEL_DT>(L, s, t0, t1);
}

template <>
const void* kernel_dt<ECC_KERNEL_DT>(int ndim, int construction, bool windowed)
{
    return ndim == 2 ? kernel_c<2, ECC_KERNEL_DT>(construction, windowed)
                     : kernel_c<3, ECC_KERNEL_DT>(construction, windowed);
}

template <>
hipError_t launch_batch_dt<ECC_KERNEL_DT>(const BatchLaunch& B, int construction, hipStream_t s, hipEvent_t t0,
                                          hipEvent_t t1)
{
    return construction == CONS_TOP ? launch_batch_w<ECC_KERNEL_DT, CONS_TOP>(B, s, t0, t1)
                                    : launch_batch_w<ECC_KERNEL_DT, CONS_VERTEX>(B, s, t0, t1);
}

}  // namespace ecc
