// ecc_batch.hip -- the batched form: the ECCs of many images of uneven sizes and
// dimensions in one persistent launch.
//
// The host cuts the bricks of all images (in order) into one contiguous run per
// workgroup, balanced by work, and lists each run as segments of single images.
// A workgroup processes its segments in order with the same marching bodies as the
// single-image kernels (ecc_kernels_dt.h), and writes one prefix-summed histogram
// row per segment.  The merge then gives every image the sum of its rows, its ECC,
// without any atomic operation on the histogram bins, so the result of an image
// does not depend on the batch it is in.
#include <algorithm>

#include "ecc_merge.h"

namespace ecc {

namespace {

using namespace dev;

// Min/max keys of AUTO-range images: block (piece, part) folds its part of a
// piece into the image's keys with atomics (the host uploads lo = ~0, hi = 0
// first).  Bound by the read of the images: one block per piece of 2^20 elements,
// loading them one by one, left most of the device idle (16 uint16 images of
// 66 MB together: 1100 us; with the parts and 16-byte loads 26 us).
template <int DT>
__device__ void minmax_part(const BatchImage& I, const BatchPiece& pc, int part, int parts, uint32_t* mm)
{
    using T = typename ValT<DT>::T;
    const int64_t len = pc.end - pc.begin;
    // parts start on whole 16-byte groups of the piece
    const int64_t chunk = ((len + parts - 1) / parts + 15) / 16 * 16;
    const int64_t b = pc.begin + (int64_t)part * chunk;
    const int64_t e = b + chunk < pc.end ? b + chunk : pc.end;
    if (b >= e) return;
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    mm_range<DT, 4>((const T*)I.data, b, e, threadIdx.x, kThreads, lo, hi);
    block_minmax(lo, hi);
    // (reading the keys first and adding only what improves them was slower:
    // 48 us for the pass)
    if (threadIdx.x == 0) {
        atomicMin(&mm[2 * pc.image], lo);
        atomicMax(&mm[2 * pc.image + 1], hi);
    }
}

// Initial min/max keys of every image: lo = ~0, hi = 0.
__global__ __launch_bounds__(kThreads) void k_mm_init(uint32_t* mm, int count)
{
    const int i = blockIdx.x * kThreads + threadIdx.x;
    if (i < count) {
        mm[2 * i] = 0xFFFFFFFFu;
        mm[2 * i + 1] = 0u;
    }
}

__global__ __launch_bounds__(kThreads) void k_minmax_batch(const BatchImage* images, const BatchPiece* pieces,
                                                           uint32_t* mm)
{
    const BatchPiece pc = pieces[blockIdx.x];
    const BatchImage& I = images[pc.image];
    const int part = (int)blockIdx.y, parts = (int)gridDim.y;
    switch (I.dtype) {
    case DT_U8: minmax_part<DT_U8>(I, pc, part, parts, mm); break;
    case DT_U16: minmax_part<DT_U16>(I, pc, part, parts, mm); break;
    default: minmax_part<DT_F32>(I, pc, part, parts, mm); break;
    }
}

// The merge of a batch of many images with few rows each: a thread adds N bins (one
// per kThreads) of its image's rows, four rows at a time, without LDS.  k_merge's
// blocks of 64 bins are launch-bound there: about 1.4 ns each (2000 images of one
// row, 4096 bins: 128000 blocks, 174 us).
template <int N>
__global__ __launch_bounds__(kThreads) void k_merge_rows(MergeArgs A)
{
    constexpr int U = 4;
    const int img = blockIdx.y;
    const int j0 = (int)blockIdx.x * kThreads * N + (int)threadIdx.x;
    const int r0 = A.slot_off[img], r1 = A.slot_off[img + 1];
    int64_t sum[N] = {};
    for (int r = r0; r < r1; r += U) {
        // rows past the last re-read it and are dropped; so are bins past the window
        int32_t x[U][N];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int32_t* row = A.partials + (size_t)A.slots[min(r + u, r1 - 1)] * (size_t)A.row_stride;
#pragma unroll
            for (int n = 0; n < N; ++n) x[u][n] = row[min(j0 + n * kThreads, A.width - 1)];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int n = 0; n < N; ++n) sum[n] += r + u < r1 ? x[u][n] : 0;
    }
    int64_t* out = A.images[img].out + A.bin_lo;
#pragma unroll
    for (int n = 0; n < N; ++n)
        if (j0 + n * kThreads < A.width) out[j0 + n * kThreads] = sum[n];
}

template <int N>
hipError_t launch_merge_rows(const MergeArgs& A, int images, hipStream_t s)
{
    constexpr int bins = kThreads * N;
    hipLaunchKernelGGL((k_merge_rows<N>), dim3((unsigned)((A.width + bins - 1) / bins), (unsigned)images), dim3(kThreads),
                       0, s, A);
    return hipGetLastError();
}

}  // namespace

BatchWork batch_work(BatchImage& im, int construction, int depth3, int depth2, int64_t planes)
{
    const int64_t xpos = axis_positions(im.g.n2, construction);
    const int64_t cols = (xpos + kLaneCols - 1) / kLaneCols;
    // waves per brick: the fraction of kBrickWaves waves' lanes that own a column,
    // (wave columns needed / wave columns covered) x (waves in bricks side by side
    // / waves), is largest (ties: the wider brick)
    int wpb = 1;
    double best_eff = -1.0;
    for (int w = (int)std::min<int64_t>(cols, kBrickWaves); w >= 1; --w) {
        const int64_t nx = (cols + w - 1) / w;
        const double eff = (double)cols / (double)(nx * w) * (double)((kBrickWaves / w) * w) / (double)kBrickWaves;
        if (eff > best_eff + 1e-9) {
            best_eff = eff;
            wpb = w;
        }
    }
    const int64_t chunk = kLaneCols * (int64_t)wpb;
    BatchWork b;
    if (im.ndim == 3) {
        im.units = units_3d(im.g, construction);
        const int64_t nzb = (im.g.n0 + depth3 - 1) / depth3;
        b.bricks = layout_3d(im.g, construction, wpb).per_z * nzb;
        b.brick_voxels = chunk * kRows3 * depth3;
        // the wave tasks' plane blocks share the planes evenly
        const int64_t nb = (im.g.n0 + planes - 1) / planes;
        im.depth = (im.g.n0 + nb - 1) / nb;
        b.steps = (int64_t)im.units.tasks * nb * im.depth;
        // a plane step is about 240 instructions (a pair volume bins twice as
        // much), a task starts with about three steps' worth
        b.cost = (double)im.units.tasks * ((double)im.g.n0 + 3.0 * (double)nb) * (im.data2 ? 300.0 : 240.0);
    } else {
        // whole chunks of rows per brick (the 2D march steps groups of rows)
        const int64_t rows = ((int64_t)(depth2 < 1 ? 1 : depth2) + kChunk2 - 1) / kChunk2 * kChunk2;
        const int64_t nyb = (im.g.n1 + rows - 1) / rows;
        b.bricks = (xpos + chunk - 1) / chunk * nyb;
        b.brick_voxels = chunk * rows;
        // the wave tasks' blocks share the image's rows evenly
        im.depth = ((nyb == 1 ? im.g.n1 : (im.g.n1 + nyb - 1) / nyb) + kChunk2 - 1) / kChunk2 * kChunk2;
        im.units = units_2d(im.g, construction, im.depth);
        b.steps = (int64_t)im.units.tasks * (im.depth / kChunk2);
        // 25 instructions a row, and about 20 rows' worth to start a task
        b.cost = (double)im.units.tasks * ((double)std::min<int64_t>(im.depth, im.g.n1) + 20.0) * 25.0;
    }
    return b;
}

hipError_t launch_minmax_batch(const BatchImage* images, const BatchPiece* pieces, int npieces, uint32_t* mm,
                               hipStream_t s)
{
    if (npieces <= 0) return hipSuccess;
    // parts per piece: about 2048 blocks, at most 32 (parts of 2^15 elements)
    const unsigned parts = (unsigned)std::min(32, std::max(1, 2048 / npieces));
    hipLaunchKernelGGL(k_minmax_batch, dim3((unsigned)npieces, parts), dim3(kThreads), 0, s, images, pieces, mm);
    return hipGetLastError();
}

hipError_t launch_mm_init(uint32_t* mm, int count, hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mm_init, dim3((count + kThreads - 1) / kThreads), dim3(kThreads), 0, s, mm, count);
    return hipGetLastError();
}

hipError_t launch_ecc_batch(const BatchLaunch& B, int construction, hipStream_t s, hipEvent_t t0, hipEvent_t t1)
{
    switch (B.dtype) {
    case DT_U8: return launch_batch_dt<DT_U8>(B, construction, s, t0, t1);
    case DT_U16: return launch_batch_dt<DT_U16>(B, construction, s, t0, t1);
    default: return launch_batch_dt<DT_F32>(B, construction, s, t0, t1);
    }
}

hipError_t launch_merge_batch(const BatchLaunch& B, hipStream_t s)
{
    // A launch takes at most 65535 images: the device reports 65536 blocks at most on
    // the grid's second axis.  (The images on the first axis, the bins on the second:
    // 16 images of 4096 bins 94 instead of 86 us a call; more of them along the third
    // axis, which adds a check to every block: 0.3 us on a single image.)
    constexpr int kMaxImages = 65535;
    for (int64_t i0 = 0; i0 < B.count; i0 += kMaxImages) {
        MergeArgs A = {};
        A.partials = B.partials;
        A.row_stride = B.row_stride;
        A.slot_off = B.slot_off + i0;
        A.slots = B.slots;
        A.images = B.images + i0;
        A.width = B.width;
        A.bin_lo = B.bin_lo;
        A.sign = 1;
        const int n = (int)std::min<int64_t>(B.count - i0, kMaxImages);
        // Up to 16 rows for every image: a thread per bin (16 images of 1000^2, 4096 bins,
        // 16 rows each: 31 and 22 us a launch; 250 of 800^2 194 and 164), or per
        // four bins where that leaves thousands of blocks (2000 of 16^2, 4096 bins: 83
        // and 74).  It adds an image's rows four at a time in turn, about 0.06 us a row,
        // so more of them take blocks of fewer bins (2 images of 500^2, 32 rows: 14.4 with
        // it and 13.6 us; 3 of 64^3, about 170 rows: 23 and 18), unless
        // those are so many that their launch takes longer than the rows (1000 of 16^2
        // and one of 3000^2, 4096 bins: 64 thousand blocks, 132 and 60 us).
        const int64_t blocks = (int64_t)n * ((B.width + 63) / 64);
        hipError_t e;
        if (B.max_rows <= 16 || 44 * (int64_t)B.max_rows <= blocks)
            e = (int64_t)n * B.width > (int64_t(4096) * kThreads) ? launch_merge_rows<4>(A, n, s) : launch_merge_rows<1>(A, n, s);
        else if (B.avg_rows <= 12)
            e = launch_merge_k<4, 64>(A, n, s);
        else
            e = B.width >= kWideMerge ? launch_merge_k<32, 32>(A, n, s) : launch_merge_k<64, 16>(A, n, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace ecc
