// ecc_merge.h -- the merge of workgroup histograms, one launch for one image or a
// batch.  The rows are prefix-summed already (flush_hist), and the prefix sum of a
// sum of histograms is the sum of their prefix sums, so the merge of the rows is the
// ECC (Sec. 2.3: the prefix sum of the VCEC): no block depends on another one.
//
// Block (b, image) sums the image's rows for BB bins: RG groups of BB threads take
// the rows in turn, sixteen rows loaded before they are added, and meet in LDS.
// Bound by latency, one round of loads for up to 16 RG rows.  With rows of plain
// counts the merge took two launches (sums of row groups, then totals and scan: 5.2
// + 5.8 us on 484 rows of 4096 bins, 4.9 + 3.8 us on 989 rows of 256), and one launch
// whose blocks waited for each other's totals 9.8 and 8.3 us; this one takes
// 7.0 and 6.6 us.
#pragma once

#include "ecc_device.h"

namespace ecc {
namespace dev {

template <int RG, int BB>
__global__ __launch_bounds__(RG * BB) void k_merge(MergeArgs A)
{
    static_assert(BB <= 64 && RG * BB <= 1024 && (RG * BB) % 64 == 0, "whole waves, bins within one");
    constexpr int U = 16, W = RG * BB / 64;
    __shared__ int64_t red[W][BB];
    const int img = blockIdx.y;
    const int c = (int)threadIdx.x % BB, g = (int)threadIdx.x / BB;
    const int j = (int)blockIdx.x * BB + c;
    int r0 = 0, r1 = A.rows;
    if (A.slots) {
        r0 = A.slot_off[img];
        r1 = A.slot_off[img + 1];
    }
    // rows past the last re-read it and are dropped; so are bins past the window
    const int32_t* col = A.partials + min(j, A.width - 1);
    int64_t sum = 0;
    for (int r = r0 + g; r < r1; r += RG * U) {
        int32_t x[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = min(r + u * RG, r1 - 1);
            x[u] = col[(size_t)(A.slots ? A.slots[k] : k) * (size_t)A.row_stride];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) sum += r + u * RG < r1 ? x[u] : 0;
    }
    // the groups within a wave, then the waves
#pragma unroll
    for (int off = BB; off < 64; off <<= 1) sum += __shfl_xor(sum, off, 64);
    if ((int)(threadIdx.x & 63) < BB) red[threadIdx.x >> 6][c] = sum;
    __syncthreads();
    if ((int)threadIdx.x >= BB || j >= A.width) return;
    int64_t v = 0;
#pragma unroll
    for (int k = 0; k < W; ++k) v += red[k][c];
    int64_t* out = (A.images ? A.images[img].out : A.out) + A.bin_lo + j;
    *out = (A.accumulate ? *out : 0) + (A.sign < 0 ? -v : v);
}

template <int RG, int BB>
inline hipError_t launch_merge_k(const MergeArgs& A, int images, hipStream_t s)
{
    hipLaunchKernelGGL((k_merge<RG, BB>), dim3((unsigned)((A.width + BB - 1) / BB), (unsigned)images), dim3(RG * BB), 0,
                       s, A);
    return hipGetLastError();
}

}  // namespace dev
}  // namespace ecc
