// ecc_smooth.hip -- separable 13-tap smoothing of a 2D float32 image, the
// smoothing step of the smoothing + ECC pipeline (Sec. 5, "Pipeline").
//
// Rows first, then columns.  Each output is the sum over k = 0..12, in that order
// and starting from 0, of w[k] times the neighbour at offset k - 6 along the axis
// (border pixels repeated), every product and sum rounded once in float32
// (__fmul_rn / __fadd_rn, no fused multiply-add).
//
// One launch when the output does not overlap the input (k_smooth_tile): a
// workgroup loads its tile and a halo of 6 into LDS, filters the tile's rows and
// the 12 halo rows' into a second LDS tile, and that tile's columns into the
// output.  A tile's neighbours read the pixels under its output, so in place the
// two passes are two launches with the intermediate image in memory (rows in ->
// tmp, columns tmp -> out).
#include "ecc_internal.h"

namespace ecc {

namespace {

constexpr int kSmoothThreads = 256;

__global__ __launch_bounds__(kSmoothThreads) void k_smooth_rows(const float* __restrict__ in, float* __restrict__ tmp,
                                                                int64_t n1, int64_t n2, Taps13 w)
{
    __shared__ float tile[kSmoothThreads + 12];
    const int64_t x0 = (int64_t)blockIdx.x * kSmoothThreads;
    const int64_t x = x0 + threadIdx.x;
    for (int64_t y = blockIdx.y; y < n1; y += gridDim.y) {
        const float* row = in + y * n2;
        for (int i = threadIdx.x; i < kSmoothThreads + 12; i += kSmoothThreads) {
            int64_t xi = x0 + i - 6;
            xi = xi < 0 ? 0 : (xi >= n2 ? n2 - 1 : xi);
            tile[i] = row[xi];
        }
        __syncthreads();
        if (x < n2) {
            float acc = 0.0f;
#pragma unroll
            for (int k = 0; k < 13; ++k) acc = __fadd_rn(acc, __fmul_rn(w.w[k], tile[threadIdx.x + k]));
            tmp[y * n2 + x] = acc;
        }
        __syncthreads();
    }
}

__global__ __launch_bounds__(kSmoothThreads) void k_smooth_cols(const float* __restrict__ tmp, float* __restrict__ out,
                                                                int64_t n1, int64_t n2, Taps13 w)
{
    const int64_t x = (int64_t)blockIdx.x * kSmoothThreads + threadIdx.x;
    if (x >= n2) return;
    for (int64_t y = blockIdx.y; y < n1; y += gridDim.y) {
        float acc = 0.0f;
#pragma unroll
        for (int k = 0; k < 13; ++k) {
            int64_t yy = y + k - 6;
            yy = yy < 0 ? 0 : (yy >= n1 ? n1 - 1 : yy);
            acc = __fadd_rn(acc, __fmul_rn(w.w[k], tmp[yy * n2 + x]));
        }
        out[y * n2 + x] = acc;
    }
}

// Tile of k_smooth_tile: 64 x 16 outputs, so 28 rows are filtered along x for 16.
// Taller tiles filter fewer rows twice but keep fewer workgroups on a CU, lower
// ones the other way: 1024^2 6.9, 6.6 and 7.4 us with 8, 16 and 32 rows, 8192^2 347,
// 264 and 301 us (two launches with the intermediate image in memory: 13.1 and 554
// us).  Small images are bound by latency, large ones by vector issue (26
// instructions per output and pass, 4 cycles each).
constexpr int kTileX = 64, kTileY = 16, kHalo = 6;
constexpr int kInX = kTileX + 2 * kHalo, kInY = kTileY + 2 * kHalo;

__global__ __launch_bounds__(kSmoothThreads) void k_smooth_tile(const float* __restrict__ in, float* __restrict__ out,
                                                                int64_t n1, int64_t n2, int64_t tiles_x, int64_t tiles,
                                                                Taps13 w)
{
    __shared__ __align__(16) float src[kInY][kInX];
    __shared__ __align__(16) float mid[kInY][kTileX];
    const int t = (int)threadIdx.x;
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const int64_t ty = tile / tiles_x;
        const int64_t y0 = ty * kTileY, x0 = (tile - ty * tiles_x) * kTileX;
        // a thread keeps its column of the tile (and a quarter of the waves its
        // halo columns), a wave a row
        const int c = t & 63, r0 = t >> 6;
        const int64_t xa = x0 - kHalo + c, xb = xa + 64;
        const int64_t ca = xa < 0 ? 0 : (xa >= n2 ? n2 - 1 : xa), cb = xb >= n2 ? n2 - 1 : xb;
#pragma unroll
        for (int r = r0; r < kInY; r += 4) {
            int64_t y = y0 - kHalo + r;
            y = y < 0 ? 0 : (y >= n1 ? n1 - 1 : y);
            const float* row = in + y * n2;
            src[r][c] = row[ca];
            if (c < kInX - 64) src[r][c + 64] = row[cb];
        }
        __syncthreads();
        // rows: four neighbouring outputs per thread from sixteen pixels
        for (int i = t; i < kInY * (kTileX / 4); i += kSmoothThreads) {
            const int r = i / (kTileX / 4), x = (i % (kTileX / 4)) * 4;
            float p[16];
#pragma unroll
            for (int k = 0; k < 4; ++k) *(float4*)&p[4 * k] = *(const float4*)&src[r][x + 4 * k];
            float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int k = 0; k < 13; ++k)
#pragma unroll
                for (int o = 0; o < 4; ++o) acc[o] = __fadd_rn(acc[o], __fmul_rn(w.w[k], p[o + k]));
            *(float4*)&mid[r][x] = make_float4(acc[0], acc[1], acc[2], acc[3]);
        }
        __syncthreads();
        // columns: four outputs below each other per thread from sixteen values
        const int64_t x = x0 + c;
        const int yb = r0 * (kTileY / 4);
        float p[kTileY / 4 + 12];
#pragma unroll
        for (int k = 0; k < kTileY / 4 + 12; ++k) p[k] = mid[yb + k][c];
        float acc[kTileY / 4] = {};
#pragma unroll
        for (int k = 0; k < 13; ++k)
#pragma unroll
            for (int o = 0; o < kTileY / 4; ++o) acc[o] = __fadd_rn(acc[o], __fmul_rn(w.w[k], p[o + k]));
#pragma unroll
        for (int o = 0; o < kTileY / 4; ++o) {
            const int64_t y = y0 + yb + o;
            if (x < n2 && y < n1) out[y * n2 + x] = acc[o];
        }
        __syncthreads();   // the tiles are read before the next one overwrites them
    }
}

}  // namespace

hipError_t launch_smooth13_tile(const float* in, float* out, int64_t n1, int64_t n2, const Taps13& w, hipStream_t s)
{
    const int64_t tiles_x = (n2 + kTileX - 1) / kTileX, tiles = tiles_x * ((n1 + kTileY - 1) / kTileY);
    const unsigned grid = (unsigned)(tiles < (int64_t(1) << 20) ? tiles : int64_t(1) << 20);
    hipLaunchKernelGGL(k_smooth_tile, dim3(grid), dim3(kSmoothThreads), 0, s, in, out, n1, n2, tiles_x, tiles, w);
    return hipGetLastError();
}

hipError_t launch_smooth13(const float* in, float* out, float* tmp, int64_t n1, int64_t n2, const Taps13& w,
                           hipStream_t s)
{
    const dim3 grid((unsigned)((n2 + kSmoothThreads - 1) / kSmoothThreads), (unsigned)(n1 < 65535 ? n1 : 65535));
    hipLaunchKernelGGL(k_smooth_rows, grid, dim3(kSmoothThreads), 0, s, in, tmp, n1, n2, w);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_smooth_cols, grid, dim3(kSmoothThreads), 0, s, tmp, out, n1, n2, w);
    return hipGetLastError();
}

}  // namespace ecc
