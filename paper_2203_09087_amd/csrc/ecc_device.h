// ecc_device.h -- device-side building blocks shared by the single-image and
// the batched kernels (binning, histograms, wave helpers).  The marching bodies
// are in ecc_march.h.
//
// What is computed (Wang, Wagner, Chen, SoCG 2022):
//   VCEC[j] = sum over cells of the cubical complex whose value has bin j of
//             (-1)^dim  (Sec. 2.3), and the ECC is its prefix sum (Eq. (1)).
//
// How the cells are counted here.  A cell of a d-dimensional cubical complex is
// a product of one choice per axis: a single position or a pair of adjacent
// positions.  Vertex filtration (voxels are vertices, a cell takes the largest
// value of its voxels): a single is one voxel index k (dimension 0 along the
// axis), a pair the edge {k, k+1} (dimension 1).  Top filtration (the paper's,
// Sec. 2.1: voxels are top cells, a face takes the smallest value of the voxels
// that contain it): a single is the voxel interval k (dimension 1), a pair the
// lattice point between voxels k-1 and k with voxel set {k-1, k} (dimension 0),
// the points before the first and after the last voxel included (their outside
// voxel is ignored).  Fix the choices on all axes but the first ("the marching
// axis") and take, at every position p of that axis, the max (vertex) or min
// (top) over the chosen voxels: a "type function" C(p).  The cells of that type
// are the 1D complex of C along the marching axis with an overall sign
// (-1)^(number of pairs) (vertex) or (-1)^(number of singles) (top), and a 1D
// complex is counted by crediting each interval {p, p+1} to the position that
// attains its value: position p adds +-(1 - [p wins its left interval] -
// [p wins its right interval]) at C(p) (vertex; the top filtration's points are
// credited the same way, with -1 for the voxel itself).  Both reduce to
//     count(p) = d(p) - d(p-1),   d(p) = -[C(p) > C(p+1)] = sign bit of C(p+1) - C(p),
// with C beyond the image = the sentinel and d(-1) = -1 (vertex ties go to the
// later position, top ties to the earlier one; the VCEC does not depend on
// either, since an interval's value is that of whichever position attains it).
// 3D: the marching axis is z and the types are the four choices in (y, x),
// two per axis; 2D: the marching axis is y and the types are the two in x.
// Nothing is compared position by position and no per-voxel cell logic remains:
// a type function is one max/min (the right neighbour through a DPP lane move), a
// count a comparison and a subtraction.  How the counts reach the histogram and how
// the waves divide an image is in ecc_march.h.
#pragma once

#include "ecc_internal.h"

namespace ecc {
namespace dev {


constexpr int kThreads = 256;

// ------------------------------------------------------------------ binning
//
// The kernels compare KEYS, the bins themselves (windows: the bins clamped to the
// window, ecc_march.h): the order is that of the bins.

template <int DT> struct ValT;
template <> struct ValT<DT_U8> { using T = uint8_t; };
template <> struct ValT<DT_U16> { using T = uint16_t; };
template <> struct ValT<DT_F32> { using T = float; };

// Bin of one value.
template <int DT>
__device__ __forceinline__ uint32_t bin_of(typename ValT<DT>::T v, const BinParams& p)
{
    if constexpr (DT == DT_F32) {
        // clamp(floor(((double)x - lo) * scale), 0, nbins-1) without branches:
        // fmin maps NaN to nbins-1, and the saturating conversion clamps below.  A flat range
        // (hi == lo) carries scale = +inf and base = the next double above lo, so
        // x <= lo gives -inf -> 0, x > lo gives +inf or 0*inf = NaN -> nbins-1.
        const float x = v;
        double t = __dmul_rn(__dsub_rn((double)x, p.base), p.scale);
        t = __builtin_fmin(t, (double)(p.nbins - 1));
        // the conversion saturates: negative values and -inf give 0
        uint32_t b;
        asm("v_cvt_u32_f64 %0, %1" : "=v"(b) : "v"(t));
        return b;
    } else {
        const uint32_t a = min(max((uint32_t)v, p.ilo), p.ihi) - p.ilo;
        // floor(a * nbins / D): a * nbins < 2^32 is exact in double, and rcp is
        // 1/D rounded up, so the product never falls below an integer it should
        // reach and stays below the next one (a < D <= 65536).
        const uint32_t n = __umul24(a, (uint32_t)p.nbins);
        return (uint32_t)__dmul_rn((double)n, p.rcp);
    }
}

// Binning parameters from the min/max keys of an image (AUTO range).  Keys are
// order-preserving: integers as themselves, finite floats through the sign-flip
// map; lo_key > hi_key means no (finite) value was seen, which gives [0, 0].
__device__ __forceinline__ double key_to_double(uint32_t k, int dtype)
{
    if (dtype != DT_F32) return (double)k;
    const uint32_t u = (k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k;
    return (double)__uint_as_float(u);
}

__device__ __forceinline__ BinParams params_from_keys(uint32_t lo_key, uint32_t hi_key, int dtype, int32_t nbins)
{
    BinParams p = {};
    p.dtype = dtype;
    p.nbins = nbins;
    const bool empty = lo_key > hi_key;
    const double dlo = empty ? 0.0 : key_to_double(lo_key, dtype);
    const double dhi = empty ? 0.0 : key_to_double(hi_key, dtype);
    if (dtype == DT_F32) {
        p.flat = (dhi == dlo) ? 1 : 0;
        p.scale = p.flat ? __builtin_inf() : __ddiv_rn((double)nbins, __dsub_rn(dhi, dlo));
        // next double above lo (lo is finite): the subtrahend of a flat range
        const double up = dlo == 0.0 ? __longlong_as_double(1ll)
                                     : __longlong_as_double(__double_as_longlong(dlo) + (dlo > 0.0 ? 1 : -1));
        p.base = p.flat ? up : dlo;
    } else {
        const uint32_t ilo = (uint32_t)dlo, ihi = (uint32_t)dhi;
        const uint32_t D = ihi - ilo + 1u;
        p.ilo = ilo;
        p.ihi = ihi;
        p.ident = (uint32_t)nbins == D ? (ilo == 0u ? kIdentRaw : kIdentLevel) : 0;   // every value lies in the range
        // 1/D rounded up: one step above the correctly rounded quotient
        p.rcp = __longlong_as_double(__double_as_longlong(__ddiv_rn(1.0, (double)D)) + 1);
    }
    return p;
}

// Folds one value into running min/max keys (non-finite floats are skipped).
template <int DT>
__device__ __forceinline__ void mm_take(typename ValT<DT>::T v, uint32_t& lo, uint32_t& hi)
{
    if constexpr (DT == DT_F32) {
        const uint32_t u = __float_as_uint(v);
        const uint32_t k = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
        const bool fin = (u & 0x7F800000u) != 0x7F800000u;
        lo = fin ? min(lo, k) : lo;
        hi = fin ? max(hi, k) : hi;
    } else {
        const uint32_t k = (uint32_t)v;
        lo = min(lo, k);
        hi = max(hi, k);
    }
}

// Folds elements [b, e) of img into running min/max keys, thread tid of nthreads:
// 16-byte loads, U in flight, the unaligned head and the tail element by element.
template <int DT, int U>
__device__ __forceinline__ void mm_range(const typename ValT<DT>::T* __restrict__ img, int64_t b, int64_t e,
                                         int64_t tid, int64_t nthreads, uint32_t& lo, uint32_t& hi)
{
    using T = typename ValT<DT>::T;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int PER = 16 / (int)sizeof(T);
    const int64_t n = e - b;
    img += b;
    int64_t head = (int64_t)(((16 - ((uintptr_t)img & 15)) & 15) / sizeof(T));
    if (head > n) head = n;
    for (int64_t i = tid; i < head; i += nthreads) mm_take<DT>(img[i], lo, hi);
    const int64_t nvec = (n - head) / PER;
    const u32x4* __restrict__ vec = (const u32x4*)(img + head);
    int64_t i = tid;
    for (; U > 1 && i + (U - 1) * nthreads < nvec; i += U * nthreads) {
        u32x4 w[U];
#pragma unroll
        for (int u = 0; u < U; ++u) w[u] = __builtin_nontemporal_load(vec + i + u * nthreads);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const T* x = (const T*)&w[u];
#pragma unroll
            for (int k = 0; k < PER; ++k) mm_take<DT>(x[k], lo, hi);
        }
    }
    for (; i < nvec; i += nthreads) {
        const u32x4 w = __builtin_nontemporal_load(vec + i);
        const T* x = (const T*)&w;
#pragma unroll
        for (int k = 0; k < PER; ++k) mm_take<DT>(x[k], lo, hi);
    }
    for (int64_t j = head + nvec * PER + tid; j < n; j += nthreads) mm_take<DT>(img[j], lo, hi);
}

// Block-wide min/max of (lo, hi); the result is valid in thread 0.
__device__ __forceinline__ void block_minmax(uint32_t& lo, uint32_t& hi)
{
    __shared__ uint32_t slo[kThreads], shi[kThreads];
    slo[threadIdx.x] = lo;
    shi[threadIdx.x] = hi;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) {
            slo[threadIdx.x] = min(slo[threadIdx.x], slo[threadIdx.x + s]);
            shi[threadIdx.x] = max(shi[threadIdx.x], shi[threadIdx.x + s]);
        }
        __syncthreads();
    }
    lo = slo[0];
    hi = shi[0];
}

// ------------------------------------------------------------ wave helpers

__device__ __forceinline__ uint32_t lane_id() { return __lane_id(); }

// lane i <- lane i+1 (lane 63 gets 0; it owns no position)
__device__ __forceinline__ uint32_t from_right(uint32_t v)
{
    return __builtin_amdgcn_mov_dpp(v, 0x130 /* wave_shl:1 */, 0xF, 0xF, true);
}

// ---------------------------------------------------------- type functions

struct HistRef {
    int32_t* hist;     // LDS: `copies` copies of the window's counters, `stride` words apart
    uint32_t span;     // counters of the window
    uint32_t copy;     // LDS address of this lane's copy
    uint32_t stride;   // words from one copy to the next
    uint32_t sm;       // the sentinel key: above every key of the window
    uint32_t copies;   // copies (a power of two; lane l adds to copy l mod copies)
    uint32_t first;    // word of the window's first counter in a copy (0, or 1 after a spare word)
};

// True in every thread of the block that is the last of `total` to arrive.  Every
// wave waits until its own stores have reached the L2 (the barrier alone does not
// make it), then one wave writes the L2 back for all of them.  The write-back is what
// a small call pays for, and it runs once per fence: with a fence in every wave a
// workgroup of four paid four of them (64^2 float32, 300 bins, 8.5 us a call and
// 7.8 so; 256^2 uint8 9.4 and 8.5).
__device__ __forceinline__ bool last_to_arrive(uint32_t* counter, uint32_t total)
{
    __shared__ bool last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        last = atomicAdd(counter, 1u) == total - 1;
    }
    __syncthreads();
    if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return last;
}

// Merge of a small single-window launch inside the histogram kernel: the last
// workgroup to finish (all partial rows written and fenced) sums the prefix-summed
// rows into the ECC, then re-arms the counter.  It saves the merge launch where the
// rows are few enough for one workgroup.
__device__ __forceinline__ void fused_merge(int32_t* hist, const int32_t* partials, int width, int64_t* out,
                                            uint32_t* counter, uint32_t waves)
{
    const int rows = (int)(gridDim.x * gridDim.y);
    if (!last_to_arrive(counter, (uint32_t)rows)) return;
    // the rows as one flat array, 16 loads in flight per thread, added with LDS
    // atomics into int64 counters (the histogram's space, free after the flush);
    // element i adds to bin i mod width (tracked incrementally)
    const int bd = (int)(waves * 64u), t = (int)threadIdx.x;
    uint64_t* acc = reinterpret_cast<uint64_t*>(hist);
    for (int j = t; j < width; j += bd) acc[j] = 0;
    __syncthreads();
    constexpr int U = 16;
    const int total = rows * width;
    const int step = bd % width;
    int j = t % width;
    for (int i0 = t; i0 < total; i0 += bd * U) {
        int32_t x[U];
#pragma unroll
        for (int k = 0; k < U; ++k) x[k] = partials[min(i0 + k * bd, total - 1)];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (i0 + k * bd < total && x[k] != 0)
                atomicAdd((unsigned long long*)&acc[j], (unsigned long long)(int64_t)x[k]);
            j += step;
            if (j >= width) j -= width;
        }
    }
    __syncthreads();
    for (int b = t; b < width; b += bd) out[b] = (int64_t)acc[b];
    if (t == 0) atomicExch(counter, 0u);
}

// ------------------------------------------------------------ main kernels

// Clears every copy (the words between them too), 16 bytes a store: the array starts on
// 16 bytes and the copies are a multiple of 8 words apart.  waves: of the workgroup.
__device__ __forceinline__ void zero_hist(const HistRef& H, uint32_t waves)
{
    uint4* h = reinterpret_cast<uint4*>(H.hist);
    const uint32_t n = H.copies * H.stride / 4u;
    for (uint32_t j = threadIdx.x; j < n; j += waves * 64u) h[j] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
}

// The same word by word and copy by copy, for the batched kernel: it clears once per
// segment, and the compiler holds the wide store's zeros and places in registers through
// all of them, which spills 4 to 20 of the marching bodies' (a batch of one 3000^2
// float32 image 20.4 and 23.3 us, four of 8000^2 232 and 240).
__device__ __forceinline__ void zero_hist_words(const HistRef& H, int width)
{
    const int words = width + (int)H.first;
    for (uint32_t c = 0; c < H.copies; ++c)
        for (int j = threadIdx.x; j < words; j += blockDim.x) H.hist[c * H.stride + j] = 0;
    __syncthreads();
}

// The workgroup's count of bin j of the window: the sum of its copies.
__device__ __forceinline__ int32_t hist_value(const HistRef& H, int j)
{
    j += (int)H.first;
    int32_t t = H.hist[j];
    for (uint32_t c = 1; c < H.copies; ++c) t += H.hist[c * H.stride + j];
    return t;
}

// Inclusive scan of one value per lane across the wave: within rows of 16 lanes,
// then from row to row (DPP lane moves).
__device__ __forceinline__ int32_t wave_scan32(int32_t v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111 /* row_shr:1 */, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112 /* row_shr:2 */, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114 /* row_shr:4 */, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118 /* row_shr:8 */, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142 /* row_bcast:15 */, 0xA, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143 /* row_bcast:31 */, 0xC, 0xF, false);
    return v;
}

// Prefix-sums the workgroup histogram (negated with sign -1) into its partial row
// dst[0..width), or adds it to what dst holds (add).  With windows the row goes on
// from the sum of the windows before: prev (null for the first window) is the last
// word that the window before left in this row.  The merge then only adds rows
// (ecc_merge.h).  An int32 holds every prefix: the cells at a position that lie in a
// sublevel set add up to between -2 and 1, and a workgroup counts fewer than 2^30
// positions (about 2^27 voxels; four times that where most of an image's wave tasks
// are nearly empty).  Counters may pass 2^31 on the way, 32-bit sums are exact modulo
// 2^32.  Each wave
// scans a run of 64-bin segments in place in LDS, then adds the runs before it.
__device__ __forceinline__ void flush_hist(const HistRef& H, int32_t* dst, int width, bool add, int sign,
                                           uint32_t nwaves, const int32_t* prev = nullptr)
{
    __shared__ int32_t run_total[kMaxWaves];
    __syncthreads();
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6), waves = (int)nwaves;
    const int segs = (width + 63) / 64, per = (segs + waves - 1) / waves;
    const int s0 = min(w * per, segs), s1 = min(s0 + per, segs);
    int32_t run = 0;
    for (int s = s0; s < s1; ++s) {
        const int j = s * 64 + lane;
        const int32_t v = wave_scan32(j < width ? hist_value(H, j) : 0) + run;
        if (j < width) H.hist[j + (int)H.first] = v;
        run = __builtin_amdgcn_readlane(v, 63);
    }
    if (lane == 0) run_total[w] = run;
    // (read before the barrier: the row is overwritten after it)
    const int32_t from = prev ? (sign < 0 ? -*prev : *prev) : 0;
    __syncthreads();
    int32_t before = from;
    for (int k = 0; k < waves; ++k) before += k < w ? run_total[k] : 0;
#pragma unroll 4
    for (int s = s0; s < s1; ++s) {
        const int j = s * 64 + lane;
        if (j < width) {
            const int32_t v = H.hist[j + (int)H.first] + before;
            dst[j] = (add ? dst[j] : 0) + (sign < 0 ? -v : v);
        }
    }
}

// Values the whole wave shares, read back from the first lane so that the
// compiler treats them as uniform: the binning parameters may come from device
// memory, and brick coordinates come out of integer divisions that the compiler
// expands into vector arithmetic.  Without this, branches on them are lowered
// as divergent and the row masks that depend on them leave scalar registers.
__device__ __forceinline__ uint32_t uniform_u32(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ int64_t uniform_i64(int64_t v)
{
    const uint32_t lo = uniform_u32((uint32_t)v), hi = uniform_u32((uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double uniform_f64(double v)
{
    return __longlong_as_double((long long)uniform_i64((int64_t)__double_as_longlong(v)));
}
// Binning parameters as uniform values, read back from the first lane.  Loaded
// through a pointer they arrive in vector registers (the kernels also write global
// memory, so the compiler does not load them through the scalar cache); in scalar
// registers the binning reads them directly and the marching bodies keep the
// vector registers.
template <int DT>
__device__ __forceinline__ BinParams uniform_params(BinParams p)
{
    p.nbins = (int32_t)uniform_u32((uint32_t)p.nbins);
    if constexpr (DT == DT_F32) {
        p.base = uniform_f64(p.base);
        p.scale = uniform_f64(p.scale);
    } else {
        p.ilo = uniform_u32(p.ilo);
        p.ihi = uniform_u32(p.ihi);
        p.rcp = uniform_f64(p.rcp);
    }
    return p;
}
// The launch's parameters; with an AUTO range every workgroup folds the min/max
// pass's key pairs itself (up to 8 KB from the L2: about 1 us at the start of the
// launch, where a launch of its own that did it once took 2.6 to 4.8 us).
template <int DT>
__device__ __forceinline__ BinParams load_params(const EccLaunch& L, uint32_t waves)
{
    if (!L.mm) return uniform_params<DT>(L.params);
    __shared__ uint32_t wlo[kMaxWaves], whi[kMaxWaves];
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    const uint2* pairs = (const uint2*)L.mm;
    for (int i = (int)threadIdx.x; i < L.mm_count; i += (int)(waves * 64u)) {
        const uint2 p = pairs[i];
        lo = min(lo, p.x);
        hi = max(hi, p.y);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, off, 64));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
        wlo[threadIdx.x >> 6] = lo;
        whi[threadIdx.x >> 6] = hi;
    }
    __syncthreads();
    for (int k = 0; k < (int)waves; ++k) {
        lo = min(lo, wlo[k]);
        hi = max(hi, whi[k]);
    }
    return uniform_params<DT>(params_from_keys(lo, hi, DT, L.params.nbins));
}
__device__ __forceinline__ const void* uniform_ptr(const void* p) { return (const void*)uniform_i64((int64_t)p); }

// Raw buffer loads: one 32-bit per-lane byte offset (the column) plus one scalar
// byte offset (the row) against a resource whose base is the brick's first row.
// The base is the same for the whole wave; reading it back from the first lane
// lets the compiler keep the resource in scalar registers (otherwise it may not
// prove uniformity and wraps every load in a loop over distinct resources).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_at(const void* base)
{
    const uint64_t a = (uint64_t)base;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    void* u = (void*)(((uint64_t)hi << 32) | lo);
    return __builtin_amdgcn_make_buffer_rsrc(u, (short)0, -1, 0x00020000);
}

template <typename T> __device__ __forceinline__ T buffer_load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff);
template <> __device__ __forceinline__ uint8_t buffer_load<uint8_t>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __builtin_amdgcn_raw_buffer_load_b8(r, (int)voff, (int)soff, 0);
}
template <> __device__ __forceinline__ uint16_t buffer_load<uint16_t>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __builtin_amdgcn_raw_buffer_load_b16(r, (int)voff, (int)soff, 0);
}
template <> __device__ __forceinline__ float buffer_load<float>(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (int)voff, (int)soff, 0));
}

// Advances a scalar offset by `step`; the empty asm keeps the compiler from
// precomputing every row's offset into its own register.
__device__ __forceinline__ uint32_t advance(uint32_t off, uint32_t step)
{
    off += step;
    asm volatile("" : "+s"(off));
    return off;
}

// Index of this wave in its workgroup, known to the compiler to be wave-uniform.
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

}  // namespace dev
}  // namespace ecc
