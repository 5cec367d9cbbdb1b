// ecc_march.h -- the marching bodies of the histogram kernels: two positions per
// lane, 16-bit keys packed in one register, one histogram add per voxel.
//
// The method (ecc_device.h): the cells of one type (a single position or a pair
// per axis) are counted along the marching axis as d(p) - d(p-1) at the value
// of the type function C(p).  A type's value is the key of one of its voxels, so
// the counts of the types of an anchor (y, x) -- T0 the voxel, T1 its pair in y,
// T2 its pair in x, T3 the square -- are first handed to that voxel: T2 (T3) to
// the left or the right voxel (column pair), whichever attains it, then T1's
// sum to the upper or the lower one.  The handed-over sums are added up per
// voxel in registers and one LDS add per voxel remains (four before).
//
// What bounds it.  One add per type kept the LDS busy for 69% of the cycles of
// a 512^3 float32 field (71% of that bank conflicts) next to 71% of the vector
// issue slots, and neither gave way alone.  Here every type, comparison and
// hand-over works on two positions at once: v_pk_max_u16 / v_pk_sub_i16 on
// packed keys, one v_perm_b32 that turns the four sign bits of two differences
// into four byte masks, and plain 32-bit arithmetic on byte fields (count + 16
// per byte, so no field ever borrows from the next one).  Every vector
// instruction of such a mix takes 4 cycles of its SIMD (measured: 2 only while all
// its waves run nothing but plain 32-bit adds, ands and shifts), so the packed
// forms halve the time of what they do.  A row of two positions takes 47 (float32,
// 14 of them binning 7/6 rows), the LDS is busy 22% of the cycles.  512^3 float32,
// 4096 bins: 0.142 to 0.120 ms (5.5 TB/s past the L2, 1.24 times the image, beside
// 0.1 ms of vector issue); 256^3 uint8, 256 bins: 0.033 to 0.021 ms.
//
// Fields.  A register of byte fields holds [A.a, A.b, B.a, B.b]: two quantities
// A and B (bytes 0-1 and 2-3) of the lane's positions a and b.  A field is a
// small signed count plus a multiple of 16; the low four bits of the final
// field, sign-extended, are the voxel's count (between -7 and 7: the Euler
// characteristic change of adding one voxel in three dimensions, or a part of
// it at a brick's faces).
//
// Ties.  A cell goes to one voxel that attains its value: the later plane, then
// the left column, then the upper row.  This is one fixed order of the voxels,
// so every cell is counted once; the VCEC does not depend on it.
#pragma once

#include "ecc_device.h"

namespace ecc {
namespace dev {

typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ u16x2 as_pk(uint32_t v) { return __builtin_bit_cast(u16x2, v); }
__device__ __forceinline__ uint32_t pk_max(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(as_pk(a), as_pk(b)));
}
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(as_pk(a), as_pk(b)));
}
__device__ __forceinline__ uint32_t pk_sub(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, as_pk(a) - as_pk(b));
}
// a - b, 0 where b is larger
__device__ __forceinline__ uint32_t pk_subsat(uint32_t a, uint32_t b)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(as_pk(a), as_pk(b)));
}
template <int CONS>
__device__ __forceinline__ uint32_t pk_op(uint32_t a, uint32_t b)
{
    return CONS == CONS_VERTEX ? pk_max(a, b) : pk_min(a, b);
}
__device__ __forceinline__ uint32_t halves(uint32_t v) { return v * 0x10001u; }

// The four sign bits of two packed differences as byte masks (0x00 or 0xFF):
// bytes 0, 1 = lo's halves, bytes 2, 3 = hi's (v_perm_b32 selectors 8..11 replicate
// a half's sign bit over a byte).
__device__ __forceinline__ uint32_t signs(uint32_t hi, uint32_t lo)
{
    return __builtin_amdgcn_perm(hi, lo, 0x0B0A0908u);
}
// The two sign bits of one packed difference in bytes 0, 1 (bytes 2, 3 zero).
__device__ __forceinline__ uint32_t signs_low(uint32_t v)
{
    return __builtin_amdgcn_perm(v, v, 0x0C0C0908u);
}

// lane i <- lane i-1 (lane 0 gets 0)
__device__ __forceinline__ uint32_t from_left(uint32_t v)
{
    return __builtin_amdgcn_mov_dpp(v, 0x138 /* wave_shr:1 */, 0xF, 0xF, true);
}

// Added to every byte field: fields stay positive and the low four bits unchanged.
constexpr uint32_t kFieldBias = 0x10101010u;

// a + b + c in one instruction (left to itself the compiler regroups the sums of
// the fields' shares into more two-operand additions)
__device__ __forceinline__ uint32_t add3(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t d;
    asm("v_add3_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
__device__ __forceinline__ uint32_t add_bias(uint32_t a, uint32_t b)
{
    uint32_t d;
    asm("v_add3_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(kFieldBias));
    return d;
}

// Keys of the packed bodies are bins: 0 .. nbins-1 with one window (sentinel
// S = nbins, whose counter is a spare word), or with windows 0 = below the
// window, 1 .. width = its bins, width + 1 = above it (= the sentinel: binning
// is monotone, so the clamped keys order every cell whose value lies in the
// window as its bins do).  Every key is below 2^15, so a packed difference's sign
// is the comparison.
// What a lane's two positions a (low half) and b (high half) need: the byte
// offsets of their columns (row offsets folded in), the sentinel in the halves
// outside the image, and the owned positions as 0x01 in their bytes (a: bytes
// 0, 2; b: bytes 1, 3).
struct Lanes {
    uint32_t xa, xb;
    uint32_t oob;
    uint32_t own;
};

// Histogram of the packed bodies: keys are counter words (see above).  `copy` is
// the lane's copy as an LDS address (the array's own place included, so that an
// add needs no further address arithmetic).
typedef __attribute__((address_space(3))) int32_t lds_int;
template <bool WIN>
__device__ __forceinline__ HistRef march_hist(int32_t* hist, int32_t width, uint32_t stride, uint32_t copies)
{
    const uint32_t base = (uint32_t)(uintptr_t)(lds_int*)hist;
    return HistRef{hist, (uint32_t)width, base + (__lane_id() & (copies - 1u)) * stride * 4u, stride,
                   (uint32_t)width + (WIN ? 1u : 0u), copies, WIN ? 1u : 0u};
}
__device__ __forceinline__ void lds_add(uint32_t addr, int32_t v)
{
    __hip_atomic_fetch_add((lds_int*)(uintptr_t)addr, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Uniform parts of the key clamp of a window.
struct WinKeys {
    uint32_t floor, sub, top;   // packed: max(key, floor) - sub, at most top
};
template <bool WIN>
__device__ __forceinline__ WinKeys win_keys(int32_t bin_lo, int32_t width)
{
    WinKeys w = {};
    if constexpr (WIN) {
        const uint32_t lo = (uint32_t)bin_lo;
        w.floor = halves(lo > 0 ? lo - 1u : 0u);
        w.sub = halves((lo - 1u) & 0xFFFFu);
        w.top = halves((uint32_t)width + 1u);
    }
    return w;
}

// Packed keys of two values.
template <int DT, int IDENT, bool WIN>
__device__ __forceinline__ uint32_t pair_key(typename ValT<DT>::T a, typename ValT<DT>::T b, const BinParams& p,
                                             const WinKeys& w, uint32_t oob)
{
    uint32_t k;
    if constexpr (DT == DT_F32) {
        k = bin_of<DT>(a, p) | (bin_of<DT>(b, p) << 16);
    } else {
        k = (uint32_t)a | ((uint32_t)b << 16);
        if constexpr (IDENT != kIdentRaw) k = pk_min(pk_subsat(k, halves(p.ilo)), halves(p.ihi - p.ilo));
        if constexpr (IDENT == 0) {
            // bin_of on both halves; v_mad_u32_u16 takes a half and multiplies it
            uint32_t na, nb;
            asm("v_mad_u32_u16 %0, %1, %2, 0" : "=v"(na) : "v"(k), "s"(p.nbins));
            asm("v_mad_u32_u16 %0, %1, %2, 0 op_sel:[1,0,0,0]" : "=v"(nb) : "v"(k), "s"(p.nbins));
            k = (uint32_t)__dmul_rn((double)na, p.rcp) | ((uint32_t)__dmul_rn((double)nb, p.rcp) << 16);
        }
    }
    if constexpr (WIN) k = pk_min(pk_sub(pk_max(k, w.floor), w.sub), w.top);
    return pk_max(k, oob);
}

// Adds the counts of the lane's two positions (low four bits of bytes 0 and 1 of
// `sums`) at their keys.  The LDS address, 4 * key + the lane's copy, is one
// v_mad_u32_u16 on either half.  One window: counts of 0 are added too (a mask
// per add costs more than the adds it saves on rough data).  Windows: most
// keys lie outside, and their adds would all meet in two words, so only the
// others add.
template <bool WIN>
__device__ __forceinline__ void add_pair(const HistRef& H, uint32_t key, uint32_t sums)
{
    uint32_t aa, ab;
    asm("v_mad_u32_u16 %0, %1, 4, %2" : "=v"(aa) : "v"(key), "v"(H.copy));
    asm("v_mad_u32_u16 %0, %1, 4, %2 op_sel:[1,0,0,0]" : "=v"(ab) : "v"(key), "v"(H.copy));
    const int32_t va = (int32_t)(sums << 28) >> 28, vb = (int32_t)(sums << 20) >> 28;
    if constexpr (WIN) {
        if (va != 0 && (key & 0xFFFFu) - 1u < H.span) lds_add(aa, va);
        if (vb != 0 && (key >> 16) - 1u < H.span) lds_add(ab, vb);
    } else {
        lds_add(aa, va);
        lds_add(ab, vb);
    }
}

// Planes [z0, zend) of a strip of R rows (image rows ys .. ys + R; the last one
// only completes pairs) for one wave.  FULL: every row lies inside the image.
// Otherwise the rows outside [r_lo, r_hi) of the strip read the nearest row
// inside and carry the sentinel, whose cells all count 0.  PAIR: the volume is
// the elementwise max (vertex) or min (top) of L.data and L.data2, taken on the
// keys.
//
// Registers.  A step takes the strip row by row: the next plane's key of the row
// after it, the row's types there, the counts of its types in the current plane,
// and the row's loaded registers take the plane after that at once (a whole step
// ahead of their use).  Steps go up and down the rows in turn, so that a row's new
// types can take the registers that the row before it has just freed and are
// back in place after two steps: one set of types and one spare row instead of two
// sets.
template <int DT, int CONS, int R, bool WIN, bool FULL, int IDENT, bool PAIR>
__device__ __forceinline__ void march_3d(const EccLaunch& L, const BinParams& P, const HistRef& H, const Lanes& N,
                                         int64_t ys, uint32_t z0, uint32_t zend, int r_lo, int r_hi)
{
    using T = typename ValT<DT>::T;
    const uint32_t S = halves(H.sm);
    const WinKeys W = win_keys<WIN>(L.bin_lo, L.width);
    const uint32_t n0 = (uint32_t)L.g.n0;
    const uint32_t row_bytes = (uint32_t)(L.g.n2 * (int64_t)sizeof(T));
    const int64_t pass_off = (int64_t)blockIdx.y * L.pass_stride;
    const char* img = (const char*)L.data + pass_off;
    const char* img2 = PAIR ? (const char*)L.data2 + pass_off : nullptr;
    const int64_t first_row = (ys + (FULL ? 0 : r_lo)) * (int64_t)row_bytes;
    const int64_t plane_bytes = L.g.n1 * (int64_t)row_bytes;
    constexpr int R2 = PAIR ? R + 1 : 1;
    T raw[R + 1][2], raw2[R2][2];   // the loaded plane

    __amdgpu_buffer_rsrc_t rs, rs2;
    uint32_t soff;
    // Starts the loads of plane z (the volume's last plane past it: a load under a
    // condition would cost a copy of every loaded register).
    auto open_plane = [&](uint32_t z, bool up) {
        const int64_t off = first_row + (int64_t)(z < n0 ? z : n0 - 1u) * plane_bytes;
        rs = rsrc_at(img + off);
        if constexpr (PAIR) rs2 = rsrc_at(img2 + off);
        soff = up ? 0u : (uint32_t)(FULL ? R : r_hi - 1 - r_lo) * row_bytes;
    };
    auto load_row = [&](int r, bool up) {
        raw[r][0] = buffer_load<T>(rs, N.xa, soff);
        raw[r][1] = buffer_load<T>(rs, N.xb, soff);
        if constexpr (PAIR) {
            raw2[r][0] = buffer_load<T>(rs2, N.xa, soff);
            raw2[r][1] = buffer_load<T>(rs2, N.xb, soff);
        }
        if (up) {
            if (FULL || (r >= r_lo && r + 1 < r_hi)) soff = advance(soff, row_bytes);
        } else {
            if (FULL || (r > r_lo && r < r_hi)) soff = advance(soff, 0u - row_bytes);
        }
    };
    // the key of the loaded row r; outside: N.oob, or the sentinel past the last plane
    auto key = [&](int r, uint32_t outside) -> uint32_t {
        const uint32_t oob = (FULL || (r >= r_lo && r < r_hi)) ? outside : S;
        uint32_t k = pair_key<DT, IDENT, WIN>(raw[r][0], raw[r][1], P, W, oob);
        if constexpr (PAIR) k = pk_op<CONS>(k, pair_key<DT, IDENT, WIN>(raw2[r][0], raw2[r][1], P, W, oob));
        return k;
    };

    // Signs of the types: T0, T3 plus; T1, T2 minus.  A type's field per plane is
    // D (plus) or 1 - D (minus) with D = [C(z) > C(z+1)], so that the previous
    // field minus this one is the signed count; 0 at positions not owned.
    constexpr uint32_t M01 = 0xFFFF0000u, M23 = 0x0000FFFFu;
    uint32_t t0[R + 1], t1[R], t2[R], t3[R];   // types of the current plane (t0[R]: the row after the strip)
    uint32_t q01[R], q23[R];                   // fields of the previous plane; q23 carries the bias

    // Counts row r of the current plane, whose types compare with the next plane's
    // as d01, d23, and hands the counts to the voxels.  The sum of the row's own
    // voxels is u + h + the share that the row above hands down (one add3); below
    // is the share it hands to the row below.
    struct Sums {
        uint32_t u, h, below;
    };
    auto row = [&](int r, uint32_t d01, uint32_t d23) -> Sums {
        const uint32_t f01 = (d01 ^ M01) & N.own, f23 = (d23 ^ M23) & N.own;
        const uint32_t c01 = q01[r] - f01, c23 = q23[r] - f23;
        q01[r] = f01;
        q23[r] = f23 | kFieldBias;
        // column pairs: the left position attains T2 (T3) or the right one does
        const uint32_t nx = CONS == CONS_VERTEX ? signs(pk_sub(t1[r], t3[r]), pk_sub(t0[r], t2[r]))
                                                : signs(pk_sub(t3[r], t1[r]), pk_sub(t2[r], t0[r]));
        const uint32_t right = c23 & nx;
        // (the empty asm keeps the lane move inside this addition)
        uint32_t t = c01 + from_left(right);
        asm("" : "+v"(t));
        const uint32_t b = add_bias(t, c23 - right);
        // row pairs: this row attains T1 or the next one does
        const uint32_t ny = signs_low(CONS == CONS_VERTEX ? pk_sub(t0[r], t1[r]) : pk_sub(t1[r], t0[r]));
        const uint32_t h = b >> 16;
        const uint32_t below = h & ny;
        return Sums{b - below, h, below};
    };
    auto inside = [&](int r) { return FULL || (r >= r_lo && r < r_hi); };

    // Counts plane z against plane z + 1 (loaded), whose types replace it, and
    // loads plane z + 2.
    auto step_up = [&](uint32_t z) {
        const uint32_t outside = z + 1 < n0 ? N.oob : S;
        open_plane(z + 2, true);
        uint32_t k0 = key(0, outside);
        load_row(0, true);
        uint32_t x0 = pk_op<CONS>(k0, from_right(k0)), above = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t k1 = key(r + 1, outside);
            load_row(r + 1, true);
            const uint32_t x1 = pk_op<CONS>(k1, from_right(k1));
            const uint32_t n1 = pk_op<CONS>(k0, k1), n3 = pk_op<CONS>(x0, x1);
            const uint32_t d01 = signs(pk_sub(n1, t1[r]), pk_sub(k0, t0[r]));
            const uint32_t d23 = signs(pk_sub(n3, t3[r]), pk_sub(x0, t2[r]));
            const Sums s = row(r, d01, d23);
            if (inside(r)) add_pair<WIN>(H, t0[r], add3(s.u, s.h, above));
            above = s.below;
            t0[r] = k0;
            t1[r] = n1;
            t2[r] = x0;
            t3[r] = n3;
            k0 = k1;
            x0 = x1;
            // rows stay apart in the schedule: mixed, they hold far more registers
            __builtin_amdgcn_sched_barrier(0);
        }
        if (inside(R)) add_pair<WIN>(H, t0[R], above);
        t0[R] = k0;
    };
    auto step_down = [&](uint32_t z) {
        const uint32_t outside = z + 1 < n0 ? N.oob : S;
        open_plane(z + 2, false);
        uint32_t k1 = key(R, outside);
        load_row(R, false);
        uint32_t x1 = pk_op<CONS>(k1, from_right(k1));
        uint32_t kn = k1;                     // the next plane's t0[r + 1]
        uint32_t lower_key = t0[R];           // the row below: its key and its sums
        Sums lower = {0u, 0u, 0u};
#pragma unroll
        for (int r = R - 1; r >= 0; --r) {
            const uint32_t k0 = key(r, outside);
            load_row(r, false);
            const uint32_t x0 = pk_op<CONS>(k0, from_right(k0));
            const uint32_t n1 = pk_op<CONS>(k0, k1), n3 = pk_op<CONS>(x0, x1);
            const uint32_t d01 = signs(pk_sub(n1, t1[r]), pk_sub(k0, t0[r]));
            const uint32_t d23 = signs(pk_sub(n3, t3[r]), pk_sub(x0, t2[r]));
            const Sums s = row(r, d01, d23);
            if (inside(r + 1))
                add_pair<WIN>(H, lower_key, r + 1 < R ? add3(lower.u, lower.h, s.below) : s.below);
            t0[r + 1] = kn;
            lower_key = t0[r];
            lower = s;
            t1[r] = n1;
            t2[r] = x0;
            t3[r] = n3;
            kn = k0;
            k1 = k0;
            x1 = x0;
            // rows stay apart in the schedule: mixed, they hold far more registers
            __builtin_amdgcn_sched_barrier(0);
        }
        if (inside(0)) add_pair<WIN>(H, lower_key, lower.u + lower.h);
        t0[0] = kn;
    };

    // the first plane's types
    {
        open_plane(z0, true);
#pragma unroll
        for (int r = 0; r < R + 1; ++r) load_row(r, true);
        open_plane(z0 + 1, true);
        uint32_t x[R + 1];
#pragma unroll
        for (int r = 0; r < R + 1; ++r) {
            t0[r] = key(r, N.oob);
            load_row(r, true);
            x[r] = pk_op<CONS>(t0[r], from_right(t0[r]));
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            t1[r] = pk_op<CONS>(t0[r], t0[r + 1]);
            t2[r] = x[r];
            t3[r] = pk_op<CONS>(x[r], x[r + 1]);
        }
    }
    // The volume's first plane wins the interval before it (D = 1), except types
    // whose cells do not exist (the sentinel), which count 0 throughout.  A later
    // brick's first plane starts with D = 0 and gets the rest from the brick
    // before it (below).
    const uint32_t first = L.z_base + (int64_t)z0 == 0 ? 0xFFFFFFFFu : 0u;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t d01 = signs(pk_sub(t1[r], S), pk_sub(t0[r], S)) & first;
        const uint32_t d23 = signs(pk_sub(t3[r], S), pk_sub(t2[r], S)) & first;
        q01[r] = (d01 ^ M01) & N.own;
        q23[r] = ((d23 ^ M23) & N.own) | kFieldBias;
    }
    uint32_t z = z0;
    for (; z + 1 < zend; z += 2) {
        step_up(z);
        step_down(z + 1);
    }
    if (z < zend) step_up(z);
    if (L.z_base + (int64_t)zend < L.n0_global) {
        // the part of plane zend's counts that this brick's last step decides
        uint32_t above = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const Sums s = row(r, 0u, 0u);
            if (inside(r)) add_pair<WIN>(H, t0[r], add3(s.u, s.h, above));
            above = s.below;
        }
        if (inside(R)) add_pair<WIN>(H, t0[R], above);
    }
}

// A wave's place in a brick of a single 3D image: its lanes, first row, planes
// and the rows of the strip inside the image.
struct Task3 {
    bool active;
    Lanes lanes;
    int64_t ys;
    int r_lo, r_hi;
};

// The slots of wave task `task`: the strip (block) of its first one, that one's
// place in it, and the slots from there to the end of the numbering.
struct Place {
    bool whole;
    int64_t strip, left;
    uint32_t c0;
};
__device__ __forceinline__ Place task_place(const Units& Y, uint32_t task)
{
    const uint32_t P = Y.slots;
    Place p;
    p.whole = task < Y.pairs_full;
    if (p.whole) {
        const uint64_t g = (uint64_t)task * (2u * kLaneCols), total = (uint64_t)(Y.sb - Y.sa) * P;
        const uint64_t s = (total >> 32) == 0 ? (uint64_t)((uint32_t)g / P) : g / P;
        p.strip = (int64_t)Y.sa + uniform_i64((int64_t)s);
        p.c0 = uniform_u32((uint32_t)(g - s * P));
        p.left = uniform_i64((int64_t)(total - g));
    } else {
        const uint32_t e = task - Y.pairs_full;
        const uint32_t i = uniform_u32(e / Y.pairs_edge);
        p.c0 = (e - i * Y.pairs_edge) * (2u * kLaneCols);
        p.strip = i < Y.sa ? (int64_t)i : (int64_t)Y.sb + (int64_t)(i - Y.sa);
        p.left = (int64_t)P - (int64_t)p.c0;
    }
    return p;
}
// Strips (blocks) passed by place c < P + 2 * 64: c / P, for narrow ones through a
// 16-bit reciprocal m = 65536 / P + 1 (exact for c < 256, P < 128).
__device__ __forceinline__ uint32_t strips_passed(uint32_t c, uint32_t P, uint32_t m)
{
    return P < 128u ? (c * m) >> 16 : (c >= P ? 1u : 0u);
}

// Wave task `task` of a plane block.
template <int DT, int CONS, int R>
__device__ __forceinline__ Task3 strip_task(const Geom& G, const Units& Y, uint32_t sm, uint32_t task)
{
    using T = typename ValT<DT>::T;
    constexpr int org = CONS == CONS_TOP ? -1 : 0;
    const int64_t n1 = G.n1, n2 = G.n2;
    const uint32_t row_bytes = (uint32_t)(n2 * (int64_t)sizeof(T));
    const uint32_t P = Y.slots;
    Task3 K;
    K.active = task < Y.tasks;
    const Place at0 = task_place(Y, task);
    const int64_t strip = at0.strip, left = at0.left;
    const uint32_t c0 = at0.c0;
    K.ys = org + strip * R;
    K.r_lo = K.ys < 0 ? (int)(-K.ys) : 0;
    K.r_hi = (int)((n1 - K.ys) < R + 1 ? (n1 - K.ys) : R + 1);
    // the lane's places, computed here for each brick: the empty asm keeps the
    // compiler from hoisting these per-lane values out of the brick loop, where
    // they would hold registers through every brick's body
    uint32_t lane = lane_id();
    asm volatile("" : "+v"(lane));
    const uint32_t m = 65536u / P + 1u;
    uint32_t x[2], oob = 0, own = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t at = (uint32_t)(h * kLaneCols) + lane;
        const bool in = (int64_t)at < left;
        const uint32_t c = in ? c0 + at : 0u;
        const uint32_t q = strips_passed(c, P, m);
        const int32_t col = org + (int32_t)(c - q * P);
        const bool ok = in && col >= 0 && col < (int32_t)n2;
        const uint32_t cx = ok ? (uint32_t)col : (col < 0 ? 0u : (uint32_t)n2 - 1u);
        x[h] = cx * (uint32_t)sizeof(T) + q * ((uint32_t)R * row_bytes);
        if (!ok) oob |= sm << (16 * h);
        if (in && lane < (uint32_t)kLaneCols) own |= 0x00010001u << (8 * h);
    }
    K.lanes = Lanes{x[0], x[1], oob, own};
    return K;
}

// Runs a wave task over planes [z0, zend).  HALF: strips with at most half their rows
// inside the image have a body of half the rows.  They are all there is of a volume of
// few rows (2000 x 2 x 2000 float32, 1000 bins: 30.7 us without and 21.7 us, 24.9 with
// the strips of 3 rows before; 2000 x 13 x 2000 69.3 and 64.8, 66.4 before).  The
// batched and the pair kernels go without: they would spill more registers (float32
// batches 1 us slower each), and gain nothing on most images.
template <int DT, int CONS, int R, bool WIN, bool PAIR, int IDENT, bool HALF>
__device__ __forceinline__ void run_march_3d_as(const EccLaunch& L, const BinParams& P, const HistRef& H,
                                                const Task3& K, uint32_t z0, uint32_t ze)
{
    const bool full = K.r_lo == 0 && K.r_hi == R + 1;
    if (full) return march_3d<DT, CONS, R, WIN, true, IDENT, PAIR>(L, P, H, K.lanes, K.ys, z0, ze, K.r_lo, K.r_hi);
    if constexpr (HALF)
        if (K.r_hi <= R / 2)
            return march_3d<DT, CONS, R / 2, WIN, false, IDENT, PAIR>(L, P, H, K.lanes, K.ys, z0, ze, K.r_lo, K.r_hi);
    march_3d<DT, CONS, R, WIN, false, IDENT, PAIR>(L, P, H, K.lanes, K.ys, z0, ze, K.r_lo, K.r_hi);
}
template <int DT, int CONS, int R, bool WIN, bool PAIR, bool HALF = false>
__device__ __forceinline__ void run_march_3d(const EccLaunch& L, const BinParams& P, const HistRef& H, const Task3& K,
                                             uint32_t z0, uint32_t ze)
{
    if (!K.active) return;
    if constexpr (DT != DT_F32) {
        const int ident = __builtin_amdgcn_readfirstlane(P.ident);
        if (ident == kIdentRaw) return run_march_3d_as<DT, CONS, R, WIN, PAIR, kIdentRaw, HALF>(L, P, H, K, z0, ze);
        if (ident == kIdentLevel) return run_march_3d_as<DT, CONS, R, WIN, PAIR, kIdentLevel, HALF>(L, P, H, K, z0, ze);
    }
    run_march_3d_as<DT, CONS, R, WIN, PAIR, 0, HALF>(L, P, H, K, z0, ze);
}

// ------------------------------------------------------------------------- 2D

// A wave's place in a 2D image: its lanes and the rows of its block.
struct Task2 {
    bool active, whole;   // whole: a block of the numbered slots (every block `depth` rows)
    Lanes lanes;
    uint32_t xl[2];       // the lane's columns in the row after the block (the last row inside the image)
    uint32_t oob_last;    // the sentinel where that row lies outside the image, or N.oob
    uint32_t first;       // 0xFF in the bytes of the positions in the image's first block
    int64_t y0;           // first row of the lanes' (first) block
};

// Rows of a 2D block for one wave: rows are the marching axis, types T0 = the row
// and T1 = op2(T0, right), with signs +, - (vertex) or -, + (top).  The counts of
// T1 go to the left or the right voxel and each voxel's sum is added once (see
// above: bytes 0-1 hold T0's fields, 2-3 T1's).  EDGE: one block for the whole
// wave, `rows` of it counted, `avail` rows readable from its first one.  Otherwise
// (whole blocks, `rows` a multiple of 8) the lanes may sit in different blocks.
// Bound by vector issue: 20 instructions a row of two positions beside the
// binning, every one 4 cycles; loads run 8 rows ahead.
template <int DT, int CONS, bool WIN, int IDENT, bool EDGE>
__device__ __forceinline__ void march_2d(const void* base, uint32_t row_bytes, const BinParams& P, const WinKeys& W,
                                         const HistRef& H, const Task2& K, uint32_t rows, uint32_t avail)
{
    using T = typename ValT<DT>::T;
    constexpr int G = 8;   // rows loaded ahead
    constexpr uint32_t M = CONS == CONS_VERTEX ? 0xFFFF0000u : 0x0000FFFFu;
    const Lanes& N = K.lanes;
    const uint32_t S = halves(H.sm);
    __amdgpu_buffer_rsrc_t rs = rsrc_at(base);
    T raw[G][2];
    uint32_t soff = 0;   // byte offset of the next row to load
    // EDGE: a block's rows may span more than 4 GiB (rows of up to 2^27 bytes, blocks of
    // any depth), so the loads start anew, from the next row's 64-bit address, before a
    // row's offset passes 2^30 by more than 8 rows.
    const char* from = (const char*)base;
    auto keep_offsets_small = [&]() {
        if (soff > (1u << 30)) {
            from += soff;
            rs = rsrc_at(from);
            soff = 0;
        }
    };
    // loads row r (relative to the block): EDGE stays on the last readable row;
    // otherwise the row after the block takes the lanes' own places
    auto load = [&](int k, uint32_t r, bool last) {
        if (EDGE) {
            raw[k][0] = buffer_load<T>(rs, N.xa, soff);
            raw[k][1] = buffer_load<T>(rs, N.xb, soff);
            soff = advance(soff, r + 1 < avail ? row_bytes : 0u);
        } else {
            raw[k][0] = buffer_load<T>(rs, last ? K.xl[0] : N.xa, last ? 0u : soff);
            raw[k][1] = buffer_load<T>(rs, last ? K.xl[1] : N.xb, last ? 0u : soff);
            soff = advance(soff, row_bytes);
        }
    };
    uint32_t t0, t1, q;
    auto count = [&](uint32_t d) {
        const uint32_t f = (d ^ M) & N.own, c = q - f;
        q = f | kFieldBias;
        const uint32_t nx = signs_low(CONS == CONS_VERTEX ? pk_sub(t0, t1) : pk_sub(t1, t0));
        const uint32_t h = c >> 16, right = h & nx;
        uint32_t x = c + from_left(right);
        asm("" : "+v"(x));
        add_pair<WIN>(H, t0, x + (h - right));
    };
    load(0, 0, false);
    t0 = pair_key<DT, IDENT, WIN>(raw[0][0], raw[0][1], P, W, N.oob);
    t1 = pk_op<CONS>(t0, from_right(t0));
    // the image's first row wins the interval before it (D = 1), except types
    // whose cells do not exist (the sentinel)
    q = (((signs(pk_sub(t1, S), pk_sub(t0, S)) & K.first) ^ M) & N.own) | kFieldBias;
#pragma unroll
    for (int k = 0; k < G; ++k) load(k, 1u + (uint32_t)k, !EDGE && k == G - 1 && rows == (uint32_t)G);
    // counts row r - 1 against the loaded row r
    auto row = [&](int k, uint32_t oob) {
        const uint32_t n0 = pair_key<DT, IDENT, WIN>(raw[k][0], raw[k][1], P, W, oob);
        const uint32_t n1 = pk_op<CONS>(n0, from_right(n0));
        count(signs(pk_sub(n1, t1), pk_sub(n0, t0)));
        t0 = n0;
        t1 = n1;
    };
    // groups of G rows that need no check, then the rest
    const uint32_t plain = EDGE ? (rows < avail ? rows : rows - 1u) / G * G : rows - G;
    uint32_t y = 0;
    for (; y < plain; y += G) {
        if (EDGE) keep_offsets_small();
#pragma unroll
        for (int k = 0; k < G; ++k) {
            // the row's registers take the next group's row as soon as its key is made
            const uint32_t n0 = pair_key<DT, IDENT, WIN>(raw[k][0], raw[k][1], P, W, N.oob);
            load(k, y + 1u + (uint32_t)(k + G), k == G - 1 && y + 2 * G >= rows);
            const uint32_t n1 = pk_op<CONS>(n0, from_right(n0));
            count(signs(pk_sub(n1, t1), pk_sub(n0, t0)));
            t0 = n0;
            t1 = n1;
        }
    }
    if (EDGE) {
#pragma unroll
        for (int k = 0; k < G; ++k)
            if (y + (uint32_t)k < rows) row(k, y + 1u + (uint32_t)k < avail ? N.oob : S);
    } else {
#pragma unroll
        for (int k = 0; k < G; ++k) row(k, k == G - 1 ? K.oob_last : N.oob);
    }
    // the part of the next block's first row that this block's last row decides
    // (at the image's last row the keys are the sentinel and the counts 0)
    if (!EDGE || rows < avail) count(0u);
}

// Wave task `task` of a 2D image.
template <int DT, int CONS>
__device__ __forceinline__ Task2 block_task(const Geom& G, const Units& Y, int64_t depth, uint32_t sm, uint32_t task)
{
    using T = typename ValT<DT>::T;
    constexpr int org = CONS == CONS_TOP ? -1 : 0;
    const uint32_t row_bytes = (uint32_t)(G.n2 * (int64_t)sizeof(T));
    const uint32_t P = Y.slots;
    Task2 K;
    K.active = task < Y.tasks;
    const Place at0 = task_place(Y, task);
    K.whole = at0.whole;
    const int64_t block = at0.strip, left = at0.left;
    const uint32_t c0 = at0.c0;
    K.y0 = block * depth;
    // the lane's places, computed here for each brick (strip_task)
    uint32_t lane = lane_id();
    asm volatile("" : "+v"(lane));
    const uint32_t m = 65536u / P + 1u;
    const uint32_t block_bytes = (uint32_t)depth * row_bytes;
    uint32_t x[2], oob = 0, own = 0, oob_last = 0, first = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t at = (uint32_t)(h * kLaneCols) + lane;
        const bool in = (int64_t)at < left;
        const uint32_t c = in ? c0 + at : 0u;
        const uint32_t q = K.whole ? strips_passed(c, P, m) : 0u;
        const int32_t col = org + (int32_t)(c - q * P);
        const bool ok = in && col >= 0 && col < (int32_t)G.n2;
        const uint32_t cx = ok ? (uint32_t)col : (col < 0 ? 0u : (uint32_t)G.n2 - 1u);
        x[h] = cx * (uint32_t)sizeof(T) + q * block_bytes;
        // the row after the block, or its last row where the image ends with it
        const bool ends = K.whole && (block + (int64_t)q + 1) * depth >= G.n1;
        K.xl[h] = x[h] + block_bytes - (ends ? row_bytes : 0u);
        if (!ok) oob |= sm << (16 * h);
        if (!ok || ends) oob_last |= sm << (16 * h);
        if (in && lane < (uint32_t)kLaneCols) own |= 0x00010001u << (8 * h);
        if (block + (int64_t)q == 0) first |= 0x00FF00FFu << (8 * h);
    }
    K.lanes = Lanes{x[0], x[1], oob, own};
    K.oob_last = oob_last;
    K.first = first;
    return K;
}

// Rows [r0, r1) of wave task K's blocks of `depth` rows (multiples of kChunk2), as a
// task of its own; inactive where the image ends before them.
__device__ __forceinline__ Task2 block_part(Task2 K, const Geom& G, int64_t depth, uint32_t row_bytes, uint32_t r0,
                                            uint32_t r1)
{
    K.y0 += (int64_t)r0;
    if (K.y0 >= G.n1) K.active = false;
    if (r0 > 0u) K.first = 0u;
    if ((int64_t)r1 < depth) {   // the row after them lies in the same block
        K.xl[0] = K.lanes.xa + (r1 - r0) * row_bytes;
        K.xl[1] = K.lanes.xb + (r1 - r0) * row_bytes;
        K.oob_last = K.lanes.oob;
    } else {
        K.xl[0] -= r0 * row_bytes;
        K.xl[1] -= r0 * row_bytes;
    }
    return K;
}

// Runs wave task K of the 2D image at data.
template <int DT, int CONS, bool WIN, int IDENT>
__device__ __forceinline__ void run_march_2d_as(const void* data, const Geom& G, int64_t depth, const BinParams& P,
                                                const WinKeys& W, const HistRef& H, const Task2& K)
{
    using T = typename ValT<DT>::T;
    const int64_t row_bytes = G.n2 * (int64_t)sizeof(T);
    const char* base = (const char*)data + K.y0 * row_bytes;
    const uint32_t avail = (uint32_t)(G.n1 - K.y0);
    const uint32_t rows = (int64_t)avail < depth ? avail : (uint32_t)depth;
    if (K.whole) march_2d<DT, CONS, WIN, IDENT, false>(base, (uint32_t)row_bytes, P, W, H, K, rows, avail);
    else march_2d<DT, CONS, WIN, IDENT, true>(base, (uint32_t)row_bytes, P, W, H, K, rows, avail);
}
template <int DT, int CONS, bool WIN>
__device__ __forceinline__ void run_march_2d(const void* data, const Geom& G, int64_t depth, const BinParams& P,
                                             const WinKeys& W, const HistRef& H, const Task2& K)
{
    if (!K.active) return;
    if constexpr (DT != DT_F32) {
        const int ident = __builtin_amdgcn_readfirstlane(P.ident);
        if (ident == kIdentRaw) return run_march_2d_as<DT, CONS, WIN, kIdentRaw>(data, G, depth, P, W, H, K);
        if (ident == kIdentLevel) return run_march_2d_as<DT, CONS, WIN, kIdentLevel>(data, G, depth, P, W, H, K);
    }
    run_march_2d_as<DT, CONS, WIN, 0>(data, G, depth, P, W, H, K);
}

}  // namespace dev
}  // namespace ecc
