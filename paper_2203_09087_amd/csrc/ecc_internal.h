// ecc_internal.h -- types shared by the host runtime and the kernels of the ECC
// library.  Not part of the public interface (include/ecc.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ecc {

enum : int32_t { DT_U8 = 0, DT_U16 = 1, DT_F32 = 2 };
enum : int32_t { CONS_VERTEX = 0, CONS_TOP = 1 };

// nbins == D = hi - lo + 1: the bin is level - lo (kIdentLevel); with lo == 0 and no
// value above hi the level itself (kIdentRaw: a full type range, or an AUTO range).
enum : int32_t { kIdentLevel = 1, kIdentRaw = 2 };

// Bin of a value (the library's reading of the paper's gray-level histogram
// index for data that is not 0..255 integers):
//   integer data: a = clamp(v, ilo, ihi) - ilo ; bin = floor(a * nbins / D),
//                 D = ihi-ilo+1 (bin = a when nbins == D), computed as the
//                 double product (a * nbins) * rcp with rcp = 1/D rounded up,
//                 which is exact because a * nbins < 2^32 and D <= 65536;
//   float data:   NaN -> nbins-1; flat range -> (x > hi ? nbins-1 : 0);
//                 otherwise clamp(floor(((double)x - lo) * scale), 0, nbins-1),
//                 scale = nbins / (hi - lo) (+inf for a flat range, which with
//                 the next double above lo as subtrahend gives the flat rule
//                 through the same formula).
struct BinParams {
    int32_t dtype;
    int32_t nbins;
    uint32_t ilo, ihi;  // integer range
    int32_t flat;       // float data, hi == lo
    int32_t ident;      // integer data: kIdentRaw, kIdentLevel or 0 (any nbins)
    double base;        // float data: subtrahend (lo, or the next double above lo if flat)
    double scale;       // float data: nbins / (hi - lo), +inf if flat
    double rcp;         // integer data: 1 / D rounded up
};

// Geometry of one image: n0 slowest.  For 2D images n0 is 1.
struct Geom {
    int64_t n0, n1, n2;
};

// Histogram window: bins [bin_lo, bin_lo + width) are accumulated in LDS.
constexpr int kMaxLdsBins = 4096;     // batches, and shapes that are set
// Bins a single image takes in one pass: one copy of 16384 counters is 64 KB of LDS,
// two workgroups per CU.  Every pass reads and bins the whole image again, which
// costs more than the one copy's conflicts: 190x310x263 uint16, 16384 bins: four passes
// 130 us, one 34; 32^3 to 2048^2 and 256^3 with 5000 to 65535 bins 1.5 to 4 times
// faster.
constexpr int kWideLdsBins = 16384;

// Brick shapes of the wave kernels (64 x-lanes, 63 of them owned).  The
// ECC_* macros exist for tuning builds; the defaults are the shipped shapes.
#ifndef ECC_ROWS3
#define ECC_ROWS3 3
#endif
#ifndef ECC_STRIP_ROWS
#define ECC_STRIP_ROWS 6   // 7/6 rows loaded and binned per row, 86 vector registers (5 waves per SIMD)
#endif
#ifndef ECC_CHUNK2
#define ECC_CHUNK2 16
#endif
#ifndef ECC_WAVES_PER_EU_3D
#define ECC_WAVES_PER_EU_3D 5   // resident waves per SIMD the 3D kernels are compiled for
#endif
#ifndef ECC_WAVES_PER_EU_BATCH
#define ECC_WAVES_PER_EU_BATCH 5   // resident waves per SIMD the batched kernel is compiled for
#endif
#ifndef ECC_WAVES_PER_EU_2D
#define ECC_WAVES_PER_EU_2D 5   // resident waves per SIMD the 2D kernels are compiled for
#endif
// A workgroup histogram is kept in several copies, lane l of every wave adding to
// copy l mod copies: equal keys of neighbouring lanes (frequent in smooth images)
// then fall into different copies, each starting 8 words further in the bank
// cycle than the one before, so they do not collide in one LDS bank.  The merge
// adds the copies.  Two copies for wide windows; a narrow window affords more
// (hist_copies), which smooth data with few bins needs.  The LDS a launch takes
// is sized to its window and copies (dynamic shared memory), so a histogram of
// few bins leaves room for more workgroups.
constexpr int kHistCopies = 2;   // copies of a window of 1025 to 8192 bins
constexpr int kMaxHistCopies = 8;
// Default copies for a window of `width` bins: 8 up to 256 bins, 4 up to 1024, 2 up
// to 8192, then one.
inline __host__ __device__ uint32_t hist_copies(int32_t width)
{
    return width <= 256 ? 8u : (width <= 1024 ? 4u : (width <= 2 * kMaxLdsBins ? (uint32_t)kHistCopies : 1u));
}
// Words from one copy to the next for a window of `width` bins (a multiple of 32
// plus 8: the 8-bank offset; at least two words are spare: the sentinel's, and with
// windows the one of the keys below the window).
inline __host__ __device__ uint32_t lds_stride(int32_t width)
{
    return ((uint32_t)width + 31u) / 32u * 32u + 8u;
}
// Positions a wave owns along x (lanes 0..62; lane 63 only supplies lane 62's
// right neighbour).
constexpr int kLaneCols = 63;
// Positions along an axis of n voxels that carry a single or a pair (the cell
// types of the kernels): n for the vertex filtration; n + 1 lattice points for
// the top filtration (the first one before voxel 0).
inline __host__ __device__ int64_t axis_positions(int64_t n, int construction)
{
    return n + (construction == CONS_TOP ? 1 : 0);
}
constexpr int kRows3 = ECC_ROWS3;      // rows per 3D brick of a batch
constexpr int kStripRows = ECC_STRIP_ROWS;   // rows per strip of a single 3D image
constexpr int kChunk2 = ECC_CHUNK2;    // rows loaded together in the 2D kernel
// Waves per workgroup of the main kernels.
constexpr int kMaxSetWaves = 9;   // the most that a launch shape can ask for
constexpr int kBatchWaves = 8;    // of a batch launch, or kMaxWaves (build_batch_tables)
constexpr int kMaxWaves = 16;

// Bricks of a 3D volume, the units in which a batch is scheduled (BatchWork).
// Ordinary bricks are an x-chunk of 63 * waves position columns x kRows3 rows (a
// strip) x `depth` planes.  A narrow tail of t < 32 columns after the full chunks
// counts as packed bricks: t + 1 lanes per strip, floor(64 / (t + 1)) strips per
// wave, for the strips whose rows (and the row after them) all lie in the image;
// the few other strips' tails count as ordinary bricks.
struct Layout3 {
    int64_t nxc;        // x-chunks of the ordinary bricks of each strip (full ones)
    int64_t nyb;        // strips
    int64_t t;          // positions of the tail (0: none)
    int64_t spw;        // tail strips per wave (0: the tail is not packed)
    int64_t sa, sb;     // strips [sa, sb) have packed tails
    int64_t npk;        // packed bricks per plane block
    int64_t per_z;      // bricks per plane block
};
inline Layout3 layout_3d(const Geom& g, int construction, int waves)
{
    Layout3 y = {};
    const int64_t cw = (int64_t)kLaneCols * waves;
    const int64_t xpos = axis_positions(g.n2, construction);
    const int64_t org = construction == CONS_TOP ? -1 : 0;
    y.nyb = (axis_positions(g.n1, construction) + kRows3 - 1) / kRows3;
    y.nxc = xpos / cw;
    y.t = xpos - y.nxc * cw;
    // strip s reads rows org + 3s .. org + 3s + 3 (the last one completes pairs)
    y.sa = org < 0 ? 1 : 0;
    y.sb = g.n1 - kRows3 - 1 - org >= 0 ? (g.n1 - kRows3 - 1 - org) / kRows3 + 1 : 0;
    if (y.sb > y.nyb) y.sb = y.nyb;
    const int64_t group = y.t + 1;
    // a lane's rows are up to (3 spw + 1) rows past the wave's first: 32-bit offsets
    const int64_t row_bytes = g.n2 * 4;
    const bool pack = y.t > 0 && group <= 32 && y.sb > y.sa &&
                      (kRows3 * (64 / group) + 1) * row_bytes < (int64_t(1) << 31);
    if (pack) {
        y.spw = 64 / group;
        const int64_t per_brick = y.spw * waves;
        y.npk = (y.sb - y.sa + per_brick - 1) / per_brick;
        y.per_z = y.nxc * y.nyb + y.npk + (y.nyb - (y.sb - y.sa));
    } else {
        if (y.t > 0) y.nxc += 1;
        y.t = 0;
        y.sa = y.sb = 0;
        y.per_z = y.nxc * y.nyb;
    }
    return y;
}

// How the waves divide an image (computed on the host: the 64-bit divisions cost a
// small image more than its counting).
//
// 3D, per plane block: a strip is kStripRows rows; its slots are its position
// columns and one more (the column past the last one, which only supplies the
// sentinel to its left neighbour).  The slots of the strips whose rows (and the
// row after them) all lie in the image are numbered through, strip after strip,
// and cut into units of 63 (half a wave: 64 lanes, the last one only supplying
// its left neighbour's right one), so a unit may run from one strip's end into the
// next strip and no lane idles on row tails or narrow rows: a 512-wide row takes
// 8.14 units of 63.  A wave task is two consecutive units.  The strips that reach
// over the image's first or last rows are cut each for itself.
//
// 2D: the same with blocks of `depth` rows (a multiple of 8) in place of strips;
// a last block of fewer rows is cut for itself.  Rows too long for 32-bit offsets
// from one block into the next ones: every block for itself (and within it the
// loads start anew where a row's offset grows past 32 bits, march_2d).
struct Units {
    uint32_t slots;        // per strip (block)
    uint32_t sa, sb;       // strips (blocks) [sa, sb) are numbered through
    uint32_t pairs_full;   // wave tasks over them
    uint32_t pairs_edge;   // wave tasks of each other strip (block)
    uint32_t tasks;        // wave tasks per plane block (2D: of the image)
};
inline Units units_3d(const Geom& g, int construction)
{
    const int64_t org = construction == CONS_TOP ? -1 : 0;
    const int64_t nyb = (axis_positions(g.n1, construction) + kStripRows - 1) / kStripRows;
    const int64_t slots = axis_positions(g.n2, construction) + 1, per = 2 * kLaneCols;
    // strip s reads rows org + R s .. org + R s + R (the last one completes pairs)
    int64_t sa = org < 0 ? 1 : 0;
    int64_t sb = g.n1 - kStripRows - 1 - org >= 0 ? (g.n1 - kStripRows - 1 - org) / kStripRows + 1 : 0;
    if (sb > nyb) sb = nyb;
    if (sb <= sa) sa = sb = 0;
    const int64_t full = ((sb - sa) * slots + per - 1) / per, edge = (slots + per - 1) / per;
    return Units{(uint32_t)slots, (uint32_t)sa, (uint32_t)sb, (uint32_t)full, (uint32_t)edge,
                 (uint32_t)(full + (nyb - (sb - sa)) * edge)};
}
inline Units units_2d(const Geom& g, int construction, int64_t depth)
{
    const int64_t slots = axis_positions(g.n2, construction) + 1, per = 2 * kLaneCols;
    if (g.n1 < depth) {   // one block, by itself (what follows gives the same)
        const uint32_t tasks = (uint32_t)((slots + per - 1) / per);
        return Units{(uint32_t)slots, 0u, 0u, 0u, tasks, tasks};
    }
    const int64_t nyb = (g.n1 + depth - 1) / depth;
    // a lane's rows reach up to `span` blocks past the wave's first row
    const int64_t span = (slots + per) / slots + 2;
    const bool flat = depth % 8 == 0 && (double)span * (double)depth * (double)(g.n2 * 4) < 2147483648.0;
    const int64_t whole = flat ? g.n1 / depth : 0;
    const int64_t full = (whole * slots + per - 1) / per, edge = (slots + per - 1) / per;
    return Units{(uint32_t)slots, 0u, (uint32_t)whole, (uint32_t)full, (uint32_t)edge,
                 (uint32_t)(full + (nyb - whole) * edge)};
}

struct EccLaunch {
    const void* data;
    const void* data2;             // non-null (3D): count the elementwise max (min) of data and data2
    int ndim, dtype, construction;
    Geom g;
    Units units;                   // units_3d or units_2d of g
    uint32_t per_z, nbricks;       // 3D: workgroup bricks per plane block, and in all
    const uint32_t* mm;            // non-null: AUTO range, the mm_count min/max key pairs of the image
    int32_t mm_count;
    BinParams params;              // used when mm is null (nbins always)
    int32_t bin_lo, width;
    int32_t windowed;              // nbins > width: skip bins outside the window
    int32_t grid;                  // number of workgroups
    int32_t waves;                 // waves per workgroup, a wave task each
    int64_t depth;                 // planes (3D) or rows (2D) per workgroup brick
    // 3D slab of a larger volume (streaming): planes [0, z_own) of the g.n0 in
    // memory are counted (a plane beyond them is the collar the last one needs);
    // plane 0 is plane z_base of a volume of n0_global planes.  A whole image
    // has z_own = g.n0, z_base = 0, n0_global = g.n0.
    int64_t z_own, z_base, n0_global;
    // Several passes of the same shape in one launch (3D): workgroup row y of
    // the grid (grid x npass workgroups) counts the volume at data (and data2)
    // plus y * pass_stride bytes; its histograms go to partial rows y * grid ..
    int32_t npass;
    int64_t pass_stride;
    int32_t* partials;             // [grid * npass][row_stride] workgroup histograms, prefix-summed
    int32_t row_stride;            // bins of a whole window (the last window may be narrower: width)
    int32_t flush_add;             // add the workgroup histogram to its partial row (else write it)
    int32_t flush_sign;            // +1, or -1: the histogram enters its row negated
    int64_t* out;                  // the caller's output
    uint32_t* counter;             // the fused merge's
    int32_t fused;                 // one window, few rows: the last workgroup merges into out
    uint32_t hist_stride;          // LDS words between the histogram copies (lds_stride(width))
    uint32_t hist_copies;          // copies of the histogram (a power of two up to kMaxHistCopies)
    uint32_t lds_bytes;            // dynamic LDS of the launch
};
// Partial-row words (grid x window) up to which the histogram kernel's last
// workgroup merges the rows (fused_merge) instead of a launch of k_merge.  In us a
// call, merged so and with the launch: 64^2 float32, 500 bins (up to 2048 words) 8.5
// and 11.0; 300^2 uint8 (2 to 4 thousand) 8.3 and 10.7; 400^2 uint8 (4 to 6 thousand)
// 8.4 and 10.6, but 500x200x33 uint16, 16 bins (512 rows, 8192 words) 18.1 and 15.1: its
// LDS adds meet in few counters; 700^2 uint8 (8 to 16 thousand) 11.0 and 10.6; 60^3
// uint8 12.6 and 10.5; 150^2 float32, 4096 bins 15.0 and 11.9; 100^3 uint8 (32 to 64
// thousand) 23.3 and 10.9.
constexpr int64_t kFusedMergeWords = int64_t(1) << 12;

// ---------------------------------------------------------------- batches

// One volume of a batch, as the batched kernels see it.  The first `count`
// entries are the batch's images (their outputs, ranges and min/max keys); a 2D
// or 3D image is also the volume that is counted.  A 4D image is counted as
// signed 3D volumes (its hyperplanes and the max/min of adjacent pairs) listed
// after the images, each naming its image as `owner`; its own entry is counted
// by none.
struct BatchImage {
    const void* data;
    const void* data2;    // a pair volume: count the max (vertex) or min (top) of data and data2
    Geom g;
    int32_t ndim, dtype;
    int32_t auto_range;   // parameters come from the min/max keys mm[2*owner], mm[2*owner+1]
    int32_t sign;         // +1, or -1: the volume's histogram enters its image's rows negated
    int32_t owner;        // the image whose output, range and partial rows the volume uses
    Units units;          // wave tasks (3D: per plane block)
    int64_t depth;        // planes (3D) or rows (2D) per wave task
    BinParams params;     // explicit or default range
    int64_t* out;         // the caller's output, nbins int64
};
static_assert(sizeof(BatchImage) <= 160, "ecc_reserve's table bound counts 160 bytes per volume");

// A run of one volume's work handled by one workgroup; its histogram lands in
// partial row `slot`.  In the host's schedule [b0, b1) are bricks (BatchWork), in
// the tables of the kernel the steps that they stand for.
struct BatchSeg {
    int32_t image;
    int32_t slot;
    int64_t b0, b1;
};

// A contiguous piece of one AUTO-range image for the batched min/max pass.
struct BatchPiece {
    int32_t image;
    int32_t pad;
    int64_t begin, end;   // element range
};

struct BatchLaunch {
    const BatchImage* images;
    int32_t count;
    int32_t dtype;              // the launch serves the images of this dtype
    const BatchSeg* segs;
    const int32_t* wg_seg;      // workgroup g runs segs[wg_seg[g] .. wg_seg[g+1])
    const int32_t* slot_off;    // image i owns partial rows slots[slot_off[i] .. slot_off[i+1])
    const int32_t* slots;
    uint32_t* mm;               // [count][2] min/max keys of AUTO images
    int32_t* partials;          // [nslots][row_stride]
    int32_t row_stride;         // bins of a whole window
    int32_t avg_rows, max_rows; // partial rows per image, on average and at most
    int32_t nbins, bin_lo, width, windowed;
    int32_t grid, waves;
    int32_t pairs;              // the launch counts pair volumes (4D images)
    uint32_t hist_stride, hist_copies, lds_bytes;   // LDS layout, as in EccLaunch
};

// Launchers (ecc_batch.hip).
hipError_t launch_minmax_batch(const BatchImage* images, const BatchPiece* pieces, int npieces, uint32_t* mm,
                               hipStream_t s);
hipError_t launch_ecc_batch(const BatchLaunch& B, int construction, hipStream_t s, hipEvent_t t0 = nullptr,
                            hipEvent_t t1 = nullptr);
// Sets mm[2i] = ~0, mm[2i+1] = 0 for the `count` images (a kernel, so that the
// enqueue stays valid inside a captured graph).
hipError_t launch_mm_init(uint32_t* mm, int count, hipStream_t s);
// Merges every image's partial rows into its out[bin_lo .. bin_lo+width).
hipError_t launch_merge_batch(const BatchLaunch& B, hipStream_t s);
// How a batch image's work is scheduled.  The schedule counts in bricks: 3D, an
// x-chunk of 63 * wpb position columns x kRows3 rows x depth3 planes (layout_3d);
// 2D, a chunk x depth2 rows (a multiple of kChunk2).  The kernel divides the
// volume into wave tasks (Units) instead; a run of bricks stands for the same
// share of the steps of the volume's wave tasks, in order (3D: planes; 2D: groups of
// kChunk2 rows).
struct BatchWork {
    int64_t bricks;
    int64_t brick_voxels;   // whole brick, including any part outside the image
    int64_t steps;          // of all wave tasks of the volume
    double cost;            // time of the marching, in vector instructions of a wave
};
// Sets the image's depth (3D: at most `planes`) and units.
BatchWork batch_work(BatchImage& im, int construction, int depth3, int depth2, int64_t planes);
constexpr int kBrickWaves = 9;                 // waves that a brick's width is chosen for

// Launchers (ecc_kernels.hip: histogram kernels; ecc_reduce.hip: min/max
// and merge).  All enqueue on `s` and return the launch status.

// 13 smoothing taps (ecc_smooth.hip): tap k weights the neighbour at offset k - 6.
struct Taps13 {
    float w[13];
};
// Both passes in one launch; out must not overlap in.
hipError_t launch_smooth13_tile(const float* in, float* out, int64_t n1, int64_t n2, const Taps13& w, hipStream_t s);
// Rows (in -> tmp), then columns (tmp -> out) of an n1 x n2 float image; out may be in.
hipError_t launch_smooth13(const float* in, float* out, float* tmp, int64_t n1, int64_t n2, const Taps13& w,
                           hipStream_t s);
hipError_t launch_minmax(const void* data, int dtype, int64_t nvox, uint32_t* mm_out, int blocks,
                         hipStream_t s);
// Elementwise max (take_max) or min of the n values at a and b into out, NaN
// taken as the largest float (the reduction of images of 5+ dimensions).
hipError_t launch_combine(const void* a, const void* b, void* out, int64_t n, int dtype, bool take_max,
                          hipStream_t s);
hipError_t launch_ecc(const EccLaunch& L, hipStream_t s, hipEvent_t t0 = nullptr, hipEvent_t t1 = nullptr);
// The same for one data type, and the address of its single-image kernel
// (ecc_kernels_dt.h).
template <int DT> hipError_t launch_ecc_dt(const EccLaunch& L, hipStream_t s, hipEvent_t t0, hipEvent_t t1);
template <int DT> const void* kernel_dt(int ndim, int construction, bool windowed);
template <int DT>
hipError_t launch_batch_dt(const BatchLaunch& B, int construction, hipStream_t s, hipEvent_t t0, hipEvent_t t1);
// The merge of partial rows into out[bin_lo .. bin_lo + width) of one image or of
// every image of a batch (ecc_merge.h).
struct MergeArgs {
    const int32_t* partials;       // rows of `width` bins, row_stride words apart, prefix-summed
    int32_t row_stride;
    int rows;                      // one image: rows 0 .. rows - 1
    const int32_t* slot_off;       // a batch: image i has rows slots[slot_off[i] .. slot_off[i + 1])
    const int32_t* slots;
    const BatchImage* images;      // a batch: its images' outputs; else null, and `out`
    int64_t* out;
    int32_t width, bin_lo;
    int32_t accumulate;            // add to out instead of writing it (slabs, the 3D passes of a 4D image)
    int32_t sign;                  // -1: subtract the sums
};
constexpr int32_t kWideMerge = 1536;   // bins from which a merge block takes 32 of them, else 16
hipError_t launch_merge(const MergeArgs& A, hipStream_t s);
// Folds `blocks` min/max key pairs into the running pair acc (first: start it).
hipError_t launch_mm_fold(const uint32_t* mm, int blocks, uint32_t* acc, bool first, hipStream_t s);

// Workgroup bricks of an image (a 3D one: of one volume) for a launch shape.
int64_t wg_bricks(int ndim, int construction, const Geom& g, int waves, int64_t depth);
// Workgroups of the main kernel variant (of `waves` waves, lds_bytes of dynamic
// LDS) that fit on one CU.
int resident_wgs_per_cu(int ndim, int dtype, int construction, bool windowed, int waves, uint32_t lds_bytes);

}  // namespace ecc
