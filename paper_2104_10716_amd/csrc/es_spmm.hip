// es_spmm.hip -- edge-sampled SpMM for gfx950 (MI355X), C ABI in include/es_spmm.h.
//
// Paper: Algorithm 1 ("CacheSample"): stage 1 samples at most W entries of each
// CSR row into on-chip memory (Section 4.2, sampling rules of Section 4.4 /
// Equation 2), stage 2 multiplies the staged entries with gathered rows of the
// dense matrix (Section 4.3).
//
// Mapping to CDNA4 (differs from the paper's 512-thread CUDA blocks on purpose):
//   * A wavefront (64 lanes) owns R = 2^logR consecutive rows.  The 64/R lanes of
//     a row ("team") are E x G: G lanes span the feature columns with VEC-wide
//     loads (CH column chunks per lane), E edge slots run side by side and are
//     summed with cross-lane shuffles at the end.
//   * Each wave has a private LDS tile of kTileSlots (column, value) pairs,
//     T = kTileSlots/R per row.  Stage 1: the team's lanes evaluate the sampler
//     for slots t, t+64/R, ... and copy (colidx, vals) into the tile.  Stage 2:
//     lanes read a slot as one 64-bit LDS broadcast and issue U independent
//     VEC-wide global loads of X before the first FMA.  Rows longer than a tile
//     (full mode, or W > T) refill the tile; no barrier other than wave-level
//     ordering is needed because a tile is private to its wave.
//   * Workgroup ids are remapped so each of the 8 XCDs (one L2 each) walks one
//     contiguous range of rows.
//   * Rows that keep more than `long_k` entries (full mode on skewed graphs, or a
//     very large W) would leave one wave running long after the rest of the grid
//     has drained.  The leading workgroups of the launch split each such row
//     into 256-slot segments, deal the segments to the waves of kLongSplit
//     workgroups and add the partial sums to Y with fp32 atomics (a small
//     kernel zeroes those rows of Y first; in a small product one wave or
//     workgroup sums the row instead); the row workgroups skip them.
//     long_k is chosen on the host so that a single wave's longest row stays a
//     few percent of the whole launch.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "es_spmm.h"

#include "es_common.h"
#include "es_sampler.h"
#include "es_tile.h"
#include "es_fused_kernel.h"
#include "es_part_kernel.h"
#include "es_flat_kernel.h"
#include "es_aux_kernels.h"
#include "es_bin_kernel.h"
#include "es_pull_kernel.h"

// Workspace of es_spmm_static_ws: the cuts array of the column-partitioned
// product for up to ES_SPMM_STATIC_WS_MAX_ROWS rows, in static device memory.
// In host code this name is only a handle for hipGetSymbolAddress; the address
// kernels receive is the per-device pointer static_scratch_address() returns.
static __device__ __align__(256) unsigned char scratch[(size_t)ES_SPMM_STATIC_WS_MAX_ROWS * kParts * sizeof(int32_t)];

namespace {

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
constexpr int kMaxDevices = 64;
constexpr int kComputeUnits = 256;

// Device address of `scratch` on the current device (every GPU holds its own
// copy of the array at its own address); looked up once per device.
int static_scratch_address(void** out)
{
    static std::mutex mu;
    static void* address[kMaxDevices] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return ES_ERR_LAUNCH;
    std::lock_guard<std::mutex> guard(mu);
    if (!address[dev]) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return ES_ERR_LAUNCH;
        address[dev] = p;
    }
    *out = address[dev];
    return ES_OK;
}

struct Shape {
    int vec, G, CH;
    bool aligned;
};

int next_pow2(int v)
{
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

// Lanes x chunks that cover F columns: 128-bit accesses whenever F >= 4
// (aligned or not), 32-bit ones for F < 4.
Shape pick_shape(int F, bool aligned)
{
    Shape s;
    s.aligned = aligned;
    s.vec = (aligned || F >= 4) ? 4 : 1;
    const int q = (F + s.vec - 1) / s.vec;                 // accesses per row
    s.G = next_pow2(q);
    if (s.G < 4) s.G = 4;
    s.CH = 1;
    if (s.G > 64) {
        s.G = 64;
        s.CH = q > 128 ? 4 : 2;
    }
    return s;
}

// Rows per wave: enough edge slots per row to fill a batch of loads, but not
// more slots than a typical row has entries.
int pick_logR(const Shape& s, double mean_kept)
{
    const int U = 8 / s.CH;
    const int maxR = 64 / s.G;
    if (mean_kept < 1.0) mean_kept = 1.0;
    const double want = 64.0 * U / (s.G * mean_kept);      // R >= want
    int R = 1;
    while (R < maxR && R < want) R <<= 1;
    int logR = 0;
    while ((1 << logR) < R) ++logR;
    return logR;
}

template <int G, int CH, int VEC, bool ALIGNED, bool WIDE>
hipError_t launch_forward(const Args& a, dim3 grid, bool long_alone, hipStream_t st)
{
    if constexpr (!WIDE) {
        if (long_alone) {
            hipLaunchKernelGGL((es_spmm_small_kernel<G, CH, VEC, ALIGNED>), grid, dim3(kBlockThreads), 0, st, a);
            return hipGetLastError();
        }
    }
    if (a.long_blocks > 0) {
        const uint32_t zb = (uint32_t)((a.N + kBlockThreads - 1) / kBlockThreads);
        hipLaunchKernelGGL(es_zero_long_rows_kernel, dim3(zb), dim3(kBlockThreads), 0, st, a);
        const hipError_t err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    hipLaunchKernelGGL((es_spmm_kernel<G, CH, VEC, ALIGNED, false, WIDE>), grid, dim3(kBlockThreads), 0, st, a);
    return hipGetLastError();
}

template <int G, bool ALIGNED, bool WIDE>
hipError_t launch_flat(Args a, dim3 grid, bool partition, int32_t* cuts, hipStream_t st)
{
    if (!partition) {
        if (a.long_blocks > 0) {
            const uint32_t zb = (uint32_t)((a.N + kBlockThreads - 1) / kBlockThreads);
            hipLaunchKernelGGL(es_zero_long_rows_kernel, dim3(zb), dim3(kBlockThreads), 0, st, a);
            const hipError_t err = hipGetLastError();
            if (err != hipSuccess) return err;
        }
        if (a.mode == ES_FASTRAND)                         // with Equation 2's strided slots compiled in
            hipLaunchKernelGGL((es_spmm_flat_kernel<G, ALIGNED, WIDE, true, 2>), grid, dim3(kBlockThreads), 0, st, a);
        else if (a.mode == ES_BUCKET)
            hipLaunchKernelGGL((es_spmm_flat_kernel<G, ALIGNED, WIDE, false, 2>), grid, dim3(kBlockThreads), 0, st, a);
        else
            hipLaunchKernelGGL((es_spmm_flat_kernel<G, ALIGNED, WIDE, false, 1>), grid, dim3(kBlockThreads), 0, st, a);
        return hipGetLastError();
    }
    a.cuts = cuts;
    a.part_cols = (int32_t)((a.N + kParts - 1) / kParts);
    const uint32_t cb = (uint32_t)((a.N * kParts + kBlockThreads - 1) / kBlockThreads);
    hipLaunchKernelGGL(es_cuts_kernel, dim3(cb), dim3(kBlockThreads), 0, st, a.rowptr, a.colidx, a.N,
                       a.part_cols, cuts);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    for (int phase = 0; phase < kParts; ++phase) {
        a.phase = phase;
        if (phase == 0)
            hipLaunchKernelGGL((es_spmm_part_flat_kernel<G, ALIGNED, WIDE, false>), grid, dim3(kBlockThreads), 0, st, a);
        else
            hipLaunchKernelGGL((es_spmm_part_flat_kernel<G, ALIGNED, WIDE, true>), grid, dim3(kBlockThreads), 0, st, a);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

// The transposed product always runs the 32-bit interleaved column mapping
// (lane l owns columns l, l+G, ...): one atomic instruction then covers G
// consecutive floats of an output row instead of every fourth one, which is
// what the memory-side atomic units are fastest at (measured 4x over the
// 128-bit mapping); G is as wide as F allows for the same reason.
template <int G, int CH, bool WIDE>
hipError_t launch_backward(const Args& a, dim3 grid, hipStream_t st)
{
    int64_t fb = (a.N * (int64_t)a.F + kBlockThreads * 8 - 1) / (kBlockThreads * 8);
    if (fb > 65536) fb = 65536;
    hipLaunchKernelGGL(es_fill_zero_kernel, dim3((uint32_t)fb), dim3(kBlockThreads), 0, st, a.Y, a.N, a.F,
                       a.ldy);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL((es_spmm_kernel<G, CH, 1, false, true, WIDE>), grid, dim3(kBlockThreads), 0, st, a);
    return hipGetLastError();
}

// Longest row one wave may own.  A wave retires about E*U entries per memory
// round trip (~2 us under load) while the whole launch moves entries*(4F+8)
// bytes at a few TB/s; the bound keeps one wave's row near 5 % of the launch.  Below
// four times the mean (rounded down to a multiple of kLongMin) a row is never split,
// whatever the bound: on a small dense graph that would send nearly every row through
// the splitting and its atomics (exact product, 10 k rows of mean 300, F = 64: 159
// us at a threshold of 64, 33 now; the transposed one, whose rows are atomic either
// way: 641 and 598, 1000 rows of mean 400: 305 and 104).  Rounding up instead takes
// rows of 65 to 128 entries on one wave where the mean is 16 to 31: 40 k rows, F = 16:
// 14.7 us, 13.5 this way.
int32_t pick_long_k(const Shape& s, int logR, double entries, int F, double mean)
{
    const int U = 8 / s.CH;
    const int E = (64 >> logR) / s.G;
    double k = (double)E * U * entries * (4.0 * F + 8.0) / 2.4e8;
    if (k < 4.0 * mean) k = 4.0 * mean;
    if (k >= (double)(INT32_MAX - kLongMin)) return INT32_MAX;
    const int32_t v = ((int32_t)k / kLongMin) * kLongMin;
    return v < kLongMin ? kLongMin : v;
}

// The same for the flattened kernel, whose four waves share a row at no extra cost
// per entry: only rows that alone would keep their workgroup busy for a good part of
// the launch are split, above min(8192, 3e-4 * entries) entries, and none below four
// times the mean.  F = 128, exact product, thresholds 512 / 2048 / 8192 / 16384 / never:
// 118 M entries in 2.45 M rows (rule: 8192): 6054 / 5826 / 5677 / 5647 / 5674 us; 25 M in
// 1.3 M (7466): 1941 / 1950 / 1953 / 1993 / 2030; 6.9 M in 1.3 M (2064): 875 / 853 / 846 /
// 865 / 864; 8.7 M in 0.7 M (2610): 577 / 567 / 575 / 586 / 586.
int32_t pick_flat_long_k(double entries, double mean)
{
    double k = entries * 3.0e-4 < (double)kFlatLongRow ? entries * 3.0e-4 : (double)kFlatLongRow;
    const double whole = 4.0 * mean < (double)INT32_MAX ? 4.0 * mean : (double)INT32_MAX;
    if (k < whole) k = (double)((int32_t)whole / kLongMin * kLongMin);
    return k < (double)kLongMin ? kLongMin : (int32_t)k;
}

// Per-call overrides, parsed from an es_launch_opts_t (absent = the heuristic).
struct Overrides {
    int logR = -1;             // rows_per_wave as a power of two, -1 = heuristic
    int G = 0;                 // lanes_per_row cap, 0 = heuristic, -1 = never slice
    int32_t long_k = 0;        // long-row threshold, 0 = heuristic
    int partition = 0;         // column-partitioned product: 0 = heuristic, 1 = on, -1 = off
    int kernel = 0;            // 0 = heuristic, 1 = row kernel, 2 = flattened kernel
};

int parse_opts(const es_launch_opts_t* opts, Overrides* ov)
{
    *ov = Overrides();
    if (!opts) return ES_OK;
    if (opts->column_partition < -1 || opts->column_partition > 1) return ES_ERR_INVALID_ARG;
    ov->partition = opts->column_partition;
    if (opts->kernel < 0 || opts->kernel > 2) return ES_ERR_INVALID_ARG;
    ov->kernel = opts->kernel;
    const int32_t rpw = opts->rows_per_wave;
    if (rpw != 0) {
        if (rpw < 1 || rpw > 64 || (rpw & (rpw - 1))) return ES_ERR_INVALID_ARG;
        int lg = 0;
        while ((1 << lg) < rpw) ++lg;
        ov->logR = lg;
    }
    const int32_t lanes = opts->lanes_per_row;
    if (lanes != 0 && lanes != -1 && lanes != 4 && lanes != 8 && lanes != 16 && lanes != 32 && lanes != 64)
        return ES_ERR_INVALID_ARG;
    ov->G = lanes;
    if (opts->long_row_threshold < 0) return ES_ERR_INVALID_ARG;
    ov->long_k = opts->long_row_threshold;
    return ES_OK;
}

// Rows per wave for the kernels that only walk the sampler (materialise,
// transpose): about one lane per kept entry of a typical row; a whole wave per
// row when rows may be much longer than typical (full mode, W above a wave).
int walk_logR(int64_t N, int64_t nnz, int32_t Wk)
{
    if (Wk > kWaveSize) return 0;
    double mean = (double)nnz / (double)N;
    if (mean > (double)Wk) mean = (double)Wk;
    int logR = 6;
    while (logR > 0 && (double)(kWaveSize >> logR) < mean) --logR;
    return logR;
}

// Everything the host decides about one launch.
struct Plan {
    Shape s;
    int logR;                  // log2(rows per wave)
    int32_t long_k;            // long-row threshold
    int64_t nblocks;           // row workgroups that carry rows
    int64_t per_xcd;           // row workgroups per XCD
    int64_t grid_x, grid_y;    // launch grid (long-row workgroups included in grid_x)
    int64_t long_blocks;       // leading long-row workgroups
    bool long_alone;           // ... each long row in one of them
    bool partition;            // column-partitioned product (kParts phases, needs a workspace)
    bool flat;                 // flattened kernel (es_flat_kernel.h) instead of the row kernel
};

int check_sizes(int64_t N, int64_t nnz, int32_t F, int32_t ldx, int32_t ldy, int32_t W, int32_t mode,
                int32_t norm)
{
    if (norm < ES_NORM_NONE || norm > ES_NORM_INV_DEGREE) return ES_ERR_INVALID_ARG;
    if (N < 0 || nnz < 0 || nnz > INT32_MAX || F < 1 || ldx < F || ldy < F) return ES_ERR_INVALID_ARG;
    if (mode != ES_FULL && mode != ES_BUCKET && mode != ES_FASTRAND) return ES_ERR_INVALID_ARG;
    if (mode != ES_FULL && W < 1) return ES_ERR_INVALID_ARG;
    return ES_OK;
}

// Bytes of workspace the column-partitioned product needs for N rows.
size_t part_workspace_bytes(int64_t N)
{
    return (size_t)N * kParts * sizeof(int32_t);
}

// Rows from which the flattened kernel on 32-column slices serves the column ranges of 16-byte-aligned rows.
bool part_flat_size(int64_t N) { return (double)N * 32.0 > 4.0e6; }

// Whether to run the column-partitioned product.  It pays when a row's piece inside one
// column range is long enough to amortise the extra pass over Y (kept entries per row well
// above kParts), when an XCD's eighth of a 32-column slice of X is of the order of its
// L2, and when X as a whole is so far beyond an L2 that whole rows miss.  The larger X (the lines its rows
// touch), the shorter the rows may be, so the lines are on the product of the two, `reach`.  The row form pays
// some 0.5 us per 100 rows whatever their length, so it asks for longer rows; wide rows share that over
// slices of full lines.  Time of whole rows over that of column ranges, exact product, uniform ids, `mean: ratio`:
//  * flattened kernel (`flat`), F = 32: 130 k rows (16.6 MB) 179: 0.94, 219: 1.01, 249: 1.08, 180 k 129: 0.95, 149:
//    1.00, 248: 1.20, 233 k 130: 1.02; rows that tile no line pay more for whole rows: F = 20, 130 k 130: 0.94,
//    179: 1.04, 180 k 129: 1.13, F = 28, 130 k 130: 1.19, 180 k 248: 1.68, F = 36, 130 k 130: 1.13, F = 48 1.21;
//    F = 64 1.09 (180 k 248: 1.45), F = 128, 170 k 150: 1.32; F = 16: 130 k 298: 0.97, 150 k 219: 0.98, 249: 1.02,
//    180 k 149: 0.94, 178: 1.02.
//  * row form, F = 64: 31 k (8.0 MB) 477: 0.92, 40 k 293: 0.83, 478: 1.12, 50 k 293: 0.93, 62 k (15.9 MB) 128: 0.59, 177:
//    0.75, 245: 0.92, 294: 1.04, 90 k 246: 1.02, 120 k 179: 0.87, 248: 0.98, 297: 1.09; F = 41: 50 k 477: 0.96, 62 k
//    294: 0.86, 478: 1.13, 120 k 248: 0.99, 297: 1.07; F = 205: 31 k 293: 1.03, 62 k 245: 1.02, 294: 1.14, 130 k 298:
//    0.99, 233 k 300: 0.87 (and 490: 0.96; two and more slices of rows that tile no line).
//  * row form, wide aligned rows: F = 128: 31 k (16 MB) 244: 0.93, 292: 1.05, 50 k 177: 0.87, 245: 1.06, 120 k 179: 0.91,
//    248: 1.10; F = 192: 62 k 177: 0.94, 216: 1.08; F = 256: 31 k 176: 0.90, 244: 1.13, 70 k 180: 1.00, 120 k 179: 0.88,
//    248: 1.08; F = 300: 62 k 216: 1.09, 120 k 241: 0.99.
//  * row form on rows of one line: F = 32: 120 k 297: 0.59, 484: 0.76; F = 17: 484: 0.75, F = 31: 297: 0.98, 484: 1.24.
// From 60 k aligned rows on the flattened kernel serves the rows of the last three (0.6 - 0.8 of the row form's time,
// make_plan); the lines stay where the row form crosses.
// Ids that cluster hit on whole rows too and gain less: 0.7 - 0.86 on the flattened kernel, 0.4 - 0.7 on the
// row form; sizes do not tell them apart.
bool pick_partition(int64_t N, double mean_kept, int32_t mode, int cols_per_block, int F, bool aligned, bool flat,
                    int force)
{
    if (mode == ES_BUCKET) return false;       // first-W entries crowd into the lowest column range
    if (N < kParts * 64) return false;
    if (force > 0) return true;
    if (force < 0) return false;
    // FastRand has to walk all W slots of a row once per column range to find the
    // ones that fall inside it; measured, that costs more than the locality
    // returns (233 k rows of mean 490, F = 64, W = 256: 0.8x), so it is only run on request
    if (mode == ES_FASTRAND) return false;
    if (mean_kept < 128.0) return false;
    const double share = (double)N * cols_per_block * 4.0 / kParts;
    if (share < 0.5e6 || share > 12.0e6) return false;
    const double table = (double)N * (F < 32 ? 32 : F) * 4.0;       // no gather moves less than a line
    const double reach = table * mean_kept;
    if (flat) return F <= 16 ? table >= 19.0e6 && reach >= 4.1e9 : F % 32 != 0 || reach >= 3.6e9;
    if (F <= (aligned ? 32 : 24)) return false;
    if (!aligned && F > 64 && N > 125000) return false;
    const bool wide = aligned && (F >= 256 || (F >= 128 && F % 64 == 0));
    return mean_kept >= (wide ? 216.0 : 256.0) && reach >= (wide ? 4.5e9 : 4.0e9);
}

// Whether the exact product of rows that tile whole lines runs sliced on the flattened kernel although X is below
// 0.3 GB: a slice of X is then of the order of an L2, or a community of its rows is.  32-column slices from 40 k to 140 k rows, where a
// 64-column one outgrows an L2 (`32`), else 64-column ones (`64`), over whole rows on the row kernel, uniform ids / ids that cluster:
//  * F = 96, 41 k - 140 k x 33 - 190: `32` 0.70 - 0.97 / 0.73 - 1.01
//  * F = 128, 15 k x 100: `64` 0.88 / 1.13, 30 k x 40 - 190: 0.78 - 0.86 / 0.92 - 1.00, 41 k - 140 k x 33 - 190: `32` 0.65 - 0.93 / 0.77 - 1.01, 140 k - 600 k: `64`
//    0.96 - 1.01 / 0.70 - 0.78; short rows, 60 k x 14: `64` 0.95 / 1.11, 100 k - 450 k x 11 - 29: 0.92 - 1.04 / 0.71 - 1.00, 500 k x 6 1.1 / 1.4
//  * F = 160 and 256 to 512, 15 k - 40 k x 33 - 190: `64` 0.51 - 0.82 / 0.71 - 0.98, 41 k - 140 k: `32` 0.56 - 0.93 / 0.66 - 0.91, more: `64` 0.88 - 0.98 / 0.55 - 0.78;
//    100 k and more x 11 - 29: `64` 0.85 - 0.96 / 0.61 - 0.93
//  * F = 64 and 192, whose rows the row kernel gathers best, gain nothing from `64` on uniform ids beyond 100 k rows (1.00 - 1.08 / 0.63 - 0.90), so
//    `32` there up to 200 k rows: 100 k - 140 k x 16 - 130 0.85 - 0.98 / 0.74 - 1.01, 155 k - 200 k x 16 - 130 0.93 - 1.01 / 0.73 - 0.90; beyond, F = 64 x 80 and more `64`
//    0.99 - 1.02 / 0.70 - 0.77 (x 66: 1.04), F = 192 x 64 and more up to 0.2 GB `32` 0.99 - 1.02 / 0.71 - 0.77 (`64`
//    1.02 - 1.04 / 0.63 - 0.67; x 40 - 50 `32` 1.00 - 1.05; 0.23 GB 1.03 / 0.71)
//    F = 64, 59 k x 140: 0.82 / 1.03
// Longer rows are where column ranges begin (pick_partition).  Rows that tile no line pay for every line twice (F = 100: 1.2 - 1.5),
// and sampled rows of ids that cluster 1.2 - 2.2 (F = 128).
// 64-column slices have to tile the row (F = 160, 104 k x 14: 1.18, F = 96, 39 k x 100: 1.12); short rows of uniform ids pay for large tables
// (F = 128, 515 k x 18, 0.26 GB: 1.02).  Returns the lanes of a slice, 0: none.
int slice_exact(int64_t N, double mean, int32_t mode, int F, double table)
{
    if (mode != ES_FULL || F % 32 != 0 || F < 64 || table < 15.0e6 || table >= 300.0e6) return 0;
    if (mean >= (F == 64 ? 150.0 : 200.0)) return 0;
    const bool narrow_gain = F == 64 || F == 192;
    if (N >= 40000 && N <= (narrow_gain ? 200000 : 140000) && mean >= (narrow_gain && N >= 100000 ? 16.0 : 32.0)) return 8;
    if (narrow_gain && N >= 100000) {
        if (N <= 200000) return 0;
        return F == 64 ? (mean >= 80.0 ? 16 : 0) : (mean >= 64.0 && table < 200.0e6 ? 8 : 0);
    }
    if (F % 64 != 0 || mean < (N >= 100000 ? 10.0 : 32.0)) return 0;
    return mean < 32.0 && table >= 250.0e6 ? 0 : 16;
}

// Launch shape for N >= 1 rows.  `aligned`: F and both row strides are
// multiples of 4 and both matrices are 16-byte aligned.  `crowded`: see es_run.
int make_plan(int64_t N, int64_t nnz, int32_t F, int32_t W, int32_t mode, bool aligned, bool backward,
              const Overrides& ov, bool have_workspace, Plan* p, int64_t crowded = 0)
{
    Shape s = pick_shape(F, aligned);
    if (backward) {                                        // see launch_backward
        s.vec = 1; s.aligned = false;
        s.G = next_pow2(F);
        if (s.G < 4) s.G = 4;
        if (s.G > 64) s.G = 64;
        s.CH = F > 128 ? 4 : F > 64 ? 2 : 1;
    }
    double mean = (double)nnz / (double)N;                 // mean entries a row keeps
    const double mean_stored = mean;
    if (mode != ES_FULL && mean > (double)W) mean = (double)W;

    // Column-partitioned product?  Decided on 32-column slices, its best width on
    // all but the smallest tables.
    const int slice_cols = F < 32 ? s.G * s.CH * s.vec : 32;
    p->partition = !backward && have_workspace &&
                   pick_partition(N, mean, mode, slice_cols, F, aligned,
                                  aligned && s.vec == 4 && ov.kernel != 1 && part_flat_size(N), ov.partition);

    // The flattened kernel applies to 128-bit accesses; FastRand in the
    // partitioned product needs the row kernel's per-row walk over all W slots.
    const bool flat_applies = !backward && s.vec == 4 && !(p->partition && mode == ES_FASTRAND);
    // chosen by rule only on 16-byte-aligned rows: 32-column slices of rows that do
    // not tile 128-byte lines fetch every line twice (F = 41, 233 k rows of mean 490,
    // sampled: 0.53x; in column ranges level with the row form: 2395 / 2131 us at mean 300)
    const bool flat_allowed = flat_applies && ov.kernel != 1 && s.aligned;

    // Column slicing: fewer lanes across the feature columns, the rows swept once
    // per slice, so that the part of X in use at a time is smaller.  A slice makes
    // every row short, which the row kernel pays for per row and the flattened
    // kernel does not; so the narrow (32-column) slices go with the flattened
    // kernel.  Both sides, us (profiles/ has the sweeps):
    //  * partitioned product: the flattened kernel from 60 k rows on (row form / this, F = 64: 60 k rows of mean 300
    //    511 / 391, 100 k of mean 400 989 / 688, 170 k of mean 300 1531 / 1024; F = 256, 100 k of mean 400 3665 / 2371).
    //    Slices of 64 columns, which halve what is paid per piece, of 32 above 125 k rows, where an XCD's share of a
    //    64-column slice no longer fits its L2 and where 32 tile 128-byte lines (32 / 64 columns, F = 64: 100 k of mean 400 834 /
    //    688, 170 k of mean 300 1042 / 1024, 233 k of mean 490 2071 / 2365; F = 100: 170 k of mean 150 1970 / 1680, 233 k of
    //    mean 300 5123 / 4501).
    //  * tables of 0.3 GB and more with F >= 128: 32-column slices on the flattened
    //    kernel, so that the X rows of a community of ids come nearer to an L2.
    //    Whole rows on the row kernel / this, 0.6 GB, F = 128: ids that cluster, mean
    //    50: exact 3137 / 2242, FastRand W = 64 1400 / 1208; mean 14: 1026 / 972, 623 /
    //    644; uniform ids, mean 50: 4078 / 4338, 1904 / 2159.  At 0.15 GB, clustered,
    //    mean 50: 561 / 500, 199 / 274.  With the row kernel forced, 64-column slices
    //    from 0.5 GB.
    //  * Bucket on rows several times longer than W: 32-column slices on the row
    //    kernel (its picks crowd into the lowest-numbered columns; 233 k rows, mean
    //    490, F = 64: W = 64 452 / 393, W = 16 79 / 69).
    // Elsewhere slicing only re-reads the CSR entries.
    int slice_G = 0;
    bool sliced_by_rule = false;
    bool want_flat = false;
    if (!backward && s.vec == 4) {
        if (ov.G > 0) slice_G = ov.G;
        else if (ov.G == 0) {
            const double table = (double)N * F * 4.0;
            const int exact_lanes = slice_exact(N, mean, mode, F, table);
            if (p->partition) {
                want_flat = flat_allowed && N >= 60000;
                slice_G = want_flat && F % 32 == 0 && part_flat_size(N) ? 8 : 16;
            } else if (flat_allowed && exact_lanes > 0) {
                want_flat = true;
                slice_G = exact_lanes;
            } else if (flat_allowed && F >= 128 && table >= 300.0e6) {
                want_flat = true;
                slice_G = 8;
            } else if (mode == ES_BUCKET && F >= 64 && mean_stored >= 4.0 * W) slice_G = 8;
            else if (F >= 128 && table >= 512.0e6) slice_G = 16;
            sliced_by_rule = slice_G > 0 && slice_G < s.G;
        }
    }
    if (slice_G > 0 && slice_G < s.G) {
        s.G = slice_G;                                     // narrower column blocks, more of them
        s.CH = 1;
    }
    // The flattened kernel's row accumulators hold one column block of at most
    // 256 columns, so wider rows are sliced to that.
    p->flat = flat_applies && (ov.kernel == 2 || (ov.kernel == 0 && want_flat));
    if (p->flat) s.CH = 1;
    p->s = s;

    int logR = pick_logR(s, mean);
    // a slice gathers less per row, so sampled rows share a wave in larger numbers
    if (sliced_by_rule && mode != ES_FULL && !p->partition && (64 >> (logR + 1)) >= s.G) ++logR;
    const int32_t force_logR = ov.logR;
    if (force_logR >= 0) {
        logR = force_logR;
        while ((64 >> logR) < s.G) --logR;                 // at least one edge slot per row
    }
    p->logR = logR;

    int64_t rows_per_block = (int64_t)kWavesPerBlock << logR;
    if (p->flat) {                                         // a workgroup's run: 1 or 2 rows per edge slot of its waves
        rows_per_block = flat_rows(s.G, mode == ES_FULL && !p->partition ? 1 : 2);
        logR = 0;
        while (((int64_t)kWavesPerBlock << logR) < rows_per_block) ++logR;
        p->logR = logR;
    }
    p->nblocks = (N + rows_per_block - 1) / rows_per_block;
    p->per_xcd = (p->nblocks + kNumXcd - 1) / kNumXcd;
    const int cols_per_block = s.G * s.CH * s.vec;
    p->grid_y = ((int64_t)F + cols_per_block - 1) / cols_per_block;

    // rows that may keep more than long_k entries exist only in full mode or
    // for W above the bound (nnz is a hint, so it does not gate the launch)
    double entries = (double)nnz;
    if (mode != ES_FULL && entries > (double)N * W) entries = (double)N * W;
    // Crowded rows: those that are not empty are about as long as the stored graph's, whatever the mean of
    // all, and four times that mean may be less than each of them; the threshold is at least twice the
    // stored mean.  Transposed Bucket product, split from four times the kept mean / from there (scatter): 10 k
    // rows of mean 390, W = 16, F = 128: 142 us / 43 (73); 30 k of mean 229, W = 22, F = 20: 103 / 52 (78); 233 k
    // of mean 488, W = 16, F = 20: 335 / 251 (375).  From the whole stored mean's four times the longest rows of graphs
    // with hubs hold the launch up (60 k of mean 279, W = 8, F = 64: 126 us, 85 from twice).
    const double row_mean = (double)crowded / (2.0 * (double)N) > mean ? (double)crowded / (2.0 * (double)N) : mean;
    p->long_k = p->flat ? pick_flat_long_k(entries, mean) : pick_long_k(s, logR, entries, F, row_mean);
    // the long-row part costs a second small launch and a scan of the row
    // pointers; below one tile per row that is more than the tail it removes
    if (mode != ES_FULL && p->long_k < kTileSlots) p->long_k = kTileSlots;
    if (ov.long_k > 0) p->long_k = ov.long_k;
    const bool may_be_long = mode == ES_FULL || W > p->long_k;
    p->long_blocks = may_be_long ? ((N + kLongScanRows - 1) / kLongScanRows) * kLongSplit : 0;
    p->grid_x = p->per_xcd * kNumXcd + p->long_blocks;
    // Long rows without atomics (es_spmm_small_kernel) save the launch that zeroes
    // such rows (2.5 us on the host, 1.5 us on the GPU) and cost a chain of round
    // trips per row, so the rule bounds the longest row there can be -- all columns of
    // a row are different, so min(entries, N) -- and how many there can be.  One row
    // of n entries, us on the GPU, this form / split with atomics: F = 16: n = 300: 4.8 /
    // 6.9, 3000: 6.6 / 7.2, 4000: 7.3 / 7.4, 6000: 8.6 / 7.8; F = 64: 1000: 6.4 / 8.8,
    // 2000: 8.4 / 8.8, 3000: 10.4 / 9.0; no long row at all: 2.8 / 4.3.
    const double longest = entries < (double)N ? entries : (double)N;
    p->long_alone = !backward && !p->flat && !p->partition && p->long_blocks > 0 &&
                    longest * (F + 64.0) <= 262144.0 && entries * (F + 64.0) <= 5.0 * 262144.0;
    if (p->partition && p->flat) {                         // one sweep per launch, no long-piece handling
        p->long_k = INT32_MAX;
        p->long_blocks = 0;
        p->grid_x = p->per_xcd * kNumXcd;
    } else if (p->partition) {
        // a wave serves kPartGroups consecutive rows, one at a time; every launch
        // sweeps the rows twice, pieces above long_k first (es_part_kernel.h)
        p->logR = 0;
        p->long_k = ov.long_k > 0 ? ov.long_k : kPartLongPiece;
        const int64_t rows_per_part_block = (int64_t)kWavesPerBlock * kPartGroups;
        p->nblocks = (N + rows_per_part_block - 1) / rows_per_part_block;
        p->per_xcd = (p->nblocks + kNumXcd - 1) / kNumXcd;
        p->long_blocks = p->per_xcd * kNumXcd;
        p->grid_x = 2 * p->long_blocks;
    }
    if (p->grid_x > INT32_MAX || p->grid_y > 65535) return ES_ERR_UNSUPPORTED;
    return ES_OK;
}

template <int G, int CH, int VEC, bool ALIGNED, bool WIDE>
hipError_t launch_partitioned(Args a, dim3 grid, int32_t* cuts, hipStream_t st)
{
    a.cuts = cuts;
    a.part_cols = (int32_t)((a.N + kParts - 1) / kParts);
    const uint32_t cb = (uint32_t)((a.N * kParts + kBlockThreads - 1) / kBlockThreads);
    hipLaunchKernelGGL(es_cuts_kernel, dim3(cb), dim3(kBlockThreads), 0, st, a.rowptr, a.colidx, a.N,
                       a.part_cols, cuts);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    for (int phase = 0; phase < kParts; ++phase) {
        a.phase = phase;
        hipLaunchKernelGGL((es_spmm_part_kernel<G, CH, VEC, ALIGNED, WIDE>), grid, dim3(kBlockThreads), 0, st, a);
        err = hipGetLastError();
        if (err != hipSuccess) return err;
    }
    return hipSuccess;
}

// Shared host path of es_spmm_norm (X -> Y) and es_spmm_backward (dY -> dX).  `crowded`
// > 0: the graph is the transpose of a Bucket sample of one of that many entries, whose
// rows get shorter from the first to the last, most of them empty: row workgroups go
// round the XCDs in order instead of a contiguous range each (row kernel), and the
// long-row threshold follows the stored graph (make_plan).
int es_run(const int32_t* rowptr, const int32_t* colidx, const float* vals, const float* X, float* Y,
           int64_t N, int64_t nnz, int32_t F, int32_t ldx, int32_t ldy, int32_t W, int32_t mode,
           uint64_t seed, int32_t norm, bool backward, const es_launch_opts_t* opts, void* workspace,
           size_t workspace_bytes, void* stream, int64_t crowded = 0)
{
    const int bad = check_sizes(N, nnz, F, ldx, ldy, W, mode, norm);
    if (bad != ES_OK) return bad;
    Overrides ov;
    const int bad_opts = parse_opts(opts, &ov);
    if (bad_opts != ES_OK) return bad_opts;
    if (N == 0) return ES_OK;
    if (!rowptr || !X || !Y) return ES_ERR_INVALID_ARG;
    if (nnz > 0 && !colidx) return ES_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(X) % 4 || reinterpret_cast<uintptr_t>(Y) % 4)
        return ES_ERR_INVALID_ARG;
    const bool aligned = (F % 4 == 0) && (ldx % 4 == 0) && (ldy % 4 == 0) &&
                         (reinterpret_cast<uintptr_t>(X) % 16 == 0) &&
                         (reinterpret_cast<uintptr_t>(Y) % 16 == 0);
    if (workspace && reinterpret_cast<uintptr_t>(workspace) % 16) return ES_ERR_INVALID_ARG;
    const bool have_ws = workspace && workspace_bytes >= part_workspace_bytes(N);
    Plan p;
    const int rc = make_plan(N, nnz, F, W, mode, aligned, backward, ov, have_ws, &p, crowded);
    if (rc != ES_OK) return rc;
    const Shape& s = p.s;

    Args a;
    a.rowptr = rowptr; a.colidx = colidx; a.vals = vals; a.X = X; a.Y = Y;
    a.N = N; a.seed = seed; a.F = F; a.ldx = ldx; a.ldy = ldy;
    a.W = (mode == ES_FULL) ? INT32_MAX : W;
    a.mode = mode; a.logR = p.logR; a.norm = norm; a.long_k = p.long_k;
    a.nblocks = (uint32_t)p.nblocks;
    a.blocks_per_xcd = crowded > 0 && !p.flat && !p.partition && !p.long_alone ? 0u : (uint32_t)p.per_xcd;
    a.long_blocks = (uint32_t)p.long_blocks;
    a.cuts = nullptr; a.part_cols = 0; a.phase = 0;

    const dim3 grid((uint32_t)p.grid_x, (uint32_t)p.grid_y);
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t err = hipErrorInvalidValue;
    // RowKey form: the gathered matrix is X (forward) or dX (backward, the
    // matrix passed as Y here); its largest row offset in RowKey units must fit 32 bits
    const int64_t gather_ld = backward ? ldy : ldx;
    const bool key_aligned = !backward && s.aligned;
    const int64_t stride_units = key_aligned ? gather_ld / 4 : gather_ld;
    const bool wide = (uint64_t)N * (uint64_t)stride_units > 0xFFFFFFFFull;
    a.stride_units = wide ? 0u : (uint32_t)stride_units;
#define ES_LAUNCH(G_, CH_, V_, A_, W_)                                                              \
    (p.partition ? launch_partitioned<G_, CH_, V_, A_, W_>(a, grid, static_cast<int32_t*>(workspace), st) \
                 : launch_forward<G_, CH_, V_, A_, W_>(a, grid, p.long_alone, st))
#define ES_CASE(G_, CH_, V_, A_)                                                          \
    if (!backward && !p.flat && s.G == G_ && s.CH == CH_ && s.vec == V_ && s.aligned == A_) \
        err = wide ? ES_LAUNCH(G_, CH_, V_, A_, true) : ES_LAUNCH(G_, CH_, V_, A_, false);
    ES_CASE(4, 1, 4, true) ES_CASE(8, 1, 4, true) ES_CASE(16, 1, 4, true) ES_CASE(32, 1, 4, true)
    ES_CASE(64, 1, 4, true) ES_CASE(64, 2, 4, true) ES_CASE(64, 4, 4, true)
    ES_CASE(4, 1, 4, false) ES_CASE(8, 1, 4, false) ES_CASE(16, 1, 4, false) ES_CASE(32, 1, 4, false)
    ES_CASE(64, 1, 4, false) ES_CASE(64, 2, 4, false) ES_CASE(64, 4, 4, false)
    ES_CASE(4, 1, 1, false)
#define ES_BWD(G_, CH_)                         \
    if (backward && s.G == G_ && s.CH == CH_)   \
        err = wide ? launch_backward<G_, CH_, true>(a, grid, st) : launch_backward<G_, CH_, false>(a, grid, st);
    ES_BWD(4, 1) ES_BWD(8, 1) ES_BWD(16, 1) ES_BWD(32, 1) ES_BWD(64, 1) ES_BWD(64, 2) ES_BWD(64, 4)
    // the run kernel's 32-bit form: byte offsets from one 24-bit multiply
    const uint64_t stride_bytes = (uint64_t)ldx * 4u;
    const bool flat_wide = N > (1 << 24) || stride_bytes >= (1u << 24) || (uint64_t)N * stride_bytes > kFlatMaxBytes;
#define ES_FLAT(G_, A_)                                                                         \
    if (p.flat && s.G == G_ && s.aligned == A_)                                                 \
        err = flat_wide ? launch_flat<G_, A_, true>(a, grid, p.partition, static_cast<int32_t*>(workspace), st)  \
                       : launch_flat<G_, A_, false>(a, grid, p.partition, static_cast<int32_t*>(workspace), st);
    ES_FLAT(4, true) ES_FLAT(8, true) ES_FLAT(16, true) ES_FLAT(32, true) ES_FLAT(64, true)
    ES_FLAT(4, false) ES_FLAT(8, false) ES_FLAT(16, false) ES_FLAT(32, false) ES_FLAT(64, false)
#undef ES_FLAT
#undef ES_BWD
#undef ES_CASE
#undef ES_LAUNCH
    return err == hipSuccess ? ES_OK : ES_ERR_LAUNCH;
}

int build_transposed(const int32_t* rowptr, const int32_t* colidx, const float* vals, int64_t N,
                     int64_t nnz, int32_t W, int32_t mode, uint64_t seed, int32_t norm, int32_t* out_ptr,
                     int32_t* out_end, int32_t* out_idx, float* out_vals, int32_t* out_pos, void* stream);

// Whether the pull backward tests entries against the rows' bits in LDS before it looks their rows up
// (es_pull_filtered_kernel).  That spares most of the lookups, but holds only 16 waves per compute unit, which gather less
// at a time: columns have to be long, the columns of dY that a mean row's kept entries gather (`gathered`; rows that tile no line
// cost another one) few, and the lookups' table beyond what an L2 serves also where ids cluster, which sizes do not
// show.  Time over that of es_pull_kernel, uniform ids / ids that cluster, 0.11 gathered <= mean unless said:
//  * 8 to 50 M entries: 0.61 - 1.06 / 0.85 - 1.38 (40 k rows of mean 310: 1.15 - 1.36, 60 k of 290: 0.96 - 1.36, 100 k of 268: 0.93 - 1.19,
//    150 k of 264: 0.87 - 1.14)
//  * from 50 M on, mean 257 to 280: 0.73 - 0.99 / 0.81 - 1.05, 281 to 300: 0.77 - 0.96 / 0.80 - 1.01; 300 to 370, ids that cluster, gathered up to 6
//    a mean entry 0.76 - 1.00, 6 to 9.1 0.81 - 1.05; 370 and more 0.61 - 0.95 / 0.73 - 1.00; gathered 9.1 to 12 a mean entry 0.80 - 1.11 / 0.87 - 1.12
//    whatever the mean, more 0.83 - 1.14 / 0.96 - 1.14
//  * fewer entries where the mean row is 400 and more, gathered at most 6 a mean entry: 70 k to 110 k rows 0.58 - 0.84 / 0.71 - 1.00 (the ids in 10, 24, 40 or 64
//    blocks); 60 k up to 1.02, 40 k up to 1.17
//  * F = 3: 0.77 - 1.08; where the lines below hold, F = 8: 0.64 - 1.01, F = 16 to 1300 0.58 - 1.00 (1600 calls)
bool pull_filtered(int64_t N, int64_t nnz, int32_t F, int32_t W, int32_t mode, uint64_t seed)
{
    if (mode != ES_FASTRAND || seed == 0 || N > kPullFilterRows || F < 8) return false;
    const double mean = (double)nnz / (double)N;
    const double gathered = (mean < W ? mean : W) * (F % 32 ? (double)F + 31.0 : (double)F);
    if (nnz < 50000000) return N >= 70000 && mean >= 400.0 && gathered <= 6.0 * mean;
    return gathered <= 28.0 * (mean - 270.0) && 0.11 * gathered <= mean;
}

// Entries a column from which the passes of es_pull_kernel hold 8 chunks (8 / 4, us: mean 60, W = 8 147 / 133, mean 90, ids that
// cluster 285 / 263, 110, Bucket W = 8 52.6 / 54.7, 150, W = 8 62.6 / 63.2 and rotated 414 / 403, 300, Bucket W = 8 33.7 / 44.3).
constexpr int64_t kPullLongColumn = 96;

struct PullGraph {
    const int32_t *ptr, *row, *idx, *slot;
    const float* vals;
    const int2* rows;                  // this call's (length, rotation) per row of A
};

template <int G, int CH, int VEC, bool ALIGNED, int MAXC>
void launch_pull_passes(const Args& a, const PullGraph& t, dim3 grid, bool wide, hipStream_t st)
{
    if (wide)
        hipLaunchKernelGGL((es_pull_kernel<G, CH, VEC, ALIGNED, true, MAXC>), grid, dim3(kBlockThreads), 0, st, a, t.ptr,
                           t.row, t.idx, t.slot, t.vals, t.rows);
    else
        hipLaunchKernelGGL((es_pull_kernel<G, CH, VEC, ALIGNED, false, MAXC>), grid, dim3(kBlockThreads), 0, st, a, t.ptr,
                           t.row, t.idx, t.slot, t.vals, t.rows);
}

template <int G, int CH, int VEC, bool ALIGNED>
hipError_t launch_pull(const Args& a, const PullGraph& t, dim3 grid, int64_t nnz, bool wide, bool filtered, hipStream_t st)
{
    if constexpr (VEC == 4) {                              // rows of fewer than 4 columns are never filtered
        if (filtered) {
            const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(es_pull_filtered_kernel<G, CH, VEC, ALIGNED>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, kPullLdsBytes);
            if (err != hipSuccess) return err;
            const uint32_t lds = (uint32_t)(kPullTileBytes + (a.N + 7) / 8 * (int64_t)sizeof(uint32_t));
            const int64_t blocks = (a.N + kPullWaves - 1) / kPullWaves;
            const dim3 fgrid((uint32_t)(blocks < kComputeUnits ? blocks : kComputeUnits), grid.y);
            hipLaunchKernelGGL((es_pull_filtered_kernel<G, CH, VEC, ALIGNED>), fgrid, dim3(kPullThreads), lds, st, a, t.ptr,
                               t.row, t.slot, t.vals, t.rows);
            return hipGetLastError();
        }
    }
    const bool rotated = a.mode == ES_FASTRAND && a.seed != 0;
    if (nnz < kPullLongColumn * a.N &&
        pull_short_form<G, CH, ALIGNED>(rotated, pull_needs_rows(a.mode, a.seed, a.norm), nnz <= 12 * a.N))
        launch_pull_passes<G, CH, VEC, ALIGNED, kPullChunks>(a, t, grid, wide, st);
    else
        launch_pull_passes<G, CH, VEC, ALIGNED, 8>(a, t, grid, wide, st);
    return hipGetLastError();
}

// Layout of the binned transposed product's workspace (es_bin_kernel.h); bytes == 0:
// the scatter is the faster form, or this one does not apply.
struct BinPlan {
    int64_t capacity;                  // kept entries at most
    int log_width, nbins, walkers;
    bool local;                        // a walker's entries fit its registers (es_bin_local_kernel)
    size_t records, counts, base, t_ptr, t_row, t_val, bytes;
};

// How the exact product runs on the transposed sample: the row kernel on whole rows.  Time of the whole call with the forward
// rule's form (slices on the flattened kernel) over that: Bucket samples crowd into few rows, which the row kernel deals round
// the XCDs: 233 k rows of mean 483, F = 128, W = 16 3.18, W = 64 2.17, 170 k of 13, F = 128 1.14, 1 M of 47, ids that cluster, W = 8 / 64
// 1.25 / 0.89.  FastRand, uniform ids: 60 k of 59, F = 256, W = 64 0.65, 170 k of 13, F = 128 1.12, 1 M of 13 1.14 - 1.18, 2 M of 19
// 0.92 - 1.12; ids that cluster: 60 k of 48, F = 256 1.36 - 1.41, 1 M of 47, W = 16 / 64 0.93 - 0.96 / 0.78 - 0.84, W = 8 1.14.
constexpr es_launch_opts_t kBinProduct = {0, 0, 0, -1, 1};

// Whether the scatter would send so many requests that sorting is the faster.  From 1.1 M on it is, counted on the
// min(nnz, N W) entries that can be kept; below 0.7 M the two are level or the scatter is ahead.  Between
// them the line is on the entries that are kept: nearly all of those where nnz and N W are far apart, half of
// them in power-law rows whose mean is near W, so nnz N W / (nnz + N W) is asked for.  Time of this form over the scatter's, 2.5 k
// to 700 k rows, W = 1 to 4096, by requests per entry and that estimate:
//  * 2 (F <= 32): below 0.52 M 0.6 - 1.23 (90 k power-law rows, W = 4 of 4: 0.71 M at most 25.9 / 30.6 us, 62 k, W = 8: 0.88 M
//    27.7 / 30.6), from there 0.51 - 0.99.  More rows than the walkers' threads (five launches instead of two): 0.98 - 1.145 up
//    to 1.1 M (350 k rows, 0.70 M: 54.4 / 62.2).
//  * 3 and 4: below 0.44 M 0.47 - 1.10 (26 k power-law rows, W = 8, F = 49: 0.74 M 25.4 / 28.1), from there 0.38 - 1.01
//  * 5 and more: from 0.36 M on 0.32 - 0.95
bool enough_requests(int64_t N, int64_t nnz, int32_t F, int32_t W)
{
    const int64_t per_entry = ((int64_t)F + 15) / 16;
    const double most = (double)(nnz < N * W ? nnz : N * W) * (double)per_entry;
    if (most >= 1.1e6) return true;
    if (most < 0.7e6 || (per_entry <= 2 && N > (int64_t)kBinWalkers * kBinLocalRows)) return false;
    const double stored = (double)nnz, bound = (double)N * (double)W;
    return stored * bound / (stored + bound) * (double)per_entry >= (per_entry <= 2 ? 0.52e6 : per_entry <= 4 ? 0.44e6 : 0.36e6);
}

// Where the lines lie: the scatter moves one 64-byte request per kept entry and 16
// columns, 20.5 G of them a second; this form takes some 20 us of launches and first
// round trips, 0.03 us per 1000 kept entries to sort them, and the gather.  us, scatter / this:
//  * enough requests (enough_requests); F = 128: 170 k rows, 2.1 M entries at most 406 / 110; F = 64: 233 k, 14.9 M
//    2923 / 1048; a column that all rows hold, 20 k to 1 M rows: always this.
//  * F <= 16: with one request per entry the sort costs what it saves: 160 k, 2.0 M 60 / 66; 2.4 M rows,
//    10.5 M 382 / 399; 160 k, 7.6 M 191 / 159.
//  * rows longer than a line of 128 bytes of which few entries are kept: count and fill wait for
//    a line each per row (Bucket) or per kept entry (FastRand), the scatter for one, with more waves to wait in.
//    The more so the longer the rows, so the row has to be worth the more requests.  233 k rows of mean 488,
//    F = 20 (2 requests an entry), Bucket and FastRand: W = 4 113 / 182 and 121 / 206, W = 8 202 / 209 and 212 / 260,
//    W = 16 382 / 244 and 388 / 362; F = 64, W = 4: 209 / 181 and 210 / 234; mean 200, F = 20, W = 4: 106 / 117 and
//    106 / 150, W = 8 196 / 141 and 196 / 192; 170 k of mean 99, W = 4: 77 / 77 and 76 / 92.  Ids that cluster
//    cross earlier (mean 385, F = 64, FastRand W = 4: 0.77 of the scatter's time), hubs earlier still.
BinPlan plan_bins(int64_t N, int64_t nnz, int32_t F, int32_t W, int32_t mode)
{
    BinPlan p = {};
    if (mode != ES_BUCKET && mode != ES_FASTRAND) return p;    // exact rows have no bound on their length
    if (W < 1 || W > kBinMaxW || F <= 16 || N < 1 || N > (1 << kBinRowBits) || nnz < 1 || nnz > INT32_MAX) return p;
    p.capacity = nnz < N * W ? nnz : N * W;
    if (!enough_requests(N, nnz, F, W)) return p;
    const double mean = (double)nnz / (double)N, row_requests = (double)W * ((F + 15) / 16);
    if (mean > 32.0 && mean > W && row_requests < (mode == ES_FASTRAND ? 5.0 + mean / 25.0 : 1.5 + mean / 46.0)) return p;
    // only where both the gather this form ends in (some million columns are more than its grid covers) and the
    // scatter can run, so that a call is refused or accepted whatever workspace there is, and refused before a launch
    Plan product;
    Overrides ov;
    if (parse_opts(&kBinProduct, &ov) != ES_OK ||
        make_plan(N, p.capacity, F, 0, ES_FULL, false, false, ov, false, &product) != ES_OK ||
        make_plan(N, nnz, F, W, mode, false, true, Overrides(), false, &product) != ES_OK) return p;
    // blocks of N / 1024 columns up to N / 2048: enough workgroups for the sort, runs of records long enough to write
    while (p.log_width < 32 - kBinRowBits && (N >> (p.log_width + 1)) >= 1024) ++p.log_width;
    p.nbins = (int)((N + ((int64_t)1 << p.log_width) - 1) >> p.log_width);
    p.walkers = (int)((N + kWaveSize - 1) / kWaveSize < kBinWalkers ? (N + kWaveSize - 1) / kWaveSize : kBinWalkers);
    const auto take = [&p](size_t bytes) { const size_t at = p.bytes; p.bytes += (bytes + 255) / 256 * 256; return at; };
    const int64_t walker_rows = (N + p.walkers - 1) / p.walkers;
    p.local = walker_rows <= kBinLocalRows && walker_rows * W <= (int64_t)kBinLocalRows * kBinLocalPer;
    p.records = take((size_t)p.capacity * sizeof(uint2));
    p.counts = take((size_t)p.walkers * (p.local ? p.nbins + 1 : p.nbins) * sizeof(int32_t));
    p.base = take((size_t)(p.local ? p.walkers : p.nbins + 1) * sizeof(int32_t));
    p.t_ptr = take((size_t)(N + 1) * sizeof(int32_t));
    p.t_row = take((size_t)p.capacity * sizeof(int32_t));
    p.t_val = take((size_t)p.capacity * sizeof(float));
    return p;
}

// The transposed product through `workspace`, laid out by plan_bins.
int run_binned(const int32_t* rowptr, const int32_t* colidx, const float* vals, const float* dY, float* dX,
               int64_t N, int64_t nnz, int32_t F, int32_t ldy, int32_t ldx, int32_t W, int32_t mode, uint64_t seed,
               int32_t norm, const BinPlan& p, void* workspace, void* stream)
{
    unsigned char* ws = static_cast<unsigned char*>(workspace);
    BinArgs a;
    a.rowptr = rowptr; a.colidx = colidx; a.vals = vals;
    a.records = reinterpret_cast<uint2*>(ws + p.records);
    a.counts = reinterpret_cast<int32_t*>(ws + p.counts);
    a.base = reinterpret_cast<int32_t*>(ws + p.base);
    a.t_ptr = reinterpret_cast<int32_t*>(ws + p.t_ptr);
    a.t_row = reinterpret_cast<int32_t*>(ws + p.t_row);
    a.t_val = reinterpret_cast<float*>(ws + p.t_val);
    a.N = N; a.capacity = p.capacity; a.seed = seed; a.W = W; a.mode = mode; a.norm = norm;
    a.log_width = p.log_width; a.nbins = p.nbins; a.walkers = p.walkers;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (p.local) {
        const uint32_t lds = (uint32_t)(p.nbins + 1) * sizeof(int32_t);
        hipLaunchKernelGGL(es_bin_local_kernel, dim3((uint32_t)p.walkers), dim3(kBinLocalRows), lds, st, a);
        if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
        hipLaunchKernelGGL(es_bin_sort_kernel<true>, dim3((uint32_t)p.nbins), dim3(kBlockThreads), 0, st, a);
        if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
    } else {
        const uint32_t lds = (uint32_t)p.nbins * sizeof(int32_t);
        hipLaunchKernelGGL(es_bin_walk_kernel<false>, dim3((uint32_t)p.walkers), dim3(kBinThreads), lds, st, a);
        if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
        hipLaunchKernelGGL(es_bin_scan_kernel, dim3((uint32_t)(p.nbins + kWaveSize - 1) / kWaveSize), dim3(kBinScanThreads), 0, st, a);
        if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
        hipLaunchKernelGGL(es_bin_base_kernel, dim3(1), dim3(kBinScanThreads), 0, st, a);
        if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
        hipLaunchKernelGGL(es_bin_walk_kernel<true>, dim3((uint32_t)p.walkers), dim3(kBinThreads), lds, st, a);
        if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
        hipLaunchKernelGGL(es_bin_sort_kernel<false>, dim3((uint32_t)p.nbins), dim3(kBlockThreads), 0, st, a);
        if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
    }
    return es_run(a.t_ptr, a.t_row, a.t_val, dY, dX, N, p.capacity, F, ldy, ldx, 0, ES_FULL, 0, ES_NORM_NONE, false,
                  &kBinProduct, nullptr, 0, stream, mode == ES_BUCKET ? nnz : 0);
}

}  // namespace

extern "C" {

const char* es_spmm_status_string(int status)
{
    switch (status) {
        case ES_OK: return "ES_OK";
        case ES_ERR_INVALID_ARG: return "ES_ERR_INVALID_ARG: null pointer, negative size, ld < F, W < 1 or unknown mode";
        case ES_ERR_UNSUPPORTED:
            return "ES_ERR_UNSUPPORTED: shape outside what the kernels cover (or more rows than "
                   "es_spmm_static_ws holds a workspace for: use es_spmm_ws)";
        case ES_ERR_LAUNCH: return "ES_ERR_LAUNCH: the HIP runtime rejected the launch";
        default: return "unknown es_spmm status";
    }
}

int32_t es_spmm_max_W(int32_t F) { return F < 1 ? 0 : INT32_MAX; }

int32_t es_spmm_tile_slots(int32_t rows_per_wave)
{
    if (rows_per_wave == 0) return kTileSlots;
    if (rows_per_wave < 1 || rows_per_wave > 64 || (rows_per_wave & (rows_per_wave - 1))) return 0;
    return kTileSlots / rows_per_wave;
}

int es_spmm(const int32_t* rowptr, const int32_t* colidx, const float* vals, const float* X,
            float* Y, int64_t N, int64_t nnz, int32_t F, int32_t ldx, int32_t ldy, int32_t W,
            int32_t mode, uint64_t seed, void* stream)
{
    return es_spmm_norm(rowptr, colidx, vals, X, Y, N, nnz, F, ldx, ldy, W, mode, seed, ES_NORM_NONE,
                        stream);
}

int es_spmm_norm(const int32_t* rowptr, const int32_t* colidx, const float* vals, const float* X,
                 float* Y, int64_t N, int64_t nnz, int32_t F, int32_t ldx, int32_t ldy, int32_t W,
                 int32_t mode, uint64_t seed, int32_t norm, void* stream)
{
    return es_run(rowptr, colidx, vals, X, Y, N, nnz, F, ldx, ldy, W, mode, seed, norm, false, nullptr,
                  nullptr, 0, stream);
}

int es_spmm_ex(const int32_t* rowptr, const int32_t* colidx, const float* vals, const float* X,
               float* Y, int64_t N, int64_t nnz, int32_t F, int32_t ldx, int32_t ldy, int32_t W,
               int32_t mode, uint64_t seed, int32_t norm, const es_launch_opts_t* opts, void* stream)
{
    return es_run(rowptr, colidx, vals, X, Y, N, nnz, F, ldx, ldy, W, mode, seed, norm, false, opts,
                  nullptr, 0, stream);
}

size_t es_spmm_workspace_bytes(int64_t N) { return N < 0 ? 0 : part_workspace_bytes(N); }

int es_spmm_ws(const int32_t* rowptr, const int32_t* colidx, const float* vals, const float* X,
               float* Y, int64_t N, int64_t nnz, int32_t F, int32_t ldx, int32_t ldy, int32_t W,
               int32_t mode, uint64_t seed, int32_t norm, const es_launch_opts_t* opts, void* workspace,
               size_t workspace_bytes, void* stream)
{
    return es_run(rowptr, colidx, vals, X, Y, N, nnz, F, ldx, ldy, W, mode, seed, norm, false, opts,
                  workspace, workspace_bytes, stream);
}

int es_spmm_static_ws(const int32_t* rowptr, const int32_t* colidx, const float* vals, const float* X,
                      float* Y, int64_t N, int64_t nnz, int32_t F, int32_t ldx, int32_t ldy, int32_t W,
                      int32_t mode, uint64_t seed, int32_t norm, const es_launch_opts_t* opts, void* stream)
{
    // argument errors first (as every entry point), then the capacity of the
    // static array, then -- the first thing that touches the GPU -- its address
    const int bad = check_sizes(N, nnz, F, ldx, ldy, W, mode, norm);
    if (bad != ES_OK) return bad;
    Overrides ov;
    const int bad_opts = parse_opts(opts, &ov);
    if (bad_opts != ES_OK) return bad_opts;
    if (N > ES_SPMM_STATIC_WS_MAX_ROWS) return ES_ERR_UNSUPPORTED;
    if (N == 0) return ES_OK;
    if (!rowptr || !X || !Y || (nnz > 0 && !colidx)) return ES_ERR_INVALID_ARG;
    void* ws = nullptr;
    const int rc = static_scratch_address(&ws);
    if (rc != ES_OK) return rc;
    return es_run(rowptr, colidx, vals, X, Y, N, nnz, F, ldx, ldy, W, mode, seed, norm, false, opts, ws,
                  sizeof(scratch), stream);
}

int es_spmm_backward(const int32_t* rowptr, const int32_t* colidx, const float* vals,
                     const float* dY, float* dX, int64_t N, int64_t nnz, int32_t F, int32_t ldy,
                     int32_t ldx, int32_t W, int32_t mode, uint64_t seed, int32_t norm, void* stream)
{
    return es_run(rowptr, colidx, vals, dY, dX, N, nnz, F, ldy, ldx, W, mode, seed, norm, true, nullptr,
                  nullptr, 0, stream);
}

size_t es_spmm_backward_workspace_bytes(int64_t N, int64_t nnz, int32_t F, int32_t W, int32_t mode)
{
    return plan_bins(N, nnz, F, W, mode).bytes;
}

int es_spmm_backward_ws(const int32_t* rowptr, const int32_t* colidx, const float* vals,
                        const float* dY, float* dX, int64_t N, int64_t nnz, int32_t F, int32_t ldy,
                        int32_t ldx, int32_t W, int32_t mode, uint64_t seed, int32_t norm,
                        void* workspace, size_t workspace_bytes, void* stream)
{
    const BinPlan p = plan_bins(N, nnz, F, W, mode);
    const bool sound = check_sizes(N, nnz, F, ldy, ldx, W, mode, norm) == ES_OK && rowptr && colidx && dY && dX &&
                       reinterpret_cast<uintptr_t>(dY) % 4 == 0 && reinterpret_cast<uintptr_t>(dX) % 4 == 0;
    if (reinterpret_cast<uintptr_t>(workspace) % 256) return ES_ERR_INVALID_ARG;
    if (sound && workspace && p.bytes && workspace_bytes >= p.bytes)
        return run_binned(rowptr, colidx, vals, dY, dX, N, nnz, F, ldy, ldx, W, mode, seed, norm, p, workspace, stream);
    return es_run(rowptr, colidx, vals, dY, dX, N, nnz, F, ldy, ldx, W, mode, seed, norm, true, nullptr,
                  nullptr, 0, stream);
}

int es_spmm_backward_ex(const int32_t* rowptr, const int32_t* colidx, const float* vals,
                        const float* dY, float* dX, int64_t N, int64_t nnz, int32_t F, int32_t ldy,
                        int32_t ldx, int32_t W, int32_t mode, uint64_t seed, int32_t norm,
                        const es_launch_opts_t* opts, void* stream)
{
    return es_run(rowptr, colidx, vals, dY, dX, N, nnz, F, ldy, ldx, W, mode, seed, norm, true, opts,
                  nullptr, 0, stream);
}

int es_spmm_launch_info(int64_t N, int64_t nnz, int32_t F, int32_t ldx, int32_t ldy, int32_t W,
                        int32_t mode, int32_t aligned16, int32_t backward,
                        const es_launch_opts_t* opts, es_launch_info_t* info)
{
    if (!info) return ES_ERR_INVALID_ARG;
    Overrides ov;
    const int bad_opts = parse_opts(opts, &ov);
    if (bad_opts != ES_OK) return bad_opts;
    const int bad = check_sizes(N, nnz, F, ldx, ldy, W, mode, ES_NORM_NONE);
    if (bad != ES_OK) return bad;
    if (N == 0) return ES_ERR_INVALID_ARG;
    const bool aligned = aligned16 && (F % 4 == 0) && (ldx % 4 == 0) && (ldy % 4 == 0);
    Plan p;
    const int rc = make_plan(N, nnz, F, W, mode, aligned, backward != 0, ov, true, &p);
    if (rc != ES_OK) return rc;
    info->vector_width = p.s.vec;
    info->aligned = p.s.aligned ? 1 : 0;
    info->lanes_per_row = p.s.G;
    info->chunks_per_lane = p.s.CH;
    info->rows_per_wave = 1 << p.logR;
    info->edge_slots = p.flat ? 64 / p.s.G : (64 >> p.logR) / p.s.G;
    info->loads_in_flight = 8 / p.s.CH;
    info->tile_slots_per_row = kTileSlots >> p.logR;
    info->long_row_threshold = p.long_k;
    info->long_row_workgroups = p.long_blocks;
    info->grid_x = p.grid_x;
    info->grid_y = p.grid_y;
    info->flattened = p.flat ? 1 : 0;
    info->column_ranges = p.partition ? kParts : 1;
    return ES_OK;
}

int es_spmm_materialize(const int32_t* rowptr, const int32_t* colidx, const float* vals, int64_t N,
                        int64_t nnz, int32_t W, int32_t mode, uint64_t seed, int32_t* out_rowptr,
                        int32_t* out_colidx, float* out_vals, void* stream)
{
    if (N < 0 || nnz < 0 || nnz > INT32_MAX) return ES_ERR_INVALID_ARG;
    if (mode != ES_FULL && mode != ES_BUCKET && mode != ES_FASTRAND) return ES_ERR_INVALID_ARG;
    if (mode != ES_FULL && W < 1) return ES_ERR_INVALID_ARG;
    if (!out_rowptr) return ES_ERR_INVALID_ARG;
    if (N > 0 && (!rowptr || !out_colidx || !out_vals)) return ES_ERR_INVALID_ARG;
    if (nnz > 0 && !colidx) return ES_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int32_t Wk = (mode == ES_FULL) ? INT32_MAX : W;
    const int64_t nscan = N == 0 ? 1 : (N + kScanRows - 1) / kScanRows;
    if (nscan > INT32_MAX) return ES_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(es_kept_scan_local_kernel, dim3((uint32_t)nscan), dim3(kBlockThreads), 0, st,
                       rowptr, N, Wk, mode, out_rowptr);
    if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
    if (N == 0) return ES_OK;
    if (nscan > 1) {
        hipLaunchKernelGGL(es_kept_scan_blocks_kernel, dim3(1), dim3(kBlockThreads), 0, st, N, out_rowptr);
        if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
        hipLaunchKernelGGL(es_kept_scan_add_kernel, dim3((uint32_t)(nscan - 1)), dim3(kBlockThreads), 0,
                           st, N, out_rowptr);
        if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
    }
    const int logR = walk_logR(N, nnz, Wk);
    const int64_t rows_per_block = (int64_t)kWavesPerBlock << logR;
    const int64_t nblocks = (N + rows_per_block - 1) / rows_per_block;
    if (nblocks > INT32_MAX) return ES_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(es_materialize_kernel, dim3((uint32_t)nblocks), dim3(kBlockThreads), 0, st,
                       rowptr, colidx, vals, N, Wk, mode, seed, logR, out_rowptr, out_colidx, out_vals);
    return hipGetLastError() == hipSuccess ? ES_OK : ES_ERR_LAUNCH;
}

int es_spmm_materialize_transposed(const int32_t* rowptr, const int32_t* colidx, const float* vals,
                                   int64_t N, int64_t nnz, int32_t W, int32_t mode, uint64_t seed,
                                   int32_t norm, int32_t* out_ptr, int32_t* out_end, int32_t* out_idx,
                                   float* out_vals, void* stream)
{
    return build_transposed(rowptr, colidx, vals, N, nnz, W, mode, seed, norm, out_ptr, out_end, out_idx,
                            out_vals, nullptr, stream);
}

int es_spmm_transpose_graph(const int32_t* rowptr, const int32_t* colidx, const float* vals, int64_t N,
                            int64_t nnz, int32_t* t_ptr, int32_t* t_end, int32_t* t_row, int32_t* t_idx,
                            int32_t* t_slot, float* t_vals, int32_t* t_pinv, void* stream)
{
    if (N > 0 && (!t_idx || !t_slot || !t_pinv)) return ES_ERR_INVALID_ARG;
    // t_idx first receives every entry's CSR position, then becomes its entry number
    const int rc = build_transposed(rowptr, colidx, vals, N, nnz, 0, ES_FULL, 0, ES_NORM_NONE, t_ptr, t_end,
                                    t_row, t_vals, t_idx, stream);
    if (rc != ES_OK || N == 0) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t pb = (N + kBlockThreads - 1) / kBlockThreads;
    if (pb > INT32_MAX) return ES_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(es_pinv_kernel, dim3((uint32_t)pb), dim3(kBlockThreads), 0, st, rowptr, N, t_pinv);
    if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
    int64_t eb = (nnz + kBlockThreads - 1) / kBlockThreads;
    if (eb > 65536) eb = 65536;
    if (eb > 0) {
        hipLaunchKernelGGL(es_pull_entries_kernel, dim3((uint32_t)eb), dim3(kBlockThreads), 0, st, rowptr,
                           t_pinv, t_row, nnz, t_idx, t_slot);
        if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
    }
    return ES_OK;
}

int es_spmm_backward_pull(const int32_t* rowptr, const int32_t* t_ptr, const int32_t* t_row,
                          const int32_t* t_idx, const int32_t* t_slot, const float* t_vals,
                          const int32_t* t_pinv, int32_t* t_rows, const float* dY, float* dX, int64_t N,
                          int64_t nnz, int32_t F, int32_t ldy, int32_t ldx, int32_t W, int32_t mode,
                          uint64_t seed, int32_t norm, void* stream)
{
    const int bad = check_sizes(N, nnz, F, ldy, ldx, W, mode, norm);
    if (bad != ES_OK) return bad;
    if (N == 0) return ES_OK;
    if (!rowptr || !t_ptr || !dY || !dX) return ES_ERR_INVALID_ARG;
    if (!t_pinv || !t_rows || reinterpret_cast<uintptr_t>(t_rows) % 8) return ES_ERR_INVALID_ARG;
    if (nnz > 0 && (!t_row || !t_idx || !t_slot || !t_vals)) return ES_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(dY) % 4 || reinterpret_cast<uintptr_t>(dX) % 4) return ES_ERR_INVALID_ARG;
    const bool aligned = (F % 4 == 0) && (ldx % 4 == 0) && (ldy % 4 == 0) &&
                         (reinterpret_cast<uintptr_t>(dY) % 16 == 0) &&
                         (reinterpret_cast<uintptr_t>(dX) % 16 == 0);
    const Shape s = pick_shape(F, aligned);
    Args a;
    a.rowptr = rowptr; a.colidx = nullptr; a.vals = nullptr; a.X = dY; a.Y = dX;
    a.N = N; a.seed = seed; a.F = F; a.ldx = ldy; a.ldy = ldx;
    a.W = (mode == ES_FULL) ? INT32_MAX : W;
    a.mode = mode; a.logR = 0; a.norm = norm; a.long_k = INT32_MAX;
    const int64_t nblocks = (N + kWavesPerBlock - 1) / kWavesPerBlock;
    const int64_t per_xcd = (nblocks + kNumXcd - 1) / kNumXcd;
    a.nblocks = (uint32_t)nblocks; a.blocks_per_xcd = (uint32_t)per_xcd; a.long_blocks = 0;
    a.cuts = nullptr; a.part_cols = 0; a.phase = 0;
    const int cols_per_block = s.G * s.CH * s.vec;
    const int64_t grid_y = ((int64_t)F + cols_per_block - 1) / cols_per_block;
    if (per_xcd * kNumXcd > INT32_MAX || grid_y > 65535) return ES_ERR_UNSUPPORTED;
    const int64_t stride_units = s.aligned ? ldy / 4 : ldy;          // rows of dY are what gets gathered
    const bool wide = (uint64_t)N * (uint64_t)stride_units > 0xFFFFFFFFull;
    a.stride_units = wide ? 0u : (uint32_t)stride_units;
    const dim3 grid((uint32_t)(per_xcd * kNumXcd), (uint32_t)grid_y);
    hipStream_t st = static_cast<hipStream_t>(stream);
    // per-row (length, rotation) of this call
    int2* rows = reinterpret_cast<int2*>(t_rows);
    const int64_t rb = (N + kBlockThreads - 1) / kBlockThreads;
    if (rb > INT32_MAX) return ES_ERR_UNSUPPORTED;
    if (pull_needs_rows(mode, seed, norm)) {
        hipLaunchKernelGGL(es_pull_rows_kernel, dim3((uint32_t)rb), dim3(kBlockThreads), 0, st, rowptr, t_pinv, N,
                           mode, seed, a.W, rows);
        if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
    }
    const PullGraph t = {t_ptr, t_row, t_idx, t_slot, t_vals, rows};
    const bool filtered = !wide && pull_filtered(N, nnz, F, W, mode, seed);
    hipError_t err = hipErrorInvalidValue;
#define ES_PULL(G_, CH_, V_, A_)                                         \
    if (s.G == G_ && s.CH == CH_ && s.vec == V_ && s.aligned == A_)      \
        err = launch_pull<G_, CH_, V_, A_>(a, t, grid, nnz, wide, filtered, st);
    ES_PULL(4, 1, 4, true) ES_PULL(8, 1, 4, true) ES_PULL(16, 1, 4, true) ES_PULL(32, 1, 4, true)
    ES_PULL(64, 1, 4, true) ES_PULL(64, 2, 4, true) ES_PULL(64, 4, 4, true)
    ES_PULL(4, 1, 4, false) ES_PULL(8, 1, 4, false) ES_PULL(16, 1, 4, false) ES_PULL(32, 1, 4, false)
    ES_PULL(64, 1, 4, false) ES_PULL(64, 2, 4, false) ES_PULL(64, 4, 4, false)
    ES_PULL(4, 1, 1, false)
#undef ES_PULL
    return err == hipSuccess ? ES_OK : ES_ERR_LAUNCH;
}

}  // extern "C"

namespace {

// Transposed (sampled) graph: count the kept entries per column, scan, then
// drop every entry into its column's segment through a per-column cursor.
int build_transposed(const int32_t* rowptr, const int32_t* colidx, const float* vals, int64_t N,
                     int64_t nnz, int32_t W, int32_t mode, uint64_t seed, int32_t norm, int32_t* out_ptr,
                     int32_t* out_end, int32_t* out_idx, float* out_vals, int32_t* out_pos, void* stream)
{
    if (N < 0 || nnz < 0 || nnz > INT32_MAX) return ES_ERR_INVALID_ARG;
    if (mode != ES_FULL && mode != ES_BUCKET && mode != ES_FASTRAND) return ES_ERR_INVALID_ARG;
    if (mode != ES_FULL && W < 1) return ES_ERR_INVALID_ARG;
    if (norm < ES_NORM_NONE || norm > ES_NORM_INV_DEGREE) return ES_ERR_INVALID_ARG;
    if (!out_ptr) return ES_ERR_INVALID_ARG;
    if (N > 0 && (!rowptr || !out_end || !out_idx || !out_vals)) return ES_ERR_INVALID_ARG;
    if (nnz > 0 && !colidx) return ES_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int32_t Wk = (mode == ES_FULL) ? INT32_MAX : W;
    const int64_t nscan = N == 0 ? 1 : (N + kScanRows - 1) / kScanRows;
    if (nscan > INT32_MAX) return ES_ERR_UNSUPPORTED;
#define ES_CHECK_LAUNCH() if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH
    int64_t fb = (N + 1 + kBlockThreads - 1) / kBlockThreads;
    if (fb > 65536) fb = 65536;
    hipLaunchKernelGGL(es_fill_int_kernel, dim3((uint32_t)fb), dim3(kBlockThreads), 0, st, out_ptr, N + 1, 0);
    ES_CHECK_LAUNCH();
    if (N == 0) return ES_OK;

    const int logR = walk_logR(N, nnz, Wk);
    const int64_t rows_per_block = (int64_t)kWavesPerBlock << logR;
    const int64_t nblocks = (N + rows_per_block - 1) / rows_per_block;
    if (nblocks > INT32_MAX) return ES_ERR_UNSUPPORTED;

    hipLaunchKernelGGL(es_transpose_kernel<false>, dim3((uint32_t)nblocks), dim3(kBlockThreads), 0, st,
                       rowptr, colidx, vals, N, Wk, mode, seed, norm, logR, out_ptr, out_end, out_idx,
                       out_vals, out_pos);
    ES_CHECK_LAUNCH();
    hipLaunchKernelGGL(es_kept_scan_local_kernel, dim3((uint32_t)nscan), dim3(kBlockThreads), 0, st,
                       static_cast<const int32_t*>(nullptr), N, Wk, mode, out_ptr);
    ES_CHECK_LAUNCH();
    if (nscan > 1) {
        hipLaunchKernelGGL(es_kept_scan_blocks_kernel, dim3(1), dim3(kBlockThreads), 0, st, N, out_ptr);
        ES_CHECK_LAUNCH();
        hipLaunchKernelGGL(es_kept_scan_add_kernel, dim3((uint32_t)(nscan - 1)), dim3(kBlockThreads), 0,
                           st, N, out_ptr);
        ES_CHECK_LAUNCH();
    }
    hipLaunchKernelGGL(es_copy_int_kernel, dim3((uint32_t)fb), dim3(kBlockThreads), 0, st, out_ptr, out_end, N);
    ES_CHECK_LAUNCH();
    hipLaunchKernelGGL(es_transpose_kernel<true>, dim3((uint32_t)nblocks), dim3(kBlockThreads), 0, st,
                       rowptr, colidx, vals, N, Wk, mode, seed, norm, logR, out_ptr, out_end, out_idx,
                       out_vals, out_pos);
    ES_CHECK_LAUNCH();
#undef ES_CHECK_LAUNCH
    return ES_OK;
}

}  // namespace

extern "C" {

int es_spmm_validate_csr(const int32_t* rowptr, const int32_t* colidx, int64_t N, int64_t nnz,
                         int32_t* report, void* stream)
{
    if (N < 0 || nnz < 0 || nnz > INT32_MAX || !rowptr || !report) return ES_ERR_INVALID_ARG;
    if (nnz > 0 && !colidx) return ES_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipLaunchKernelGGL(es_fill_int_kernel, dim3(1), dim3(kBlockThreads), 0, st, report, (int64_t)4, 0);
    if (hipGetLastError() != hipSuccess) return ES_ERR_LAUNCH;
    int64_t blocks = (N + kWavesPerBlock - 1) / kWavesPerBlock;
    if (blocks < 1) blocks = 1;
    if (blocks > 16384) blocks = 16384;
    hipLaunchKernelGGL(es_validate_csr_kernel, dim3((uint32_t)blocks), dim3(kBlockThreads), 0, st, rowptr,
                       colidx, N, nnz, report);
    return hipGetLastError() == hipSuccess ? ES_OK : ES_ERR_LAUNCH;
}

int es_spmm_sample_edges(const int32_t* rowptr, int64_t N, int32_t W, int32_t mode, uint64_t seed,
                         int32_t rows_per_wave, int32_t* pos, int32_t* cnt, void* stream)
{
    if (N < 0 || W < 1) return ES_ERR_INVALID_ARG;
    if (mode != ES_BUCKET && mode != ES_FASTRAND) return ES_ERR_INVALID_ARG;
    if (rows_per_wave < -1 || rows_per_wave > 64 ||
        (rows_per_wave > 0 && (rows_per_wave & (rows_per_wave - 1))))
        return ES_ERR_INVALID_ARG;
    if (N == 0) return ES_OK;
    if (!rowptr || !pos || !cnt) return ES_ERR_INVALID_ARG;
    if (N * (int64_t)W > INT32_MAX) return ES_ERR_UNSUPPORTED;
    int logR = 0;
    while ((1 << logR) < rows_per_wave) ++logR;
    const int64_t rows_per_block = (int64_t)kWavesPerBlock << logR;
    const int64_t nblocks = (N + rows_per_block - 1) / rows_per_block;
    if (nblocks > INT32_MAX) return ES_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(es_sample_edges_kernel, dim3((uint32_t)nblocks), dim3(kBlockThreads), 0,
                       static_cast<hipStream_t>(stream), rowptr, N, W, mode, seed,
                       rows_per_wave < 0 ? -1 : logR, pos, cnt);
    return hipGetLastError() == hipSuccess ? ES_OK : ES_ERR_LAUNCH;
}

}  // extern "C"
