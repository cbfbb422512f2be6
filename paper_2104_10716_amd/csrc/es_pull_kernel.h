// es_pull_kernel.h -- the transposed sampled product as a gather over the transposed graph (no atomics).
#ifndef ES_SPMM_PULL_KERNEL_H
#define ES_SPMM_PULL_KERNEL_H

#include <type_traits>

#include "es_tile.h"

namespace {

// ---------------------------------------------------------------------------
// dX = sample_W(A)^T dY without scattering: row c of the output sums, over the
// STORED entries (r, c) of A, the ones the sampler keeps for row r.  The
// transposed graph (built once per graph by es_spmm_transpose_graph) lists for
// every column c its entries as (row r, entry number idx inside row r, value).
// Whether the forward pass keeps entry idx of a row of n entries follows from
// inverting the sampling rule (Section 4.4):
//     full, or n <= W       kept
//     Bucket                kept iff idx < W
//     FastRand, n > W       slot i reads entry (off + i*P) mod n, so entry idx is
//                           read by slot i = ((idx - off) * P^-1) mod n
//                                          = (slot0 - shift) mod n,
//                           slot0 = idx * P^-1 mod n   (per entry, stored: it does
//                                                       not depend on W or the seed)
//                           shift = off * P^-1 mod n   (per row, recomputed per call
//                                                       from the seed: es_pull_rows_kernel)
//                           kept iff i < W.
// So one structure serves every W, mode and seed (a new seed per training
// iteration costs one pass over the rows), the per-entry test is a subtract and
// two compares, and the result is bit-reproducible.
// ---------------------------------------------------------------------------

// (a * b) mod n for a, b < n < 2^31: quotient estimated in double (off by at
// most one), remainder fixed up in integers.
__device__ __forceinline__ uint32_t mulmod31(uint32_t a, uint32_t b, uint32_t n)
{
    const uint64_t prod = (uint64_t)a * b;
    const uint64_t q = (uint64_t)((double)a * (double)b / (double)n);
    int64_t rem = (int64_t)(prod - q * n);
    if (rem < 0) rem += n;
    if (rem < 0) rem += n;
    if (rem >= (int64_t)n) rem -= n;
    if (rem >= (int64_t)n) rem -= n;
    return (uint32_t)rem;
}

// Inverse of the row's FastRand multiplier modulo its length (extended Euclid;
// the multiplier is coprime to n by construction).  One thread per row.
__global__ void __launch_bounds__(kBlockThreads)
es_pinv_kernel(const int32_t* __restrict__ rowptr, int64_t N, int32_t* __restrict__ pinv)
{
    const int64_t r = (int64_t)blockIdx.x * kBlockThreads + threadIdx.x;
    if (r >= N) return;
    const int64_t n = (int64_t)rowptr[r + 1] - rowptr[r];
    int64_t inv = 0;
    if (n > 1) {
        int64_t a = fastrand_multiplier((uint32_t)n) % n, b = n, x0 = 1, x1 = 0;   // a*x0 = a (mod n), a*x1 = b
        while (b != 0) {
            const int64_t q = a / b;
            int64_t t = a - q * b; a = b; b = t;
            t = x0 - q * x1; x0 = x1; x1 = t;
        }
        inv = x0 % n;                                   // a == gcd == 1 here
        if (inv < 0) inv += n;
    }
    pinv[r] = (int32_t)inv;
}

// After the transposed fill: turn every entry's CSR position into its entry
// number inside its row (in place) and store the slot that reads it under
// Equation 2 without rotation.
__global__ void __launch_bounds__(kBlockThreads)
es_pull_entries_kernel(const int32_t* __restrict__ rowptr, const int32_t* __restrict__ pinv,
                       const int32_t* __restrict__ t_row, int64_t nnz, int32_t* __restrict__ t_idx,
                       int32_t* __restrict__ t_slot)
{
    for (int64_t j = (int64_t)blockIdx.x * kBlockThreads + threadIdx.x; j < nnz;
         j += (int64_t)gridDim.x * kBlockThreads) {
        const int32_t r = t_row[j];
        const int32_t base = rowptr[r];
        const uint32_t n = (uint32_t)(rowptr[r + 1] - base);
        const uint32_t idx = (uint32_t)(t_idx[j] - base);
        t_idx[j] = (int32_t)idx;
        t_slot[j] = n > 1 ? (int32_t)mulmod31(idx, (uint32_t)pinv[r], n) : 0;
    }
}

// Per call: rows[r] = (n, shift) with shift = off * P^-1 mod n for this seed.
__global__ void __launch_bounds__(kBlockThreads)
es_pull_rows_kernel(const int32_t* __restrict__ rowptr, const int32_t* __restrict__ pinv, int64_t N,
                    int32_t mode, uint64_t seed, int32_t W, int2* __restrict__ rows)
{
    const int64_t r = (int64_t)blockIdx.x * kBlockThreads + threadIdx.x;
    if (r >= N) return;
    const uint32_t n = (uint32_t)(rowptr[r + 1] - rowptr[r]);
    uint32_t shift = 0;
    if (mode == ES_FASTRAND && n > (uint32_t)W && seed != 0)
        shift = mulmod31(fastrand_offset(seed, r, n), (uint32_t)pinv[r], n);
    rows[r] = make_int2((int)n, (int)shift);
}

// A row's length and rotation are only needed for a rotated FastRand (seed != 0)
// and for the row factor: without rotation the stored slot (or entry number) is
// below n, so "n <= W or slot < W" is just "slot < W".
__host__ __device__ __forceinline__ bool pull_needs_rows(int32_t mode, uint64_t seed, int32_t norm)
{
    return (mode == ES_FASTRAND && seed != 0) || norm != ES_NORM_NONE;
}

constexpr int kPullChunks = 4;                        // chunks of 64 entries requested together

// One wave per output row c, E = 64 / G edge slots.  Stage 1 reads the row's
// transposed entries 64 at a time, tests them, and packs the kept ones
// (row of dY as its key, value times the forward row factor) into the LDS tile;
// stage 2 is the forward kernel's gather.
// MAXC: chunks of 64 entries requested together at most.  Long columns (8) stream: a pass loads all of its chunks without a
// branch, an absent entry as the column's first.  Short ones (4) wait for one round trip after another: six waves per SIMD
// (five with 64-bit keys, five to three where a lane holds several chunks of columns, below which the form spills, and a spill costs 1.1 to 1.6
// times the time), one chunk where that holds the column, and only entries that are there are loaded.  The latter on long columns:
// 50 k rows of mean 300, F = 32, Bucket W = 8: 33.7 us, 44.3 with it.
// The two are written out, for one body with both needs 80 to 128 registers where the streaming form of 64 lanes has 72.
// Time over that of always 8, mean of less than 96 entries, 60 graphs of 3 k to 1 M rows: 4 to 16 lanes (F up to 64), the column's number in a
// scalar register, 0.57 - 1.03 (in a vector register, with six waves where this has seven, 0.59 - 1.07: 235 k rows of mean 82, F = 20, W = 22
// 149 / 159 us); 20 k rows of mean 4.5, F = 32: 17.5 / 11.8 us, 170 k of mean 14, F = 128: 133 / 110, 1 M of mean 50, ids that cluster, Bucket W = 32,
// F = 64: 999 / 727.  32 lanes, the number in a vector register: 0.76 - 1.05, uniform ids of mean 20 and more 0.93 - 1.05 (in a scalar one, with seven waves,
// up to 2 % more of them).  64 lanes:
//  * not aligned, one chunk of columns per lane, the number in a scalar register (76 vector registers; 98 without, 0.79 - 1.07): 0.76 - 1.02
//  * aligned, one chunk: rows looked up for the kept entries alone, or a mean of at most 12: ids that cluster 0.79 - 0.99, uniform ones 0.79 -
//    1.06 (F = 200 to 256, mean 8 to 30); else 0.93 - 1.04: those stream
//  * more chunks, aligned: mean of at most 12, 0.83 - 1.00, else 0.95 - 1.06: those stream; not aligned, four 0.95 - 1.01, two rotated 0.93 - 1.01, not
//    rotated 0.93 - 1.09: those stream
template <int G, int CH, bool ALIGNED>
__host__ __device__ constexpr bool pull_short_form(bool rotated, bool rows, bool few)
{
    return G < 64 || (ALIGNED ? few || (CH == 1 && rows) : CH != 2 || rotated);
}

template <int G, int CH, int VEC, bool ALIGNED, bool WIDE, int MAXC>
__global__ void __launch_bounds__(kBlockThreads, MAXC == 8 ? 0 : G < 64 ? 6 - WIDE : (CH == 1 ? 6 : CH == 2 ? 5 : 4) - (CH > 1 && !ALIGNED))
es_pull_kernel(const Args a, const int32_t* __restrict__ t_ptr, const int32_t* __restrict__ t_row,
               const int32_t* __restrict__ t_idx, const int32_t* __restrict__ t_slot,
               const float* __restrict__ t_vals, const int2* __restrict__ rows)
{
    __shared__ uint2 lds[kWavesPerBlock * kWaveTileStride];
    constexpr int LOG_G = ilog2(G);
    constexpr int E = kWaveSize / G;
    constexpr int T = kTileSlots;
    using P = Pack<VEC, ALIGNED>;
    using K = RowKey<ALIGNED, WIDE>;

    // consecutive output rows go to different XCDs: under Bucket the kept entries
    // crowd into the lowest-numbered columns, and those rows are the whole work
    const uint32_t vb = blockIdx.x;
    if (vb >= a.nblocks) return;
    const int lane = threadIdx.x & (kWaveSize - 1);
    int wave = threadIdx.x >> 6;
    if constexpr (MAXC != 8 && (G <= 16 || (G == 64 && CH == 1 && !ALIGNED))) wave = __builtin_amdgcn_readfirstlane(wave);
    const int e = lane >> LOG_G;
    const int l = lane & (G - 1);
    uint2* tile = lds + wave * kWaveTileStride;
    const unsigned long long below_me = (1ull << lane) - 1ull;

    const int64_t c = (int64_t)vb * kWavesPerBlock + wave;
    if (c >= a.N) return;
    const int32_t begin = t_ptr[c];
    const int32_t count = t_ptr[c + 1] - begin;

    LaneCols<G, CH, VEC, ALIGNED> cols;
    cols.init(blockIdx.y * (G * CH * VEC), l, a.F);
    P acc[CH];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) acc[ch].zero();

    if constexpr (MAXC == 8) {
        // MAXC * 64 entries per pass: all their loads are issued before the
        // first test, so that one pass costs two memory round trips, not sixteen
        const bool need_rows = (a.mode == ES_FASTRAND && a.seed != 0) || a.norm != ES_NORM_NONE;
        int fill = 0;
        for (int j0 = 0; j0 < count; j0 += MAXC * kWaveSize) {
            int32_t r[MAXC], pick[MAXC];
            float v[MAXC];
            bool valid[MAXC];
#pragma unroll
            for (int q = 0; q < MAXC; ++q) {
                const int jj = j0 + q * kWaveSize + lane;
                valid[q] = jj < count;
                const int64_t j = (int64_t)begin + (valid[q] ? jj : 0);
                r[q] = t_row[j];
                v[q] = t_vals[j];
                pick[q] = a.mode == ES_BUCKET ? t_idx[j] : a.mode == ES_FASTRAND ? t_slot[j] : 0;
            }
            int2 info[MAXC];
#pragma unroll
            for (int q = 0; q < MAXC; ++q) info[q] = need_rows ? rows[r[q]] : make_int2(INT32_MAX, 0);
#pragma unroll
            for (int q = 0; q < MAXC; ++q) {
                const uint32_t n = (uint32_t)info[q].x;
                int32_t slot = pick[q];                      // Bucket: entry number; FastRand: slot after rotation
                if (a.mode == ES_FASTRAND) {
                    slot -= info[q].y;
                    if (slot < 0) slot += (int32_t)n;
                }
                const bool keep = valid[q] && (n <= (uint32_t)a.W || (uint32_t)slot < (uint32_t)a.W);
                const unsigned long long m = __ballot(keep);
                if (keep) {
                    const int k = kept_count(a.mode, (int)n, a.W);
                    const float w = v[q] * row_factor(a.norm, (int)n, k);
                    tile[fill + __popcll(m & below_me)] = make_uint2(K::make(r[q], a.stride_units), __float_as_uint(w));
                }
                fill += __popcll(m);
            }
            if (fill > T - MAXC * kWaveSize) {        // the next pass might not fit: gather what is staged
                wave_lds_fence();
                consume_tile<G, CH, VEC, ALIGNED, WIDE>(tile, fill, e, E, a.X, a.ldx, cols, acc);
                wave_lds_fence();
                fill = 0;
            }
        }
        wave_lds_fence();
        consume_tile<G, CH, VEC, ALIGNED, WIDE>(tile, fill, e, E, a.X, a.ldx, cols, acc);
    } else {
        // as pull_needs_rows; written out, since through the function the kernel takes up to
        // 4 registers more (56 k rows of mean 6, F = 71: 52.2 us, 51.1 this way)
        const bool rotated = a.mode == ES_FASTRAND && a.seed != 0;
        const bool need_rows = rotated || a.norm != ES_NORM_NONE;
        int fill = 0;
        auto gather = [&]() {
            wave_lds_fence();
            consume_tile<G, CH, VEC, ALIGNED, WIDE>(tile, fill, e, E, a.X, a.ldx, cols, acc);
            wave_lds_fence();
            fill = 0;
        };
        // chunks * 64 entries from j0 on: all their loads are issued before the first test, so
        // that they cost two memory round trips
        auto pass = [&](int j0, auto chunks) {
            constexpr int C = decltype(chunks)::value;
            int32_t r[C], pick[C];
            float v[C];
            bool valid[C];
#pragma unroll
            for (int q = 0; q < C; ++q) {
                const int jj = j0 + q * kWaveSize + lane;
                valid[q] = jj < count;
                if (valid[q]) {
                    const int64_t j = (int64_t)begin + jj;
                    r[q] = t_row[j];
                    v[q] = t_vals[j];
                    pick[q] = a.mode == ES_BUCKET ? t_idx[j] : a.mode == ES_FASTRAND ? t_slot[j] : 0;
                }
            }
            int2 info[C];
#pragma unroll
            for (int q = 0; q < C; ++q) {
                // without rotation the pick is below n, so it decides alone, and only kept entries need their row
                if (!rotated) valid[q] = valid[q] && (uint32_t)pick[q] < (uint32_t)a.W;
                if (need_rows && valid[q]) info[q] = rows[r[q]];
                else info[q] = make_int2(INT32_MAX, 0);
            }
#pragma unroll
            for (int q = 0; q < C; ++q) {
                const uint32_t n = (uint32_t)info[q].x;
                bool keep = valid[q];
                if (rotated) {
                    int32_t slot = pick[q] - info[q].y;          // slot after rotation
                    if (slot < 0) slot += (int32_t)n;
                    keep = keep && (n <= (uint32_t)a.W || (uint32_t)slot < (uint32_t)a.W);
                }
                const unsigned long long m = __ballot(keep);
                if (keep) {
                    const int k = kept_count(a.mode, (int)n, a.W);
                    const float w = v[q] * row_factor(a.norm, (int)n, k);
                    tile[fill + __popcll(m & below_me)] = make_uint2(K::make(r[q], a.stride_units), __float_as_uint(w));
                }
                fill += __popcll(m);
            }
        };
        // one chunk where that holds the rest of the column: an absent one costs its instructions and branches
        for (int j0 = 0; j0 < count;) {
            const int chunks = count - j0 > kWaveSize ? MAXC : 1;
            if (fill > T - chunks * kWaveSize) gather();
            if (chunks == 1) pass(j0, std::integral_constant<int, 1>{});
            else pass(j0, std::integral_constant<int, MAXC>{});
            j0 += chunks * kWaveSize;
        }
        wave_lds_fence();
        consume_tile<G, CH, VEC, ALIGNED, WIDE>(tile, fill, e, E, a.X, a.ldx, cols, acc);
    }

#pragma unroll
    for (int m = G; m < kWaveSize; m <<= 1) {
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) acc[ch].add_xor(m);
    }
    if (e == 0) {
        float* y = a.Y + c * (int64_t)a.ldy;
#pragma unroll
        for (int ch = 0; ch < CH; ++ch)
            if (cols.ok[ch]) acc[ch].store(y + cols.off[ch], cols.first[ch]);
    }
}

// ---------------------------------------------------------------------------
// The same for a rotated FastRand (seed != 0), whose test needs the row's length and
// rotation.  Looking those up for every stored entry costs a line of the vector cache per lane
// (113 M random reads of 8 bytes from 1.9 MB: 0.43 ms, whatever the loads' cache policy), and most
// entries are dropped by it.  So a persistent workgroup of 16 waves first fills its LDS with four bits of every row's
// rotation, shift / 2^b mod 16, and an entry is looked up only if its slot can lie in the row's window:
// slot / 2^b within two steps behind those bits (2^b >= W / 2, so a window touches at most three steps),
// or slot < W (a window that wraps).  Of 233 k rows of mean 490 22 % of the entries pass at W = 16, 26, 35 and 46 % at 32, 64 and 128.
// The waves deal the columns round; a pass's gathers are under way together with the next one's lookups and the
// entries after that.  233 k rows of mean 490, F = 64, es_pull_kernel / this: W = 16 911 / 549 us, W = 64 1090 / 968: what
// is left is the stream of entries (1.36 GB) and the gathers, at 16 waves per compute unit.
// ---------------------------------------------------------------------------
constexpr int kPullWaves = 16;
constexpr int kPullThreads = kPullWaves * kWaveSize;
constexpr int kPullTile = 64 + kPullChunks * kWaveSize;   // (row, value) slots per wave
constexpr int kPullLdsBytes = 160 * 1024;
constexpr int kPullTileBytes = kPullWaves * kPullTile * (int)sizeof(uint2);
constexpr int64_t kPullFilterRows = (int64_t)(kPullLdsBytes - kPullTileBytes) * 2;   // rows whose bits fit beside the tiles

// log2 of the step: the smallest that is at least W / 2
__host__ __device__ constexpr int pull_step(uint32_t W)
{
    int b = 0;
    while (b < 30 && (2ull << b) < W) ++b;
    return b;
}

// Whether slot i of a row can be kept, from the row's bits.
__host__ __device__ __forceinline__ bool pull_may_keep(uint32_t slot, uint32_t code, uint32_t W, int b)
{
    return (((slot >> b) - code) & 15u) <= 2u || slot < W;
}

template <int G, int CH, int VEC, bool ALIGNED>
__global__ void __launch_bounds__(kPullThreads)
es_pull_filtered_kernel(const Args a, const int32_t* __restrict__ t_ptr, const int32_t* __restrict__ t_row,
                        const int32_t* __restrict__ t_slot, const float* __restrict__ t_vals,
                        const int2* __restrict__ rows)
{
    extern __shared__ __align__(16) uint32_t pull_lds[];
    constexpr int LOG_G = ilog2(G);
    constexpr int E = kWaveSize / G;
    using P = Pack<VEC, ALIGNED>;
    using K = RowKey<ALIGNED, false>;
    uint2* tile = reinterpret_cast<uint2*>(pull_lds) + (threadIdx.x >> 6) * kPullTile;
    uint32_t* codes = pull_lds + kPullTileBytes / (int)sizeof(uint32_t);
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int e = lane >> LOG_G;
    const int l = lane & (G - 1);
    const unsigned long long below_me = (1ull << lane) - 1ull;
    const uint32_t W = (uint32_t)a.W;
    const int b = pull_step(W);
    const int N = (int)a.N;                           // below kPullFilterRows

    for (int w = threadIdx.x; w * 8 < N; w += kPullThreads) {
        uint32_t word = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i)
            word |= (((uint32_t)rows[min(w * 8 + i, N - 1)].y >> b) & 15u) << (4 * i);
        codes[w] = word;
    }
    __syncthreads();

    LaneCols<G, CH, VEC, ALIGNED> cols;
    cols.init(blockIdx.y * (G * CH * VEC), l, a.F);
    P acc[CH];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) acc[ch].zero();

    // entries [at, at + left) of column c are still to be read
    struct Pass { int c; int32_t at, left; };
    struct Entries { int32_t row[kPullChunks], slot[kPullChunks]; float val[kPullChunks]; };
    const int stride = (int)gridDim.x * kPullWaves;
    const int c0 = wave * (int)gridDim.x + (int)blockIdx.x;      // neighbouring columns go to different workgroups
    int32_t ends = 0, begins = 0;                     // lane i: the column i strides behind `held`
    int held = c0 - kWaveSize * stride;
    auto column = [&](int c) {
        if (c >= N) return Pass{c, 0, 0};
        int i = (c - held) / stride;
        if (i >= kWaveSize) {
            held = c;
            i = 0;
            const int64_t mine = (int64_t)c + (int64_t)lane * stride;
            begins = mine < N ? t_ptr[mine] : 0;
            ends = mine < N ? t_ptr[mine + 1] : 0;
        }
        const int32_t from = __builtin_amdgcn_readlane(begins, i);
        return Pass{c, from, __builtin_amdgcn_readlane(ends, i) - from};
    };
    auto next = [&](const Pass& p) {
        if (p.left > kPullChunks * kWaveSize) return Pass{p.c, p.at + kPullChunks * kWaveSize, p.left - kPullChunks * kWaveSize};
        return column(p.c + stride);
    };
    auto request = [&](const Pass& p, Entries& n) {
#pragma unroll
        for (int q = 0; q < kPullChunks; ++q) {
            if (q * kWaveSize + lane < p.left) {
                const int64_t j = (int64_t)p.at + q * kWaveSize + lane;
                n.row[q] = t_row[j];
                n.slot[q] = t_slot[j];
                n.val[q] = t_vals[j];
            }
        }
    };

    // entries of the pass at hand that can be kept, and their rows' (length, rotation), on their way
    bool may[kPullChunks];
    int2 info[kPullChunks];
    auto look_up = [&](const Pass& p, const Entries& n) {
#pragma unroll
        for (int q = 0; q < kPullChunks; ++q) {
            may[q] = q * kWaveSize + lane < p.left;
            if (may[q]) {
                const uint32_t r = (uint32_t)n.row[q];
                may[q] = pull_may_keep((uint32_t)n.slot[q], codes[r >> 3] >> ((r & 7u) * 4u), W, b);
                if (may[q]) info[q] = rows[r];
            }
        }
    };

    int fill = 0;
    Pass now = column(c0);
    if (now.c >= N) return;
    Pass then = next(now);
    // One pass: its kept entries go to the tile; the next pass is looked up, the one after that
    // requested, and only then are the rows of dY gathered, so that all three are under way together.
    auto step = [&](Entries& cur, Entries& ahead) {
#pragma unroll
        for (int q = 0; q < kPullChunks; ++q) {
            bool keep = may[q];
            uint32_t n = 0;
            if (keep) {
                n = (uint32_t)info[q].x;
                int32_t slot = cur.slot[q] - info[q].y;
                if (slot < 0) slot += (int32_t)n;
                keep = n <= W || (uint32_t)slot < W;
            }
            const unsigned long long m = __ballot(keep);
            if (keep) {
                const float w = cur.val[q] * row_factor(a.norm, (int)n, kept_count(ES_FASTRAND, (int)n, a.W));
                tile[fill + __popcll(m & below_me)] = make_uint2(K::make(cur.row[q], a.stride_units), __float_as_uint(w));
            }
            fill += __popcll(m);
        }
        const Pass p = now;
        now = then;
        if (now.c < N) {
            look_up(now, ahead);
            then = next(now);
            if (then.c < N) request(then, cur);
        }
        const bool last = now.c != p.c;
        if (last || fill > kPullTile - kPullChunks * kWaveSize) {
            wave_lds_fence();
            consume_tile<G, CH, VEC, ALIGNED, false>(tile, fill, e, E, a.X, a.ldx, cols, acc);
            wave_lds_fence();
            fill = 0;
        }
        if (last) {
#pragma unroll
            for (int m = G; m < kWaveSize; m <<= 1) {
#pragma unroll
                for (int ch = 0; ch < CH; ++ch) acc[ch].add_xor(m);
            }
            if (e == 0) {
                float* y = a.Y + p.c * (int64_t)a.ldy;
#pragma unroll
                for (int ch = 0; ch < CH; ++ch)
                    if (cols.ok[ch]) acc[ch].store(y + cols.off[ch], cols.first[ch]);
            }
#pragma unroll
            for (int ch = 0; ch < CH; ++ch) acc[ch].zero();
        }
        return now.c < N;
    };
    Entries even, odd;
    request(now, even);
    if (then.c < N) request(then, odd);
    look_up(now, even);
    while (step(even, odd) && step(odd, even)) {}
}

}  // namespace

#endif  // ES_SPMM_PULL_KERNEL_H
