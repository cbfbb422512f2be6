// es_fused_kernel.h -- the fused sampling + SpMM kernel (row part, long-row part) and the small kernels that zero its atomic targets.
#ifndef ES_SPMM_FUSED_KERNEL_H
#define ES_SPMM_FUSED_KERNEL_H

#include "es_tile.h"

namespace {

// ---------------------------------------------------------------------------
// Row part of the fused kernel (Algorithm 1) for workgroup `vb` of the row
// grid.  G lanes x CH chunks x VEC floats cover one block of G*CH*VEC feature
// columns (blockIdx.y selects the block).  Rows that keep more than long_k
// entries are left to the long-row part and not stored here.
// ---------------------------------------------------------------------------
template <int G, int CH, int VEC, bool ALIGNED, bool BACKWARD, bool WIDE>
__device__ __forceinline__ void row_block(const Args& a, uint32_t vb, uint2* lds)
{
    constexpr int LOG_G = ilog2(G);
    using P = Pack<VEC, ALIGNED>;

    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x >> 6;
    const int logR = a.logR;
    const int team = kWaveSize >> logR;          // lanes per row
    const int rs = lane >> (6 - logR);           // row slot inside the wave
    const int t = lane & (team - 1);             // lane inside the team
    const int e = t >> LOG_G;                    // edge slot
    const int l = t & (G - 1);                   // column lane
    const int E = team >> LOG_G;                 // edge slots per row (>= 1)
    const int T = kTileSlots >> logR;            // tile slots per row
    uint2* tile = lds + wave * kWaveTileStride + rs * (T + E);   // E pad slots: the rows' reads of slots j .. j+E-1 miss each other's banks

    const int64_t r = ((((int64_t)vb * kWavesPerBlock) + wave) << logR) + rs;
    const bool rvalid = r < a.N;
    int32_t base = 0, n = 0;
    if (rvalid) {
        base = a.rowptr[r];
        n = a.rowptr[r + 1] - base;
    }
    const int k_row = kept_count(a.mode, n, a.W);
    const bool is_long = k_row > a.long_k;       // summed by the long-row part
    const int k = is_long ? 0 : k_row;

    LaneCols<G, CH, VEC, ALIGNED> cols;
    cols.init(blockIdx.y * (G * CH * VEC), l, a.F);

    RowSampler sampler;
    sampler.init(a.mode, a.seed, r, (uint32_t)n, (uint32_t)a.W, (uint32_t)t, (uint32_t)team);

    if (BACKWARD) {
        // transposed product: a.X is the upstream gradient, a.Y the (zeroed) output
        P dy[CH];
        if (k > 0) load_row_chunks<G, CH, VEC, ALIGNED>(a, r, n, k_row, cols, dy);
        for (int t0 = 0; t0 < k; t0 += T) {
            const int count = min(k - t0, T);
            stage_tile<ALIGNED, WIDE>(sampler, t, team, count, base, a.colidx, a.vals, a.stride_units, tile);
            wave_lds_fence();
            scatter_tile<G, CH, VEC, ALIGNED, WIDE>(tile, count, e, E, a.Y, a.ldy, cols, dy);
            wave_lds_fence();
        }
        return;
    }

    P acc[CH];
#pragma unroll
    for (int ch = 0; ch < CH; ++ch) acc[ch].zero();

    for (int t0 = 0; t0 < k; t0 += T) {
        const int count = min(k - t0, T);
        stage_tile<ALIGNED, WIDE>(sampler, t, team, count, base, a.colidx, a.vals, a.stride_units, tile);
        wave_lds_fence();
        consume_tile<G, CH, VEC, ALIGNED, WIDE>(tile, count, e, E, a.X, a.ldx, cols, acc);
        wave_lds_fence();
    }

    // ---- sum the E edge slots of each row, store ----------------------------
    for (int m = G; m < team; m <<= 1) {
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) acc[ch].add_xor(m);
    }
    if (rvalid && !is_long && e == 0) {
        float* y = a.Y + r * (int64_t)a.ldy;
        if (a.norm != ES_NORM_NONE) {
            const float f = row_factor(a.norm, n, k_row);
#pragma unroll
            for (int ch = 0; ch < CH; ++ch) acc[ch].scale(f);
        }
#pragma unroll
        for (int ch = 0; ch < CH; ++ch)
            if (cols.ok[ch]) acc[ch].store_streaming(y + cols.off[ch], cols.first[ch]);
    }
}

// ---------------------------------------------------------------------------
// Long-row part.  Workgroup (bx, by) scans rows [bx*1024, bx*1024+1024) for rows
// that keep more than long_k entries, numbers their 256-slot segments with a
// prefix sum in LDS, and its 4 waves take segments gw, gw + 4*kLongSplit, ...
// (gw = by*4 + wave).  A segment is one pass of Algorithm 1 with a whole wave on
// the row; its partial sums are added to Y (zeroed beforehand by
// es_zero_long_rows_kernel) with fp32 atomics, so the summation order across
// segments is not fixed.
// ---------------------------------------------------------------------------
struct LongScratch {
    int seg_end[kLongScanRows];                  // inclusive prefix sum of segment counts
    int wave_total[kWavesPerBlock];
};

// Sum of count(kept entries) over the long rows among the workgroup's 1024 rows;
// leaves the prefix sums in `sc`.
template <class Count>
__device__ __forceinline__ int long_scan(const Args& a, uint32_t bx, LongScratch& sc, Count&& count)
{
    constexpr int kRowsPerThread = kLongScanRows / kBlockThreads;
    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = tid >> 6;
    const int64_t row0 = (int64_t)bx * kLongScanRows;

    // thread tid owns rows row0 + tid*kRowsPerThread + i (consecutive, so the
    // prefix order is the row order)
    int nseg[kRowsPerThread];
    int mine = 0;
#pragma unroll
    for (int i = 0; i < kRowsPerThread; ++i) {
        const int64_t r = row0 + tid * kRowsPerThread + i;
        nseg[i] = 0;
        if (r < a.N) {
            const int n = a.rowptr[r + 1] - a.rowptr[r];
            const int k = kept_count(a.mode, n, a.W);
            if (k > a.long_k) nseg[i] = count(k);
        }
        mine += nseg[i];
    }
    if (__syncthreads_or(mine) == 0) return 0;   // no long row among these 1024: the common case
    int incl = mine;                             // inclusive scan inside the wave
#pragma unroll
    for (int d = 1; d < kWaveSize; d <<= 1) {
        const int up = __shfl_up(incl, d, kWaveSize);
        if (lane >= d) incl += up;
    }
    if (lane == kWaveSize - 1) sc.wave_total[wave] = incl;
    __syncthreads();
    int before = incl - mine;
    for (int w = 0; w < wave; ++w) before += sc.wave_total[w];
#pragma unroll
    for (int i = 0; i < kRowsPerThread; ++i) {
        before += nseg[i];
        sc.seg_end[tid * kRowsPerThread + i] = before;
    }
    __syncthreads();
    return sc.seg_end[kLongScanRows - 1];
}

// Number of segments of those rows.
template <int SEG>
__device__ __forceinline__ int long_segments(const Args& a, uint32_t bx, LongScratch& sc)
{
    return long_scan(a, bx, sc, [](int k) { return (k - 1) / SEG + 1; });
}

// First of the 1024 rows whose prefix exceeds `task`, in the 16-bit half HALF of
// the prefix sums or (-1) all of them.
template <int HALF>
__device__ __forceinline__ int long_row_of(const LongScratch& sc, int task)
{
    int lo = 0, hi = kLongScanRows - 1;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const int end = HALF < 0 ? sc.seg_end[mid] : (sc.seg_end[mid] >> (16 * HALF)) & 0xFFFF;
        if (end > task) hi = mid; else lo = mid + 1;
    }
    return lo;
}

// Segment number `task` of the workgroup's long rows.
struct LongSegment {
    int64_t r;
    int32_t base, n, k;                          // the row: first CSR position, stored and kept entries
    int t0, count;                               // the segment's slots
};

template <int SEG>
__device__ __forceinline__ LongSegment long_segment(const Args& a, uint32_t bx, int task, const LongScratch& sc)
{
    const int lo = long_row_of<-1>(sc, task);
    LongSegment s;
    s.r = (int64_t)bx * kLongScanRows + lo;
    s.base = a.rowptr[s.r];
    s.n = a.rowptr[s.r + 1] - s.base;
    s.k = kept_count(a.mode, s.n, a.W);
    s.t0 = (task - (lo ? sc.seg_end[lo - 1] : 0)) * SEG;
    s.count = min(s.k - s.t0, SEG);
    return s;
}

// Long rows of a small product: each is summed by one wave or, above
// alone_wave_row entries, by one workgroup whose waves take 256-slot segments in
// turn and add their partial sums through LDS, so that nothing has to be zeroed
// beforehand (a launch of its own, as long as the whole product at this size).
// What bounds a row then is the chain of memory round trips of one wave: a
// segment's entries are all requested at once, and the next segment's before the
// rows of X of this one (a row of 3999 entries, F = 16: 8.9 us without, 7.3 with).
// One wave on two segments instead leaves the other three to other rows and costs
// the row 0.6 us at F = 16, 1.6 at F = 64, 3 at F = 128, so wide rows of more than one
// segment go to the workgroup.  Many long rows in 1024: 250 of 66 entries, F = 4: 10.8
// us, split with atomics 17.4; 24 of 257, F = 128: 12.6 and 12.3.
constexpr int alone_wave_row(int G) { return G < 16 ? 2 * kLongSeg : kLongSeg; }

template <int G, int CH, int VEC, bool ALIGNED>
__device__ __forceinline__ void long_rows_alone(const Args& a, uint32_t bx, uint32_t by, uint2* lds, LongScratch& sc)
{
    constexpr int LOG_G = ilog2(G);
    constexpr int E = kWaveSize / G;
    constexpr int FB = G * CH * VEC;
    constexpr int M = kLongSeg / kWaveSize;
    using P = Pack<VEC, ALIGNED>;
    using K = RowKey<ALIGNED, false>;
    static_assert(FB * sizeof(float) <= kWaveTileStride * sizeof(uint2), "a wave's partial row fits its tile");
    // low half: rows of one wave, high half: rows of the workgroup (at most 1024 each)
    const int total = long_scan(a, bx, sc, [](int k) { return k <= alone_wave_row(G) ? 1 : 1 << 16; });
    if (total == 0) return;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x >> 6;
    const int e = lane >> LOG_G;
    const int l = lane & (G - 1);
    uint2* tile = lds + wave * kWaveTileStride;
    LaneCols<G, CH, VEC, ALIGNED> cols;
    cols.init(blockIdx.y * FB, l, a.F);

    P acc[CH];
    int n, k;
    int64_t r;
    // this wave's part of row `row` of the 1024: segments from slot t0 on, `step` slots apart
    auto sum_row = [&](int row, uint32_t t0, uint32_t step) {
        r = (int64_t)bx * kLongScanRows + row;
        const int64_t base = a.rowptr[r];
        n = a.rowptr[r + 1] - (int32_t)base;
        k = kept_count(a.mode, n, a.W);
        int32_t col[M];
        float val[M];
        auto request = [&](uint32_t at) {
            RowSampler sampler;
            sampler.init(a.mode, a.seed, r, (uint32_t)n, (uint32_t)a.W, at + lane, kWaveSize);
            uint32_t entry[M];
#pragma unroll
            for (int i = 0; i < M; ++i) entry[i] = min(sampler.next(), (uint32_t)n - 1u);   // past the row: its last
#pragma unroll
            for (int i = 0; i < M; ++i) {
                col[i] = a.colidx[base + entry[i]];
                val[i] = a.vals ? a.vals[base + entry[i]] : 1.0f;
            }
        };
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) acc[ch].zero();
        if (t0 < (uint32_t)k) request(t0);
        for (; t0 < (uint32_t)k; t0 += step) {
#pragma unroll
            for (int i = 0; i < M; ++i)
                tile[i * kWaveSize + lane] = make_uint2(K::make(col[i], a.stride_units), __float_as_uint(val[i]));
            wave_lds_fence();
            if (t0 + step < (uint32_t)k) request(t0 + step);
            consume_tile<G, CH, VEC, ALIGNED, false>(tile, min((int)((uint32_t)k - t0), kLongSeg), e, E, a.X, a.ldx, cols, acc);
            wave_lds_fence();
        }
#pragma unroll
        for (int m = G; m < kWaveSize; m <<= 1) {
#pragma unroll
            for (int ch = 0; ch < CH; ++ch) acc[ch].add_xor(m);
        }
    };
    auto store_row = [&]() {
        const float f = row_factor(a.norm, n, k);
        float* y = a.Y + r * (int64_t)a.ldy;
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) {
            acc[ch].scale(f);
            if (cols.ok[ch]) acc[ch].store(y + cols.off[ch], cols.first[ch]);
        }
    };

    for (int task = by * kWavesPerBlock + wave; task < (total & 0xFFFF); task += kLongSplit * kWavesPerBlock) {
        sum_row(long_row_of<0>(sc, task), 0, kLongSeg);
        if (e == 0) store_row();
    }
    for (int task = by; task < (total >> 16); task += kLongSplit) {
        sum_row(long_row_of<1>(sc, task), wave * kLongSeg, kWavesPerBlock * kLongSeg);
        P* part = reinterpret_cast<P*>(tile) + l;
        if (e == 0) {
#pragma unroll
            for (int ch = 0; ch < CH; ++ch) part[ch * G] = acc[ch];
        }
        __syncthreads();
        if (wave == 0 && e == 0) {
            for (int w = 1; w < kWavesPerBlock; ++w)
#pragma unroll
                for (int ch = 0; ch < CH; ++ch)
                    acc[ch].add(*(reinterpret_cast<P*>(lds + w * kWaveTileStride) + ch * G + l));
            store_row();
        }
        __syncthreads();
    }
}

template <int G, int CH, int VEC, bool ALIGNED, bool BACKWARD, bool WIDE>
__device__ __forceinline__ void long_block(const Args& a, uint32_t bx, uint32_t by, uint2* lds,
                                           LongScratch& sc)
{
    constexpr int LOG_G = ilog2(G);
    using P = Pack<VEC, ALIGNED>;

    const int total = long_segments<kLongSeg>(a, bx, sc);
    if (total == 0) return;

    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x >> 6;
    const int e = lane >> LOG_G;
    const int l = lane & (G - 1);
    constexpr int E = kWaveSize / G;
    uint2* tile = lds + wave * kWaveTileStride;
    LaneCols<G, CH, VEC, ALIGNED> cols;
    cols.init(blockIdx.y * (G * CH * VEC), l, a.F);

    const int gw = by * kWavesPerBlock + wave;
    for (int task = gw; task < total; task += kLongSplit * kWavesPerBlock) {
        const LongSegment sg = long_segment<kLongSeg>(a, bx, task, sc);
        const int64_t r = sg.r;
        const int32_t base = sg.base;
        const int n = sg.n, k = sg.k, t0 = sg.t0, count = sg.count;

        RowSampler sampler;
        sampler.init(a.mode, a.seed, r, (uint32_t)n, (uint32_t)a.W, (uint32_t)(t0 + lane), kWaveSize);
        stage_tile<ALIGNED, WIDE>(sampler, lane, kWaveSize, count, base, a.colidx, a.vals, a.stride_units, tile);
        wave_lds_fence();
        if (BACKWARD) {
            P dy[CH];
            load_row_chunks<G, CH, VEC, ALIGNED>(a, r, n, k, cols, dy);
            scatter_tile<G, CH, VEC, ALIGNED, WIDE>(tile, count, e, E, a.Y, a.ldy, cols, dy);
            wave_lds_fence();
            continue;
        }
        P acc[CH];
#pragma unroll
        for (int ch = 0; ch < CH; ++ch) acc[ch].zero();
        consume_tile<G, CH, VEC, ALIGNED, WIDE>(tile, count, e, E, a.X, a.ldx, cols, acc);
        wave_lds_fence();
#pragma unroll
        for (int m = G; m < kWaveSize; m <<= 1) {
#pragma unroll
            for (int ch = 0; ch < CH; ++ch) acc[ch].add_xor(m);
        }
        if (e == 0) {
            float* y = a.Y + r * (int64_t)a.ldy;
            if (a.norm != ES_NORM_NONE) {
                const float f = row_factor(a.norm, n, k);
#pragma unroll
                for (int ch = 0; ch < CH; ++ch) acc[ch].scale(f);
            }
#pragma unroll
            for (int ch = 0; ch < CH; ++ch)
                if (cols.ok[ch]) acc[ch].atomic_add(y + cols.off[ch], cols.first[ch]);
        }
    }
}

// ---------------------------------------------------------------------------
// The fused kernel.  The first a.long_blocks workgroups (dispatched first, so
// the splitting of long rows overlaps the bulk of the rows) run the long-row
// part; the rest run the row part, remapped so that each XCD (hardware deals
// workgroup b to XCD b % 8; long_blocks is a multiple of 8) walks one
// contiguous range of rows, or with blocks_per_xcd == 0 not remapped: the rows of a
// transposed Bucket sample get shorter from the first to the last, and as
// contiguous ranges the first XCD would have most of the work (transposed product, 233 k
// rows, W = 64 of a mean of 490, F = 64: 1.70 ms as ranges, 0.90 dealt round).
// ---------------------------------------------------------------------------
// Six waves per SIMD: the two registers more that the compiler takes otherwise cost a
// sixth of the waves.  Ids that cluster, at five / at six: 170 k rows, Bucket W = 16, mean 14, F = 128: 59.2
// us / 53.8, mean 40, F = 64: 57.2 / 51.2.  Uniform ids wait for L2 misses and are within 3 % either way (170 k of mean
// 14, F = 128: 89.9 / 92.4, 40 k of mean 40, F = 128, exact: 95.1 / 95.3).  Four chunks per lane need 88 to 96
// registers, which would spill at six.
template <int G, int CH, int VEC, bool ALIGNED, bool BACKWARD, bool WIDE>
__global__ void __launch_bounds__(kBlockThreads, CH == 4 ? 5 : 6) es_spmm_kernel(const Args a)
{
    __shared__ uint2 lds[kWavesPerBlock * kWaveTileStride];
    __shared__ LongScratch long_scratch;

    if (blockIdx.x < a.long_blocks) {
        long_block<G, CH, VEC, ALIGNED, BACKWARD, WIDE>(a, blockIdx.x / kLongSplit, long_share(blockIdx.x),
                                                  lds, long_scratch);
        return;
    }
    const uint32_t b = blockIdx.x - a.long_blocks;
    const uint32_t vb = a.blocks_per_xcd ? (b % kNumXcd) * a.blocks_per_xcd + b / kNumXcd : b;
    if (vb >= a.nblocks) return;
    row_block<G, CH, VEC, ALIGNED, BACKWARD, WIDE>(a, vb, lds);
}

// The same for a small product: a long row is one workgroup's.  A kernel of its
// own, so that the general one keeps its registers.
template <int G, int CH, int VEC, bool ALIGNED>
__global__ void __launch_bounds__(kBlockThreads) es_spmm_small_kernel(const Args a)
{
    __shared__ __align__(16) uint2 lds[kWavesPerBlock * kWaveTileStride];   // also holds partial rows, as Packs
    __shared__ LongScratch long_scratch;
    if (blockIdx.x < a.long_blocks) {
        long_rows_alone<G, CH, VEC, ALIGNED>(a, blockIdx.x / kLongSplit, long_share(blockIdx.x), lds, long_scratch);
        return;
    }
    const uint32_t b = blockIdx.x - a.long_blocks;
    const uint32_t vb = (b % kNumXcd) * a.blocks_per_xcd + b / kNumXcd;
    if (vb >= a.nblocks) return;
    row_block<G, CH, VEC, ALIGNED, false, false>(a, vb, lds);
}

// Zero-fills an [N x F] matrix with row stride ld (the transposed product
// accumulates into its output with atomics).
__global__ void __launch_bounds__(kBlockThreads)
es_fill_zero_kernel(float* __restrict__ out, int64_t N, int32_t F, int32_t ld)
{
    const int64_t total = N * (int64_t)F;
    for (int64_t i = (int64_t)blockIdx.x * kBlockThreads + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * kBlockThreads) {
        const int64_t r = i / F;
        out[r * ld + (i - r * F)] = 0.0f;
    }
}

// Zeroes Y for the rows the long-row part will accumulate into with atomics.
// Each lane tests one row; the wave then clears the flagged rows together, 64
// consecutive floats per store instruction.
__global__ void __launch_bounds__(kBlockThreads) es_zero_long_rows_kernel(const Args a)
{
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int64_t r = (int64_t)blockIdx.x * kBlockThreads + threadIdx.x;
    bool is_long = false;
    if (r < a.N) {
        const int n = a.rowptr[r + 1] - a.rowptr[r];
        is_long = kept_count(a.mode, n, a.W) > a.long_k;
    }
    unsigned long long flagged = __ballot(is_long);
    const int64_t wave_row0 = r - lane;
    while (flagged) {
        const int src = __ffsll((long long)flagged) - 1;
        flagged &= flagged - 1;
        float* y = a.Y + (wave_row0 + src) * (int64_t)a.ldy;
        for (int c = lane; c < a.F; c += kWaveSize) y[c] = 0.0f;
    }
}

}  // namespace

#endif  // ES_SPMM_FUSED_KERNEL_H
