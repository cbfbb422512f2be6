// es_bin_kernel.h -- the transposed sampled product with a workspace: kept entries sorted by column with counters in LDS.
#ifndef ES_SPMM_BIN_KERNEL_H
#define ES_SPMM_BIN_KERNEL_H

#include "es_flat_kernel.h"

namespace {

// ---------------------------------------------------------------------------
// dX = sample_W(A)^T dY with a workspace.  Scattering f * v * dY[r] to dX[c] with
// global atomics is bound by the atomic path (20.5 G requests of 64 bytes a second
// whatever the launch, a tenth of what gathers reach).  Here the sampled graph is
// transposed first and the exact forward product run on the result.  The transposition is a counting sort in two
// levels, so that no counter lies in global memory: the kept entries by blocks of
// 2^log_width columns (count per workgroup and block, prefix sums, fill: records of
// 8 bytes, the row and the column inside the block, value times row factor), then each
// block by column.  Where a walker's entries fit its registers one launch does the first level (es_bin_local_kernel).
//
// What bounds it: the product, i.e. its gathers.  170 k rows, W = 16 of a mean of 14, F =
// 128: 110 us (scatter: 406), of which the product 83.  Larger
// and denser (233 k rows, W = 64, 14.9 M entries, F = 64; Bucket / FastRand): count 67 / 82, fill 124 / 244, sort
// 218 / 209, product 477 / 512 of 900 / 1050.  Beyond every cache (2.45 M rows, W = 64, 56 M entries, F = 128): 254, 417,
// 1285 and 3373 of 5.4 ms (scatter: 21.8).  The fill's records go out 8 bytes at a time (256 walkers: 133 us; 512, with
// half as many records side by side: 259).
// Tried and slower: sums kept in LDS per column block and added to with ds_add_f32,
// which takes three clocks per lane (170 k rows: 650 us for that pass alone).
// ---------------------------------------------------------------------------
constexpr int kBinThreads = 512;                      // of a counting / filling workgroup: one row per thread at a time
constexpr int kBinWaves = kBinThreads / kWaveSize;
constexpr int kBinRowBits = 22;                       // a record holds the row in 22 bits, the column of the block in 10
constexpr int kBinMaxBlocks = 4096;                   // column blocks at most: 16 KB of counters per workgroup
static_assert(kBinMaxBlocks == (1 << kBinRowBits) >> (32 - kBinRowBits), "the most rows, in blocks of the most columns");
constexpr int kBinMaxW = 4096;                        // kept entries of a row at most: one workgroup walks them
constexpr int kBinWalkers = 256;                      // counting / filling workgroups at most

struct BinArgs {
    const int32_t* rowptr;
    const int32_t* colidx;
    const float* vals;
    uint2* records;            // [capacity]; one launch for the first level: a piece for each walker's own
    int32_t* counts;           // [walkers x nbins]: records of walker i in block b, then of all walkers before it;
                               // one launch: [walkers x (nbins + 1)]: walker i's records of all blocks before b
    int32_t* base;             // [nbins + 1]: first record of block b; one launch: [walkers]: first record of walker i
    int32_t* t_ptr;            // [N + 1], t_row and t_val [capacity]: the transposed sampled graph
    int32_t* t_row;
    float* t_val;
    int64_t N, capacity;
    uint64_t seed;
    int32_t W, mode, norm;
    int32_t log_width, nbins, walkers;
};

// Inclusive prefix sums over the workgroup's threads; `total` becomes their sum.  Ends with a barrier.
template <int THREADS>
__device__ __forceinline__ int32_t block_scan(int32_t v, int32_t* wave_total, int32_t& total)
{
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int d = 1; d < kWaveSize; d <<= 1) {
        const int32_t up = __shfl_up(v, d, kWaveSize);
        if (lane >= d) v += up;
    }
    if (lane == kWaveSize - 1) wave_total[wave] = v;
    __syncthreads();
    int32_t before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < THREADS / kWaveSize; ++w) {
        if (w < wave) before += wave_total[w];
        total += wave_total[w];
    }
    __syncthreads();
    return v + before;
}

// The first level in one launch, where a walker's kept entries fit its threads' registers (at most
// kBinLocalRows rows, kBinLocalPer entries per thread): an entry's rank in its column block comes
// from the counter's atomic, the counters' prefix sums give its place among the walker's own records, and the walker leaves
// those sums in counts[walker][0 .. nbins].  No launch for counting or prefix sums over walkers is needed: the sort
// adds up what it needs of the walkers' sums.  Whole product, count / scan / base / fill / sort / gather in place of this / sort /
// gather: 170 k rows, W = 16 of a mean of 14, F = 128: 121 / 110 us, 60 k rows, W = 60, F = 32: 94 / 82, 10 k rows, W = 250 of a
// mean of 300, F = 64: 83 / 65.
constexpr int kBinLocalRows = 1024;
constexpr int kBinLocalPer = 16;
__global__ void __launch_bounds__(kBinLocalRows) es_bin_local_kernel(const BinArgs a)
{
    extern __shared__ int32_t counter[];              // [nbins + 1]
    __shared__ int32_t first[kBinLocalRows];
    __shared__ int32_t src[kBinLocalRows];
    __shared__ uint32_t len[kBinLocalRows], mul[kBinLocalRows], rot[kBinLocalRows];
    __shared__ float factor[kBinLocalRows];
    __shared__ int32_t wave_total[kBinLocalRows / kWaveSize];
    const int tid = threadIdx.x;
    for (int b = tid; b <= a.nbins; b += kBinLocalRows) counter[b] = 0;
    const int64_t r_begin = a.N * blockIdx.x / a.walkers, r_end = a.N * (blockIdx.x + 1) / a.walkers;
    const int64_t r = r_begin + tid;
    int32_t k = 0;
    if (r < r_end) {
        const int32_t p = a.rowptr[r];
        const int32_t n = a.rowptr[r + 1] - p;
        k = kept_count(a.mode, n, a.W);
        src[tid] = p;
        const bool strided = a.mode == ES_FASTRAND && n > a.W;
        len[tid] = strided ? (uint32_t)n : 0u;
        mul[tid] = strided ? fastrand_multiplier((uint32_t)n) : 0u;
        rot[tid] = strided ? fastrand_offset(a.seed, r, (uint32_t)n) : 0u;
        factor[tid] = row_factor(a.norm, n, k);
    }
    int32_t total;
    first[tid] = block_scan<kBinLocalRows>(k, wave_total, total) - k;
    __syncthreads();
    // The walker's own records begin where those of the rows before it can end at most, rowptr[r] or W for each of
    // them, and end where the next walker's begin.  (An nnz below rowptr[N] cuts entries off.)
    const int32_t own = (int32_t)max((int64_t)0, min(min((int64_t)src[0], r_begin * a.W), a.capacity));
    total = (int32_t)min((int64_t)total, a.capacity - own);
    // this thread's entries: row and column inside the block, value; block | rank << 12
    uint32_t key[kBinLocalPer], place[kBinLocalPer];
    float val[kBinLocalPer];
#pragma unroll
    for (int m = 0; m < kBinLocalPer; ++m) {
        const int32_t i = tid + m * kBinLocalRows;
        if (i < total) {
            int q = 0;                                // last row that starts at or before entry i
#pragma unroll
            for (int d = kBinLocalRows / 2; d >= 1; d >>= 1) q += first[q + d] <= i ? d : 0;
            uint32_t entry = (uint32_t)(i - first[q]);
            const uint32_t n_q = len[q];
            if (n_q) {                                // Equation 2; W <= 4096, so the product stays below 2^24
                entry = rot[q] + small_mod(entry * mul[q], n_q);
                if (entry >= n_q) entry -= n_q;
            }
            const int64_t p = (int64_t)src[q] + entry;
            key[m] = (uint32_t)a.colidx[p];
            val[m] = (a.vals ? a.vals[p] : 1.0f) * factor[q];
            place[m] = (uint32_t)q;
        }
    }
#pragma unroll
    for (int m = 0; m < kBinLocalPer; ++m) {
        if (tid + m * kBinLocalRows < total) {
            const uint32_t col = key[m], b = col >> a.log_width;
            key[m] = (uint32_t)(r_begin + place[m]) | ((col - (b << a.log_width)) << kBinRowBits);
            place[m] = b | (uint32_t)atomicAdd(&counter[b], 1) << 12;
        }
    }
    __syncthreads();
    constexpr int PER = kBinMaxBlocks / kBinLocalRows;
    int32_t mine[PER], sum = 0;
    const int b0 = tid * PER;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        mine[i] = b0 + i < a.nbins ? counter[b0 + i] : 0;
        sum += mine[i];
    }
    int32_t all;
    int32_t at = block_scan<kBinLocalRows>(sum, wave_total, all) - sum;
    int32_t* out = a.counts + (int64_t)blockIdx.x * (a.nbins + 1);
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (b0 + i < a.nbins) {
            counter[b0 + i] = at;
            out[b0 + i] = at;
        }
        at += mine[i];
    }
    if (tid == 0) {
        out[a.nbins] = all;
        a.base[blockIdx.x] = own;
    }
    __syncthreads();
    uint2* records = a.records + own;
#pragma unroll
    for (int m = 0; m < kBinLocalPer; ++m)
        if (tid + m * kBinLocalRows < total)
            records[counter[place[m] & 0xFFFu] + (int32_t)(place[m] >> 12)] = make_uint2(key[m], __float_as_uint(val[m]));
}

// Walks the kept entries of this workgroup's rows, 512 rows at a time laid end to
// end: every thread then takes entries, whatever rows they are of.  FILL == false
// counts them per column block, FILL == true writes the records.
template <bool FILL>
__global__ void __launch_bounds__(kBinThreads) es_bin_walk_kernel(const BinArgs a)
{
    extern __shared__ int32_t counter[];              // [nbins]
    __shared__ int32_t first[kBinThreads];
    __shared__ int32_t src[kBinThreads];
    __shared__ uint32_t len[kBinThreads], mul[kBinThreads], rot[kBinThreads];
    __shared__ float factor[kBinThreads];
    __shared__ int32_t wave_total[kBinWaves];
    const int tid = threadIdx.x;
    const int lane = tid & (kWaveSize - 1);
    const int wave = tid >> 6;
    int32_t* mine = a.counts + (int64_t)blockIdx.x * a.nbins;
    for (int b = tid; b < a.nbins; b += kBinThreads) counter[b] = FILL ? a.base[b] + mine[b] : 0;
    const int64_t r_begin = a.N * blockIdx.x / a.walkers, r_end = a.N * (blockIdx.x + 1) / a.walkers;
    for (int64_t r0 = r_begin; r0 < r_end; r0 += kBinThreads) {
        const int64_t r = r0 + tid;
        int32_t n = 0, k = 0;
        if (r < r_end) {
            const int32_t p = a.rowptr[r];
            n = a.rowptr[r + 1] - p;
            k = kept_count(a.mode, n, a.W);
            src[tid] = p;
            const bool strided = a.mode == ES_FASTRAND && n > a.W;
            len[tid] = strided ? (uint32_t)n : 0u;
            mul[tid] = strided ? fastrand_multiplier((uint32_t)n) : 0u;
            rot[tid] = strided ? fastrand_offset(a.seed, r, (uint32_t)n) : 0u;
            if (FILL) factor[tid] = row_factor(a.norm, n, k);
        }
        int32_t incl = k;
#pragma unroll
        for (int d = 1; d < kWaveSize; d <<= 1) {
            const int32_t up = __shfl_up(incl, d, kWaveSize);
            if (lane >= d) incl += up;
        }
        if (lane == kWaveSize - 1) wave_total[wave] = incl;
        __syncthreads();
        int32_t before = incl - k, total = 0;
#pragma unroll
        for (int w = 0; w < kBinWaves; ++w) {
            if (w < wave) before += wave_total[w];
            total += wave_total[w];
        }
        first[tid] = before;
        __syncthreads();
        constexpr int M = 4;                          // entries per thread requested together
        for (int32_t i0 = tid; i0 < total; i0 += M * kBinThreads) {
            int32_t col[M], row[M];
            float val[M];
#pragma unroll
            for (int m = 0; m < M; ++m) {
                const int32_t i = min(i0 + m * kBinThreads, total - 1);
                int q = 0;                            // last row that starts at or before entry i
#pragma unroll
                for (int d = kBinThreads / 2; d >= 1; d >>= 1) q += first[q + d] <= i ? d : 0;
                uint32_t entry = (uint32_t)(i - first[q]);
                const uint32_t n_q = len[q];
                if (n_q) {                            // Equation 2; W <= 4096, so the product stays below 2^24
                    entry = rot[q] + small_mod(entry * mul[q], n_q);
                    if (entry >= n_q) entry -= n_q;
                }
                const int64_t p = (int64_t)src[q] + entry;
                row[m] = q;
                col[m] = a.colidx[p];
                if (FILL) val[m] = a.vals ? a.vals[p] : 1.0f;
            }
#pragma unroll
            for (int m = 0; m < M; ++m) {
                if (i0 + m * kBinThreads >= total) break;
                const int32_t b = col[m] >> a.log_width;
                const int32_t at = atomicAdd(&counter[b], 1);
                if (FILL && at < a.capacity)
                    a.records[at] = make_uint2((uint32_t)(r0 + row[m]) | ((uint32_t)(col[m] - (b << a.log_width)) << kBinRowBits),
                                               __float_as_uint(val[m] * factor[row[m]]));
            }
        }
        __syncthreads();
    }
    if (!FILL)
        for (int b = tid; b < a.nbins; b += kBinThreads) mine[b] = counter[b];
}

// counts[i][b] becomes the records of block b that walkers before i hold; base[b]
// becomes their number in all walkers.  A workgroup takes 64 blocks, a wave a
// sixteenth of the walkers.
constexpr int kBinScanThreads = 1024;
__global__ void __launch_bounds__(kBinScanThreads) es_bin_scan_kernel(const BinArgs a)
{
    constexpr int WAVES = kBinScanThreads / kWaveSize;
    constexpr int PER = kBinWalkers / WAVES;          // walkers of a wave at most
    __shared__ int32_t sums[WAVES][kWaveSize];
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x >> 6;
    const int b = blockIdx.x * kWaveSize + lane;
    const int i0 = wave * PER;
    int32_t v[PER];
    int32_t sum = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        v[i] = (b < a.nbins && i0 + i < a.walkers) ? a.counts[(int64_t)(i0 + i) * a.nbins + b] : 0;
        sum += v[i];
    }
    sums[wave][lane] = sum;
    __syncthreads();
    int32_t before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
        if (w < wave) before += sums[w][lane];
        total += sums[w][lane];
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (b < a.nbins && i0 + i < a.walkers) a.counts[(int64_t)(i0 + i) * a.nbins + b] = before;
        before += v[i];
    }
    if (wave == 0 && b < a.nbins) a.base[b] = total;
}

// One workgroup: base[b] from the blocks' totals to their first records.
__global__ void __launch_bounds__(kBinScanThreads) es_bin_base_kernel(const BinArgs a)
{
    constexpr int WAVES = kBinScanThreads / kWaveSize;
    constexpr int PER = kBinMaxBlocks / kBinScanThreads;
    __shared__ int32_t wave_total[WAVES];
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x >> 6;
    int32_t count[PER];
    int32_t mine = 0;
    const int b0 = threadIdx.x * PER;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        count[i] = b0 + i < a.nbins ? a.base[b0 + i] : 0;
        mine += count[i];
    }
    int32_t incl = mine;
#pragma unroll
    for (int d = 1; d < kWaveSize; d <<= 1) {
        const int32_t up = __shfl_up(incl, d, kWaveSize);
        if (lane >= d) incl += up;
    }
    if (lane == kWaveSize - 1) wave_total[wave] = incl;
    __syncthreads();
    int32_t at = incl - mine;
    for (int w = 0; w < wave; ++w) at += wave_total[w];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (b0 + i <= a.nbins) a.base[b0 + i] = at;   // base[nbins]: all of them
        at += count[i];
    }
    if (threadIdx.x == kBinScanThreads - 1 && a.nbins == kBinMaxBlocks) a.base[a.nbins] = at;
}

// The m-th record that a sorting thread requests in its step from i on, the last one
// in place of what lies behind it.  Unsigned: i runs up to a step behind `end`, which may be 2^31 - 1.
constexpr int kBinSortM = 8;                          // records per thread requested together
constexpr uint32_t kBinSortStep = kBinSortM * kBlockThreads;
__host__ __device__ constexpr uint32_t bin_record(uint32_t i, int m, uint32_t end)
{
    return i + m * kBlockThreads < end ? i + m * kBlockThreads : end - 1;
}
static_assert(bin_record(INT32_MAX - 1u, kBinSortM - 1, INT32_MAX) == INT32_MAX - 1u && INT32_MAX - 1u + kBinSortStep > INT32_MAX,
              "the last records of the largest graph");

// Sorts column block blockIdx.x by column into the transposed graph.  LOCAL: the block's records lie in one
// piece per walker (es_bin_local_kernel).
template <bool LOCAL>
__global__ void __launch_bounds__(kBlockThreads) es_bin_sort_kernel(const BinArgs a)
{
    constexpr int COLS = 1 << (32 - kBinRowBits);     // columns of a block at most
    constexpr int PER = COLS / kBlockThreads;
    constexpr int M = kBinSortM;
    static_assert(!LOCAL || kBinWalkers == kBlockThreads, "one thread per walker");
    __shared__ int32_t cursor[COLS];
    __shared__ int32_t wave_total[kWavesPerBlock];
    __shared__ int32_t piece[LOCAL ? kBinWalkers : 1];                // LOCAL: the walkers' first records of the block,
    __shared__ int32_t where[LOCAL ? kBinWalkers : 1];                // where walker w's lie, less piece[w]
    const int tid = threadIdx.x;
    const int64_t c0 = (int64_t)blockIdx.x << a.log_width;
    const int cols = (int)min((int64_t)1 << a.log_width, a.N - c0);
    uint32_t begin, end;                              // of the block in the transposed graph
    uint32_t shift = 0;                               // from there to the records' numbers
    if constexpr (LOCAL) {
        int32_t from = 0, n = 0;
        const int32_t own = a.base[min(tid, a.walkers - 1)];          // ahead of the counts, a line each: behind them 19.6 us, 18.6 here
        if (tid < a.walkers) {
            const int32_t* c = a.counts + (int64_t)tid * (a.nbins + 1) + blockIdx.x;
            from = c[0];
            n = c[1] - from;
        }
        int32_t before, total;                        // records of all blocks before this one, and of this one
        block_scan<kBlockThreads>(from, wave_total, before);
        piece[tid] = block_scan<kBlockThreads>(n, wave_total, total) - n;
        where[tid] = own + from - piece[tid];
        begin = (uint32_t)min((int64_t)before, a.capacity);
        end = (uint32_t)min((int64_t)before + total, a.capacity);
        shift = begin;
    } else {
        begin = (uint32_t)min((int64_t)a.base[blockIdx.x], a.capacity);
        end = (uint32_t)min((int64_t)a.base[blockIdx.x + 1], a.capacity);
    }
    const auto record_of = [&](uint32_t i) {
        if constexpr (!LOCAL) return i;
        const int32_t j = (int32_t)(i - shift);
        int w = 0;
#pragma unroll
        for (int d = kBinWalkers / 2; d >= 1; d >>= 1) w += piece[w + d] <= j ? d : 0;
        return (uint32_t)(where[w] + j);
    };
    for (int c = tid; c < COLS; c += kBlockThreads) cursor[c] = 0;
    __syncthreads();
    for (uint32_t i0 = begin + tid; i0 < end; i0 += kBinSortStep) {
        uint32_t key[M];
#pragma unroll
        for (int m = 0; m < M; ++m) key[m] = a.records[record_of(bin_record(i0, m, end))].x;
#pragma unroll
        for (int m = 0; m < M; ++m)
            if (i0 + m * kBlockThreads < end) atomicAdd(&cursor[key[m] >> kBinRowBits], 1);
    }
    __syncthreads();
    int32_t count[PER];
    int32_t mine = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) { count[i] = cursor[tid * PER + i]; mine += count[i]; }
    int32_t all;
    int32_t at = (int32_t)begin + block_scan<kBlockThreads>(mine, wave_total, all) - mine;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int c = tid * PER + i;
        cursor[c] = at;
        if (c < cols) a.t_ptr[c0 + c] = at;
        at += count[i];
    }
    if (blockIdx.x == gridDim.x - 1 && tid == 0) a.t_ptr[a.N] = (int32_t)end;
    __syncthreads();
    for (uint32_t i0 = begin + tid; i0 < end; i0 += kBinSortStep) {
        uint2 rec[M];
#pragma unroll
        for (int m = 0; m < M; ++m) rec[m] = a.records[record_of(bin_record(i0, m, end))];
#pragma unroll
        for (int m = 0; m < M; ++m)
            if (i0 + m * kBlockThreads < end) {
                const int32_t to = atomicAdd(&cursor[rec[m].x >> kBinRowBits], 1);
                a.t_row[to] = (int32_t)(rec[m].x & ((1u << kBinRowBits) - 1u));
                a.t_val[to] = __uint_as_float(rec[m].y);
            }
    }
}

}  // namespace

#endif  // ES_SPMM_BIN_KERNEL_H
