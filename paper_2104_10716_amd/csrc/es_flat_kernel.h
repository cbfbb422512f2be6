// es_flat_kernel.h -- stage 1 and stage 2 of Algorithm 1 on a flattened run of rows: edge slots are dealt entries, not rows.
#ifndef ES_SPMM_FLAT_KERNEL_H
#define ES_SPMM_FLAT_KERNEL_H

#include "es_fused_kernel.h"

namespace {

// ---------------------------------------------------------------------------
// Why: with one row (or one row per team) on a wave at a time, every row costs
// a fixed number of instructions and memory round trips, and a wave whose rows
// differ in length idles the lanes of the short ones.  Here a workgroup takes up
// to 64 consecutive rows (or the pieces of one column range of those rows), lays
// their kept entries end to end -- each row padded to a multiple of a block of
// max(8, E) entries, E = 64 / G edge slots, with absent ones, which touch no memory and
// multiply nothing -- and stages that run into LDS in bursts of 1536 or 2048 entries (stage 1
// of Algorithm 1): a table of the burst's blocks first (a binary search per block
// for its row), then every entry of the burst requested before the first is
// awaited.  Stage 2: each of the four waves multiplies an equal share of the
// run, whatever rows it holds, E entries per step, 8 steps' rows of X in flight
// together.  Because of the padding a step never straddles two rows, so "a row
// ends here" is a wave-uniform bit (scalar test); there the slots' sums are added
// across the wave with lane swaps and written to the row's place in LDS.  A row
// that crosses into the next wave's share (or the next burst) leaves the second
// part in that wave's own place; the parts are added in a fixed order, so the
// sums are bit-reproducible.  Row sums leave LDS once, coalesced (plain stores, or
// load-add-store in the later phases of the column-partitioned product).
//
// What bounds it: the L2 misses of the gathers where X is large (7.4 TB/s of them). Where
// nearly all gathers hit, the vector cache, which serves 64 bytes per clock and compute unit, be
// they one lane's or sixteen lanes': 84 M such accesses per launch of the dense social-like graph's exact product in
// column ranges (233 k rows, 113 M entries, F = 64), 60 M of them rows of X, in 264 us; with every access a hit
// still 217 us.  Hence a chunk's entries are loaded in order and permuted on their way into LDS (a permuted load
// touches three times as many lines), and the cuts lie range by range: 2.17 -> 2.06 ms, 233 k rows of mean 150,
// F = 128 1628 -> 1548 us.  Lines that miss hold back the hits behind them; the bursts put a workgroup's
// misses on the entries together (2.59 -> 2.16 ms against 256 entries per wave, requested one tile ahead).
// Co-purchase-like graph (2.45 M rows, 120 M entries, F = 128), 46 % hits: exact product 5.60 ms, FastRand W = 64 2.76.
// Tried and slower: entries kept in registers and handed to the slots by DPP, a row's 64 at a time (2.83 ms: short
// pieces fill a quarter of the lanes), non-temporal loads for rows of X far from the row's own index (9 - 20 % fewer L2
// misses, 4 - 15 % slower), seven or eight waves per SIMD with bursts of 512 or 1024 (2.26, 2.44 ms).
// Tried and slower on the form with permuted loads (2.17 ms): entries copied into LDS by the load itself (dword
// copies: 2.9 ms), a pass of 64 entries per row streamed two passes ahead (2.6 ms), 16
// column ranges (3.2 ms), two batches of gathers in flight per wave (spills or 12 waves).
// The 64-bit form branches round absent entries' gathers; over permuted loads that multiplied padding: 0.985 - 1.005 of the
// time (1.1 to 2.45 M rows, F = 128 to 448 at row stride 1024, exact and sampled: 2.45 M, F = 128 7302 / 7301, FastRand W = 64 3564 / 3533 us).
// ---------------------------------------------------------------------------
constexpr int kFlatMaxRows = 64;                      // rows of a workgroup's run at most: one per lane
constexpr int kFlatBlockMin = 8;                      // smallest unit a row is padded to
constexpr int kFlatLongRow = 8192;                    // kept entries above which a row goes to the long-row part (unless the mean is near)
constexpr int kFlatLongSeg = 2048;                    // slots per segment of such a row

// Rows of a run with G column lanes: `rps` rows per edge slot of each wave.
constexpr int flat_rows(int G, int rps) { return rps * 256 / G < kFlatMaxRows ? rps * 256 / G : kFlatMaxRows; }

template <int G_, int RPS>
struct FlatLds {
    static constexpr int G = G_;                      // lanes across the feature columns
    static constexpr int FB = 4 * G;                  // feature columns per block
    static constexpr int ROWS = flat_rows(G, RPS);    // rows of the run
    static constexpr int CAP = RPS == 1 ? 1536 : 2048;   // entries staged in one burst: about the run's mean, six or four workgroups per compute unit
    uint32_t key[CAP];                           // staged entries' rows of X (kFlatAbsent), in the order the slots read them
    float val[CAP];
    float rowsum[ROWS * FB];                     // [row][FB]
    float head[kWavesPerBlock * FB];                  // per wave: partial sum of a row that began in an earlier wave's share
    int32_t head_row[kWavesPerBlock];
    uint2 block[CAP / kFlatBlockMin];                      // staged block: CSR position (or slot) of its first entry; entries | row << 8
    uint64_t ends[CAP / kFlatBlockMin / kWaveSize];        // bit b: staged block b is the last of its row
    int32_t first[kFlatMaxRows];                         // the rows: first block of the run,
    int32_t src[kFlatMaxRows];                           // CSR position of the row's (piece's) entry 0, < 2^31
    int32_t kept[kFlatMaxRows];                          // entries the row really keeps
    uint32_t len[kFlatMaxRows];                          // FastRand on a longer row: its length n; else 0
    uint32_t mul[kFlatMaxRows];                          //   multiplier P
    uint32_t rot[kFlatMaxRows];                          //   rotation off
};

// What a lane reads when it has no entry to stage (an absent entry's value), and
// the value of every entry of an unweighted graph.
__device__ const float kFlatConst[2] = {0.0f, 1.0f};

// Lanes whose bit BIT (4 or 5) is clear get a + a', the others b + b', where a',
// b' are the values of the lane that differs in that bit alone: the row and
// half-wave swaps of gfx950 (odd rows of 16 lanes of the first operand trade
// places with even rows of the second; the upper half of the first with the lower
// half of the second), then one add.  No LDS traffic.
template <int BIT>
__device__ __forceinline__ float halve_add(float a, float b)
{
    static_assert(BIT == 4 || BIT == 5, "swaps of rows of 16 lanes and of half waves");
    if constexpr (BIT == 5) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
}

// v + the values of the lanes that differ from this one in bit BIT (2 or 3) and
// agree in the lower ones: a rotation by 2^BIT inside a row of 16 lanes.  For
// bit 2 the values must already be equal across bit 3.
template <int BIT>
__device__ __forceinline__ float all_add(float v)
{
    static_assert(BIT == 2 || BIT == 3, "rotations inside a row of 16");
    constexpr int kRowRor = 0x120 + (1 << BIT);
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kRowRor, 0xf, 0xf, true));
}


// x mod n for n < 2^31 and any x < 2^24: quotient from a float reciprocal (off by
// one at most: x and the quotient's error bound stay below 2^24).
__device__ __forceinline__ uint32_t small_mod(uint32_t x, uint32_t n)
{
    const uint32_t q = (uint32_t)((float)x * __builtin_amdgcn_rcpf((float)n));
    int32_t r = (int32_t)(x - q * n);
    if (r < 0) r += (int32_t)n;
    if (r >= (int32_t)n) r -= (int32_t)n;
    return (uint32_t)r;
}

__device__ __forceinline__ int32_t lane_of(int32_t v, int lane) { return __builtin_amdgcn_readlane(v, lane); }


// One row (piece) per lane: the workgroup's run, held alike by all of its waves.
struct FlatRow {
    int32_t src;               // CSR position of entry 0 of the row (piece)
    int32_t k;                 // entries to multiply, 0 for lanes past the run
    uint32_t len, mul, rot;    // FastRand on a longer row: slot i reads entry (rot + i * mul) mod len; len == 0: entry i
};

// How a staged entry names its row of X.
// WIDE == false: by the byte offset of the row, for a buffer load; an absent entry by an offset past the
// buffer's end, which reads as zero and touches no memory.  WIDE == true (tables of 4 GB and more): by the column id.
constexpr uint32_t kFlatAbsent = 0xFE000000u;         // + the bytes of one row (< 2^24) does not wrap
constexpr uint64_t kFlatMaxBytes = kFlatAbsent;       // largest table of the 32-bit form
constexpr uint32_t kFlatAbsentWide = 0xFFFFFFFFu;

typedef uint32_t uint4_v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float4 buffer_row(__amdgpu_buffer_rsrc_t rsrc, uint32_t at)
{
    const uint4_v t = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)at, 0, 0);
    return make_float4(__uint_as_float(t.x), __uint_as_float(t.y), __uint_as_float(t.z), __uint_as_float(t.w));
}

// Multiplies the workgroup's run: row j's sum goes to s.rowsum[j][FB] (rows
// without entries: zeros). Ends with a barrier.
template <bool ALIGNED, bool WIDE, bool STRIDED, class Lds>
__device__ __forceinline__ void flat_run(const Args& a, const FlatRow& row, int colblk, Lds& s)
{
    constexpr int G = Lds::G;
    constexpr int LOG_G = ilog2(G);
    constexpr int LOG_E = 6 - LOG_G;
    constexpr int E = kWaveSize / G;                  // edge slots
    constexpr int FB = 4 * G;                         // feature columns per block
    constexpr int BE = E < kFlatBlockMin ? kFlatBlockMin : E;   // entries per block
    constexpr int LOG_BE = ilog2(BE);
    constexpr int CAPB = Lds::CAP / BE;               // blocks per burst
    constexpr int BPC = kWaveSize / BE;               // blocks per chunk of 64 entries
    constexpr int U = 8;                              // steps per batch = gathers in flight per lane
    constexpr int BPB = U * E / BE;                   // blocks per batch (1, 2, 4 or 8)
    using P = Pack<4, ALIGNED>;

    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int e = lane >> LOG_G;
    const int l = lane & (G - 1);
    LaneCols<G, 1, 4, ALIGNED> cols;
    cols.init(colblk, l, a.F);

    // ---- the run in blocks --------------------------------------------------------
    const int32_t nb = (row.k + BE - 1) >> LOG_BE;
    int32_t incl = nb;                                // inclusive scan over the 64 rows
#pragma unroll
    for (int d = 1; d < kWaveSize; d <<= 1) {
        const int32_t up = __shfl_up(incl, d, kWaveSize);
        if (lane >= d) incl += up;
    }
    const int32_t total = lane_of(incl, kWaveSize - 1);
    const uint64_t nonempty = __ballot(row.k > 0);
    if (wave == 0) {
        s.first[lane] = incl - nb;
        s.src[lane] = row.src;
        s.kept[lane] = row.k;
        if constexpr (STRIDED) {
            s.len[lane] = row.len;
            s.mul[lane] = row.mul;
            s.rot[lane] = row.rot;
        }
    }
    for (int i = threadIdx.x * 4; i < Lds::ROWS * FB; i += kBlockThreads * 4)
        *reinterpret_cast<float4*>(&s.rowsum[i]) = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();

    // A chunk's 64 entries are loaded one per lane, in order, so that a load touches few lines, and stored in
    // the order in which the slots read them: a slot's four consecutive steps side by side (one 128-bit LDS read).
    const int c_block = lane >> LOG_BE;
    const int c_in = lane & (BE - 1);
    const int c_put = (lane >> (LOG_E + 2) << (LOG_E + 2)) + ((lane & (E - 1)) << 2) + ((lane >> LOG_E) & 3);
    const uint32_t* get_key = s.key + e * 4;
    const float* get_val = s.val + e * 4;
    const uint64_t stride = (uint64_t)a.ldx * 4u;     // bytes from one row of X to the next: up to 33 bits
    const uint32_t load_at = (uint32_t)cols.off[0] * 4u;
    const char* X = reinterpret_cast<const char*>(a.X);
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.X), 0,
                                                        (int)(uint32_t)min((uint64_t)a.N * stride, kFlatMaxBytes), 0x00027000);

    struct Batch { P x[U]; };
    auto gather = [&](int s0, Batch& bt) {
#pragma unroll
        for (int q = 0; q < U / 4; ++q) {
            const uint4 key = *reinterpret_cast<const uint4*>(get_key + (s0 + 4 * q) * E);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t k = (&key.x)[u];
                P& x = bt.x[4 * q + u];
                if constexpr (WIDE) {
                    x.zero();
                    if (k != kFlatAbsentWide) x.load(reinterpret_cast<const float*>(X + (k * stride + load_at)));
                } else {
                    x.v = buffer_row(rsrc, k + load_at);
                }
            }
        }
    };

    for (int b0 = 0; b0 < total; b0 += CAPB) {
        const int nblk = min(total - b0, CAPB);
        const int batches = (nblk + BPB - 1) / BPB;
        // ---- the burst's blocks: which row, where, how many entries --------------------
        const int chunks = (batches * U * E + kWaveSize - 1) / kWaveSize;
#pragma unroll 1
        for (int i = threadIdx.x; i < CAPB; i += kBlockThreads) {
            const int b = b0 + i;
            const int bc = min(b, total - 1);
            int r = 0;                                        // last row that starts at or before block bc and is not empty
#pragma unroll
            for (int d = kFlatMaxRows / 2; d >= 1; d >>= 1) r += s.first[r + d] <= bc ? d : 0;
            const int32_t i0 = (bc - s.first[r]) << LOG_BE;
            const int32_t left = s.kept[r] - i0;
            bool strided = false;
            if constexpr (STRIDED) strided = s.len[r] != 0;
            s.block[i] = make_uint2((uint32_t)(strided ? i0 : s.src[r] + i0),
                                    (uint32_t)(b < total ? min(left, BE) : 0) | ((uint32_t)r << 8));
            const uint64_t ends = __ballot(b < total && left <= BE);
            if (lane == 0) s.ends[i / kWaveSize] = ends;
        }
        __syncthreads();
        // ---- stage 1: the burst's entries, all requested before the first is awaited ----
        constexpr int M = 4;
#pragma unroll 1
        for (int q0 = wave; q0 < chunks; q0 += M * kWavesPerBlock) {
            int32_t col[M];
            float val[M];
            bool there[M];
#pragma unroll
            for (int i = 0; i < M; ++i) {
                const int q = min(q0 + i * kWavesPerBlock, chunks - 1);
                const uint2 blk = s.block[q * BPC + c_block];
                const int32_t cnt = (int32_t)(blk.y & 0xFFu);
                uint32_t pos = blk.x + (uint32_t)max(min(c_in, cnt - 1), 0);   // absent entries repeat one of the row's
                if constexpr (STRIDED) {
                    const uint32_t r = blk.y >> 8;
                    const uint32_t n = s.len[r];
                    if (n) {
                        uint32_t step;
                        if (a.W < 28000) step = small_mod(pos * s.mul[r], n);          // pos < W: below 2^24
                        else step = (uint32_t)(((uint64_t)pos * s.mul[r]) % n);
                        uint32_t entry = s.rot[r] + step;         // both < n < 2^31
                        if (entry >= n) entry -= n;
                        pos = (uint32_t)s.src[r] + entry;
                    }
                }
                const float* v = a.vals ? a.vals + pos : kFlatConst + 1;
                there[i] = c_in < cnt;
                v = there[i] ? v : kFlatConst;                    // absent entries: zero
                col[i] = __builtin_nontemporal_load(a.colidx + pos);
                val[i] = __builtin_nontemporal_load(v);
            }
#pragma unroll
            for (int i = 0; i < M; ++i) {
                const int q = min(q0 + i * kWavesPerBlock, chunks - 1);
                uint32_t key;
                if constexpr (WIDE) {
                    key = there[i] ? (uint32_t)col[i] : kFlatAbsentWide;
                } else {
                    key = __umul24((uint32_t)col[i], (uint32_t)stride);
                    key = there[i] ? key : kFlatAbsent;
                }
                s.key[q * kWaveSize + c_put] = key;
                s.val[q * kWaveSize + c_put] = val[i];
            }
        }
        __syncthreads();
        // ---- stage 2: every wave an equal share of the batches ------------------------
        const int first_batch = batches * wave / kWavesPerBlock;
        const int last_batch = batches * (wave + 1) / kWavesPerBlock;
        int32_t head = -1;
        if (first_batch < last_batch) {
            const int blk0 = first_batch * BPB;
            int r = __builtin_amdgcn_readfirstlane((int)(s.block[blk0].y >> 8));
            // a row that began before this wave's share leaves its sum in the wave's own place
            if (__builtin_amdgcn_readfirstlane(s.first[r]) < b0 + blk0) head = r;
            uint64_t pending = nonempty & ~((2ull << r) - 1ull);  // rows behind r
            bool at_head = head >= 0;
            P acc;
            acc.zero();
            auto flush = [&]() {
                float* dst = (at_head ? s.head + wave * FB : s.rowsum + r * FB) + l * 4;
                if constexpr (E == 1) {
                    *reinterpret_cast<float4*>(dst) = acc.v;
                } else if constexpr (E == 2) {
                    const float s0 = halve_add<5>(acc.v.x, acc.v.z);
                    const float s1 = halve_add<5>(acc.v.y, acc.v.w);
                    *reinterpret_cast<float2*>(dst + 2 * e) = make_float2(s0, s1);
                } else {
                    const float s0 = halve_add<4>(acc.v.x, acc.v.z);    // bit 4 clear: x, set: z
                    const float s1 = halve_add<4>(acc.v.y, acc.v.w);    //              y       w
                    float v = halve_add<5>(s0, s1);                     // bit 5 clear: s0, set: s1
                    if constexpr (LOG_E > 2) v = all_add<3>(v);
                    if constexpr (LOG_E > 3) v = all_add<2>(v);
                    const int top = e >> (LOG_E - 2);                   // lane bits 4, 5
                    dst[2 * (top & 1) + (top >> 1)] = v;                // slots that differ in lower bits hold the same sum
                }
                acc.zero();
                at_head = false;
                r = pending ? __builtin_ctzll(pending) : kFlatMaxRows;  // kFlatMaxRows: nothing left
                pending &= pending - 1;
            };
            auto multiply = [&](int batch, const Batch& bt) {
                const uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane(
                    (int)(reinterpret_cast<const uint32_t*>(s.ends)[batch * BPB / 32] >> (batch * BPB % 32)));
                float4 val[U / 4];
#pragma unroll
                for (int q = 0; q < U / 4; ++q)
                    val[q] = *reinterpret_cast<const float4*>(get_val + (batch * U + 4 * q) * E);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    acc.fma((&val[u / 4].x)[u & 3], bt.x[u]);
                    if (((u + 1) * E) % BE == 0 && (end & (1u << ((u * E) / BE)))) flush();
                }
            };
            Batch xa;
#pragma unroll 1
            for (int b = first_batch; b < last_batch; ++b) { gather(b * U, xa); multiply(b, xa); }
            // the share's last row may go on in the next one
            const int blk1 = last_batch * BPB - 1;
            const uint32_t ended = reinterpret_cast<const uint32_t*>(s.ends)[blk1 / 32] >> (blk1 % 32);
            if (!(__builtin_amdgcn_readfirstlane((int)ended) & 1) && r < kFlatMaxRows) flush();
        }
        if (lane == 0) s.head_row[wave] = head;
        __syncthreads();
        if (threadIdx.x < FB) {
#pragma unroll
            for (int w = 0; w < kWavesPerBlock; ++w) {
                const int32_t hr = s.head_row[w];
                if (hr >= 0) s.rowsum[hr * FB + threadIdx.x] += s.head[w * FB + threadIdx.x];
            }
        }
        __syncthreads();
    }
}

// The run of workgroup `vb`: whole sampled rows, or with PART the pieces of
// column range `part` (ACC: add to Y instead of overwriting it).
template <bool ALIGNED, bool WIDE, bool STRIDED, bool PART, bool ACC, class Lds>
__device__ __forceinline__ void flat_block(const Args& a, uint32_t vb, int part, Lds& s)
{
    constexpr int G = Lds::G;
    constexpr int ROWS = Lds::ROWS;
    constexpr int FB = 4 * G;
    constexpr int RPP = kBlockThreads / G;            // rows out per pass
    constexpr int PASSES = (ROWS + RPP - 1) / RPP;
    using P = Pack<4, ALIGNED>;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int l = threadIdx.x & (G - 1);
    const int jr = threadIdx.x / G;
    const int colblk = blockIdx.y * FB;
    LaneCols<G, 1, 4, ALIGNED> cols;
    cols.init(colblk, l, a.F);
    const int64_t r0 = (int64_t)vb * ROWS;
    FlatRow row{0, 0, 0, 0, 0};
    int32_t my_n = 0, my_k = 0;
    bool my_store = false;                            // this launch writes the row's Y
    const int64_t r = r0 + lane;
    if (lane < ROWS && r < a.N) {
        const int32_t base = a.rowptr[r];
        my_n = a.rowptr[r + 1] - base;
        my_k = kept_count(a.mode, my_n, a.W);
        if constexpr (PART) {
            const int32_t lo = a.cuts[part * a.N + r];
            const int32_t hi = (part + 1 < kParts) ? a.cuts[(part + 1) * a.N + r] : my_n;
            row.src = base + lo;
            row.k = hi - lo;
            my_store = !ACC || hi > lo;
        } else {
            my_store = my_k <= a.long_k;              // longer rows belong to the long-row part
            row.src = base;
            row.k = my_store ? my_k : 0;
            if (STRIDED && my_n > a.W) {
                row.len = (uint32_t)my_n;
                row.mul = fastrand_multiplier(row.len);
                row.rot = fastrand_offset(a.seed, r, row.len);
            }
        }
    }
    P prev[PASSES];
    if constexpr (ACC) {                              // earlier partial sums, requested ahead of the entries
#pragma unroll
        for (int pass = 0; pass < PASSES; ++pass) {
            const int64_t ry = min(r0 + min(pass * RPP + jr, ROWS - 1), a.N - 1);
            prev[pass].load_streaming(a.Y + ry * (int64_t)a.ldy + cols.off[0]);
        }
    }
    flat_run<ALIGNED, WIDE, STRIDED>(a, row, colblk, s);
#pragma unroll
    for (int pass = 0; pass < PASSES; ++pass) {
        const int j = pass * RPP + jr;
        const bool store = __shfl((int)my_store, j, kWaveSize) != 0;
        P out;
        out.v = *reinterpret_cast<const float4*>(&s.rowsum[j * FB + l * 4]);
        if (a.norm != ES_NORM_NONE)
            out.scale(row_factor(a.norm, __shfl(my_n, j, kWaveSize), __shfl(my_k, j, kWaveSize)));
        if constexpr (ACC) out.add(prev[pass]);
        if (store && cols.ok[0]) out.store_streaming(a.Y + (r0 + j) * (int64_t)a.ldy + cols.off[0], cols.first[0]);
    }
}

// Long-row part, as long_block in es_fused_kernel.h: the workgroup's share of the
// segments of the long rows among its 1024, added to Y with fp32 atomics.
template <bool ALIGNED, bool WIDE, bool STRIDED, class Lds>
__device__ __forceinline__ void flat_long_block(const Args& a, uint32_t bx, uint32_t by, Lds& s, LongScratch& sc)
{
    constexpr int G = Lds::G;
    constexpr int FB = 4 * G;
    const int total = long_segments<kFlatLongSeg>(a, bx, sc);
    const int lane = threadIdx.x & (kWaveSize - 1);
    LaneCols<G, 1, 4, ALIGNED> cols;
    cols.init(blockIdx.y * FB, threadIdx.x & (G - 1), a.F);
    for (int task = by; task < total; task += kLongSplit) {
        const LongSegment sg = long_segment<kFlatLongSeg>(a, bx, task, sc);
        FlatRow row{sg.base, lane == 0 ? sg.count : 0, 0, 0, 0};
        if (STRIDED && sg.n > a.W) {
            row.len = (uint32_t)sg.n;
            row.mul = fastrand_multiplier(row.len);
            row.rot = (uint32_t)(((uint64_t)sg.t0 * row.mul + fastrand_offset(a.seed, sg.r, row.len)) % row.len);
        } else {
            row.src += sg.t0;
        }
        flat_run<ALIGNED, WIDE, STRIDED>(a, row, blockIdx.y * FB, s);
        if (threadIdx.x < G) {
            Pack<4, ALIGNED> out;
            out.v = *reinterpret_cast<const float4*>(&s.rowsum[threadIdx.x * 4]);
            if (a.norm != ES_NORM_NONE) out.scale(row_factor(a.norm, sg.n, sg.k));
            if (cols.ok[0]) out.atomic_add(a.Y + sg.r * (int64_t)a.ldy + cols.off[0], cols.first[0]);
        }
        __syncthreads();
    }
}

// The forward kernel on flattened rows: as es_spmm_kernel, the leading
// a.long_blocks workgroups split the rows that keep more than a.long_k entries
// (those rows are left out of the flattened runs), the rest serve
// flat_rows(G, RPS) rows each, remapped so that every XCD walks one contiguous range of rows.
template <int G, bool ALIGNED, bool WIDE, bool STRIDED, int RPS>
__global__ void __launch_bounds__(kBlockThreads) es_spmm_flat_kernel(const Args a)
{
    __shared__ __align__(16) FlatLds<G, RPS> lds;
    __shared__ LongScratch sc;
    if (blockIdx.x < a.long_blocks) {
        flat_long_block<ALIGNED, WIDE, STRIDED>(a, blockIdx.x / kLongSplit, long_share(blockIdx.x), lds, sc);
        return;
    }
    const uint32_t b = blockIdx.x - a.long_blocks;
    const uint32_t vb = (b % kNumXcd) * a.blocks_per_xcd + b / kNumXcd;
    if (vb >= a.nblocks) return;
    flat_block<ALIGNED, WIDE, STRIDED, false, false>(a, vb, 0, lds);
}

// One phase of the column-partitioned exact product on flattened pieces (see
// es_part_kernel.h for the phases): XCD p = b % 8 serves column range p of the
// rows of row range (p + phase) % 8.
template <int G, bool ALIGNED, bool WIDE, bool ACC>
__global__ void __launch_bounds__(kBlockThreads) es_spmm_part_flat_kernel(const Args a)
{
    __shared__ __align__(16) FlatLds<G, 2> lds;
    const uint32_t p = blockIdx.x % kNumXcd;
    const uint32_t q = blockIdx.x / kNumXcd;
    const uint32_t vb = ((p + (uint32_t)a.phase) % kNumXcd) * a.blocks_per_xcd + q;
    if (vb >= a.nblocks) return;
    flat_block<ALIGNED, WIDE, false, true, ACC>(a, vb, (int)p, lds);
}

}  // namespace

#endif  // ES_SPMM_FLAT_KERNEL_H
