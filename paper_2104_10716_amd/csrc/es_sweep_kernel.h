// es_sweep_kernel.h -- stage 1 and stage 2 of Algorithm 1 on several hundred rows at a time, their entries in column order.
#ifndef ES_SPMM_SWEEP_KERNEL_H
#define ES_SPMM_SWEEP_KERNEL_H

#include "es_flat_kernel.h"

namespace {

constexpr int kSweepWaves = 8;
constexpr int kSweepThreads = kSweepWaves * kWaveSize;
constexpr int kSweepGroups = 512;                    // workgroups resident together: two on each of 256 compute units

template <int G_>
struct SweepLds {
    static constexpr int G = G_;
    static constexpr int FB = 4 * G;
    static constexpr int ROWS = G == 8 ? 464 : G == 16 ? 240 : 120;
    static constexpr int CAP = 1536;
    static constexpr int E = kWaveSize / G;
    static constexpr int BE = E < 8 ? 8 : E;
    static constexpr int CAPB = CAP / BE;
    int32_t col[CAP];
    float val[CAP];
    float rowsum[ROWS * FB];
    float head[kSweepWaves * FB];
    int32_t head_row[kSweepWaves];
    uint2 block[CAPB];
    uint64_t ends[(CAPB + 63) / 64];
    int32_t first[512];                               // of the window, per row: first block,
    int32_t src[ROWS];                                //   CSR position of that block,
    int32_t left[ROWS];                               //   entries of the row from there on
    int32_t wave_total[kSweepWaves];
    int32_t bounds[2];
};

// First row r with rowptr[r] + c * r >= target, by 64 probes at a time.
__device__ __forceinline__ int64_t sweep_bound(const Args& a, double c, double target)
{
    const int lane = threadIdx.x & (kWaveSize - 1);
    int64_t lo = 0, hi = a.N;                          // answer in [lo, hi]
    while (hi > lo) {
        const int64_t step = (hi - lo + kWaveSize - 1) / kWaveSize;
        const int64_t r = lo + (int64_t)lane * step;
        const bool below = r < hi && (double)a.rowptr[r] + c * (double)r < target;
        const int cnt = __popcll(__ballot(below));
        if (cnt == 0) return lo;
        const int64_t last = lo + (int64_t)(cnt - 1) * step;      // still below
        hi = min(hi, last + step);
        lo = last + 1;
    }
    return lo;
}

template <int G, bool ALIGNED>
__global__ void __launch_bounds__(kSweepThreads) es_spmm_sweep_kernel(const Args a, int windows, double per_row)
{
    using Lds = SweepLds<G>;
    __shared__ __align__(16) Lds s;
    constexpr int LOG_G = ilog2(G);
    constexpr int LOG_E = 6 - LOG_G;
    constexpr int E = Lds::E;
    constexpr int FB = Lds::FB;
    constexpr int BE = Lds::BE;
    constexpr int LOG_BE = ilog2(BE);
    constexpr int CAPB = Lds::CAPB;
    constexpr int BPC = kWaveSize / BE;
    constexpr int U = 8;
    constexpr int BPB = U * E / BE;
    constexpr int ROWS = Lds::ROWS;
    using P = Pack<4, ALIGNED>;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int e = lane >> LOG_G;
    const int l = lane & (G - 1);
    const uint32_t vb = (blockIdx.x % kNumXcd) * a.blocks_per_xcd + blockIdx.x / kNumXcd;
    if (vb >= a.nblocks) return;
    const int colblk = blockIdx.y * FB;
    LaneCols<G, 1, 4, ALIGNED> cols;
    cols.init(colblk, l, a.F);

    if (wave < 2) {
        int64_t b;
        if (per_row >= 0.0) {
            const double total = (double)a.rowptr[a.N] + per_row * (double)a.N;
            const uint32_t v = vb + wave;
            b = v == 0 ? 0 : v == a.nblocks ? a.N : sweep_bound(a, per_row, total * (double)v / (double)a.nblocks);
        } else {
            b = (int64_t)((uint64_t)a.N * (vb + wave) / a.nblocks);
        }
        if (lane == 0) s.bounds[wave] = (int32_t)b;
    }
    __syncthreads();
    const int64_t row_first = s.bounds[0], row_last = s.bounds[1];

    const int c_entry = (((lane >> (LOG_E + 2)) * 4 + (lane & 3)) << LOG_E) + ((lane & (4 * E - 1)) >> 2);
    const int c_block = c_entry >> LOG_BE;
    const int c_in = c_entry & (BE - 1);
    const int32_t* get_col = s.col + e * 4;
    const float* get_val = s.val + e * 4;
    const uint32_t stride = (uint32_t)a.ldx * 4u;
    const uint32_t load_at = (uint32_t)cols.off[0] * 4u;
    const char* X = reinterpret_cast<const char*>(a.X);

    for (int64_t r0 = row_first; r0 < row_last; r0 += ROWS) {
        const int nrows = (int)min((int64_t)ROWS, row_last - r0);
        int32_t base = 0, n = 0, k = 0;
        if ((int)threadIdx.x < nrows) {
            base = a.rowptr[r0 + threadIdx.x];
            n = a.rowptr[r0 + threadIdx.x + 1] - base;
            k = kept_count(a.mode, n, a.W);
            if (k > a.long_k) k = 0;                  // the long-row part's
        }
        const int32_t nb = (k + BE - 1) >> LOG_BE;
        const int32_t nb_full = (n + BE - 1) >> LOG_BE;
        for (int i = threadIdx.x * 4; i < ROWS * FB; i += kSweepThreads * 4)
            *reinterpret_cast<float4*>(&s.rowsum[i]) = make_float4(0.f, 0.f, 0.f, 0.f);

        int32_t lo = 0;
        for (int t = 0; t < windows; ++t) {
            int32_t hi = t + 1 == windows ? nb : min(nb, (int32_t)((int64_t)nb_full * (t + 1) / windows));
            const int32_t mine = hi - lo;
            int32_t incl = mine;
#pragma unroll
            for (int d = 1; d < kWaveSize; d <<= 1) {
                const int32_t up = __shfl_up(incl, d, kWaveSize);
                if (lane >= d) incl += up;
            }
            if (lane == kWaveSize - 1) s.wave_total[wave] = incl;
            __syncthreads();
            int32_t before = incl - mine, total = 0;
#pragma unroll
            for (int w = 0; w < kSweepWaves; ++w) {
                const int32_t wt = s.wave_total[w];
                if (w < wave) before += wt;
                total += wt;
            }
            s.first[threadIdx.x] = before;
            if ((int)threadIdx.x < ROWS) {
                s.src[threadIdx.x] = base + lo * BE;
                s.left[threadIdx.x] = k - lo * BE;
            }
            __syncthreads();
            lo = hi;
            for (int b0 = 0; b0 < total; b0 += CAPB) {
                const int nblk = min(total - b0, CAPB);
                const int batches = (nblk + BPB - 1) / BPB;
                const int chunks = (batches * U * E + kWaveSize - 1) / kWaveSize;
                for (int i = threadIdx.x; i < CAPB; i += kSweepThreads) {
                    const int b = b0 + i;
                    const int bc = min(b, total - 1);
                    int r = 0;
#pragma unroll
                    for (int d = 256; d >= 1; d >>= 1) r += s.first[r + d] <= bc ? d : 0;
                    // among rows that start at the same block the last one holds it (the others are empty)
                    const int32_t i0 = (bc - s.first[r]) << LOG_BE;
                    const int32_t left = s.left[r] - i0;
                    const int next = r + 1 < 512 ? s.first[r + 1] : total;
                    s.block[i] = make_uint2((uint32_t)(s.src[r] + i0), (uint32_t)(b < total ? min(left, BE) : 0) | ((uint32_t)r << 8));
                    const uint64_t ends = __ballot(b < total && bc + 1 == next);
                    if (lane == 0) s.ends[i / kWaveSize] = ends;
                }
                __syncthreads();
                constexpr int M = Lds::CAP / kSweepThreads;
                {
                    int32_t col[M];
                    float val[M];
#pragma unroll
                    for (int i = 0; i < M; ++i) {
                        const int q = min(wave + i * kSweepWaves, chunks - 1);
                        const uint2 blk = s.block[q * BPC + c_block];
                        const int32_t cnt = (int32_t)(blk.y & 0xFFu);
                        const uint32_t pos = blk.x + (uint32_t)max(min(c_in, cnt - 1), 0);
                        const float* v = a.vals ? a.vals + pos : kFlatConst + 1;
                        v = c_in < cnt ? v : kFlatConst;
                        col[i] = __builtin_nontemporal_load(a.colidx + pos);
                        val[i] = __builtin_nontemporal_load(v);
                    }
#pragma unroll
                    for (int i = 0; i < M; ++i) {
                        const int q = min(wave + i * kSweepWaves, chunks - 1);
                        s.col[q * kWaveSize + lane] = col[i];
                        s.val[q * kWaveSize + lane] = val[i];
                    }
                }
                __syncthreads();
                const int first_batch = batches * wave / kSweepWaves;
                const int last_batch = batches * (wave + 1) / kSweepWaves;
                int32_t head = -1;
                if (first_batch < last_batch) {
                    const int blk0 = first_batch * BPB;
                    const int rr = __builtin_amdgcn_readfirstlane((int)(s.block[blk0].y >> 8));
                    if (wave > 0 && __builtin_amdgcn_readfirstlane(s.first[rr]) < b0 + blk0) head = rr;
                    bool at_head = head >= 0;
                    P acc;
                    acc.zero();
                    auto flush = [&](int r) {
                        if constexpr (E == 2) {
                            const float s0 = halve_add<5>(acc.v.x, acc.v.z);
                            const float s1 = halve_add<5>(acc.v.y, acc.v.w);
                            float* dst = (at_head ? s.head + wave * FB : s.rowsum + r * FB) + l * 4 + 2 * e;
                            if (at_head) { dst[0] = s0; dst[1] = s1; }
                            else { unsafeAtomicAdd(dst, s0); unsafeAtomicAdd(dst + 1, s1); }
                        } else {
                            const float s0 = halve_add<4>(acc.v.x, acc.v.z);
                            const float s1 = halve_add<4>(acc.v.y, acc.v.w);
                            float v = halve_add<5>(s0, s1);
                            if constexpr (LOG_E > 2) v = all_add<3>(v);
                            const int top = e >> (LOG_E - 2);
                            const int at = l * 4 + 2 * (top & 1) + (top >> 1);
                            if (at_head) s.head[wave * FB + at] = v;
                            else if (LOG_E == 2 || (e & 1) == 0) unsafeAtomicAdd(&s.rowsum[r * FB + at], v);
                        }
                        acc.zero();
                        at_head = false;
                    };
                    bool open = false;
                    int row_open = 0;
#pragma unroll 1
                    for (int b = first_batch; b < last_batch; ++b) {
                        P x[U];
#pragma unroll
                        for (int q = 0; q < U / 4; ++q) {
                            const int4 col = *reinterpret_cast<const int4*>(get_col + (b * U + 4 * q) * E);
#pragma unroll
                            for (int u = 0; u < 4; ++u)
                                x[4 * q + u].load(reinterpret_cast<const float*>(
                                    X + (uint32_t)(__umul24((uint32_t)(&col.x)[u], stride) + load_at)));
                        }
                        const uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane(
                            (int)(reinterpret_cast<const uint32_t*>(s.ends)[b * BPB / 32] >> (b * BPB % 32)));
                        const int info = (int)s.block[b * BPB + (lane & (BPB - 1))].y;
                        float4 val[U / 4];
#pragma unroll
                        for (int q = 0; q < U / 4; ++q)
                            val[q] = *reinterpret_cast<const float4*>(get_val + (b * U + 4 * q) * E);
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            constexpr int kSteps = BE / E;          // steps per block
                            const int blk = u / kSteps;
                            if (end & (1u << blk)) {                // the row's last block may hold absent entries: 0 * inf
                                const int32_t meta = lane_of(info, blk);
                                if ((u % kSteps) * E + e < (meta & 0xFF)) acc.fma((&val[u / 4].x)[u & 3], x[u]);
                                if ((u + 1) % kSteps == 0) flush(meta >> 8);
                            } else {
                                acc.fma((&val[u / 4].x)[u & 3], x[u]);
                            }
                        }
                        row_open = lane_of(info, BPB - 1) >> 8;
                        open = !(end & (1u << (BPB - 1))) && (b + 1) * BPB <= nblk;
                    }
                    if (open) flush(row_open);
                }
                if (lane == 0) s.head_row[wave] = head;
                __syncthreads();
                if (threadIdx.x < FB) {
#pragma unroll
                    for (int w = 0; w < kSweepWaves; ++w) {
                        const int32_t hr = s.head_row[w];
                        if (hr >= 0) s.rowsum[hr * FB + threadIdx.x] += s.head[w * FB + threadIdx.x];
                    }
                }
            }
            __syncthreads();
        }
        // the rows leave LDS
        s.first[threadIdx.x] = __float_as_int(a.norm != ES_NORM_NONE ? row_factor(a.norm, n, kept_count(a.mode, n, a.W)) : 1.0f);
        s.src[min((int)threadIdx.x, ROWS - 1)] = 0;
        __syncthreads();
        constexpr int RPP = kSweepThreads / G;
        for (int j = threadIdx.x / G; j < nrows; j += RPP) {
            const int ll = threadIdx.x & (G - 1);
            P out;
            out.v = *reinterpret_cast<const float4*>(&s.rowsum[j * FB + ll * 4]);
            if (a.norm != ES_NORM_NONE) out.scale(__int_as_float(s.first[j]));
            if (cols.ok[0]) out.store_streaming(a.Y + (r0 + j) * (int64_t)a.ldy + cols.off[0], cols.first[0]);
        }
        __syncthreads();
    }
}

}  // namespace

#endif  // ES_SPMM_SWEEP_KERNEL_H
