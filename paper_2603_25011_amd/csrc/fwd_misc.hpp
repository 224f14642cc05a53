// Mask compaction and packing plan (feed the fused forward), and the join of cut sequences.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fwd_mfma.hpp"

namespace lsr {

constexpr int PREP_THREADS = 256;

// One workgroup per sequence: len[b] = number of valid tokens, pos[b, 0..len) = their positions in
// ascending order.  The attention mask M of Sec. 2 may be arbitrary, so this is a stream
// compaction (ballot + popcount prefix), not a search for the first padding token.
__global__ __launch_bounds__(PREP_THREADS) void fwd_prep_kernel(const uint8_t* __restrict__ mask,
                                                                 int* __restrict__ len,
                                                                 int* __restrict__ pos, int S) {
    __shared__ int s_wave_total[PREP_THREADS / 64];
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const uint8_t* mrow = mask + (size_t)b * S;
    int* prow = pos + (size_t)b * S;
    int base = 0;
    for (int s0 = 0; s0 < S; s0 += PREP_THREADS) {
        const int s = s0 + tid;
        const bool flag = s < S && mrow[s] != 0;
        const unsigned long long bal = __ballot(flag);
        const int rank = __popcll(bal & ((1ull << lane) - 1ull));
        if (lane == 0) s_wave_total[wave] = __popcll(bal);
        __syncthreads();
        int before = 0, total = 0;
#pragma unroll
        for (int w = 0; w < PREP_THREADS / 64; ++w) {
            const int t = s_wave_total[w];
            before += w < wave ? t : 0;
            total += t;
        }
        if (flag) prow[base + before + rank] = s;
        base += total;
        __syncthreads();
    }
    if (tid == 0) len[b] = base;
}

// Packing plan for the MFMA forward.  Every sequence takes ceil(len / seg) segments of seg rows (one
// segment if it has no valid token, so that its zero output is still written; seg = 32, or 8 for batches
// of short sequences); seg0 is the exclusive prefix sum of the segment counts and seg0[B] the length of
// the segment list.  One workgroup; B is small next to the GEMM.
constexpr int PLAN_THREADS = 256;

__global__ __launch_bounds__(PLAN_THREADS) void fwd_plan_kernel(const int* __restrict__ len, int* __restrict__ blk0,
                                                                 int B, int seg) {
    __shared__ int s_scan[PLAN_THREADS];
    const int tid = threadIdx.x;
    int base = 0;
    for (int b0 = 0; b0 < B; b0 += PLAN_THREADS) {
        const int b = b0 + tid;
        int n = 0;
        if (b < B) {
            n = (len[b] + seg - 1) / seg;
            n = n > 0 ? n : 1;
        }
        s_scan[tid] = n;
        __syncthreads();
        for (int off = 1; off < PLAN_THREADS; off <<= 1) {
            const int add = tid >= off ? s_scan[tid - off] : 0;
            __syncthreads();
            s_scan[tid] += add;
            __syncthreads();
        }
        if (b < B) blk0[b] = base + s_scan[tid] - n;
        base += s_scan[PLAN_THREADS - 1];
        __syncthreads();
    }
    if (tid == 0) blk0[B] = base;
}

// Row table of the packed layout, one workgroup per sequence: packed row k of the sequence reads
// token pos[min(k, len-1)] (the tail of the last segment repeats the last valid token), and every
// segment records its sequence and whether it begins it, ends it, and whether the sequence is empty.
constexpr int FWD_ROWS_THREADS = 256;

__global__ __launch_bounds__(FWD_ROWS_THREADS) void fwd_rows_kernel(const int* __restrict__ len,
                                                                     const int* __restrict__ pos,
                                                                     const int* __restrict__ blk0,
                                                                     int2* __restrict__ rows,
                                                                     int* __restrict__ blk_meta, int S, int seg) {
    const int b = blockIdx.x;
    const int n = len[b];
    const int g0 = blk0[b];
    const int nblk = blk0[b + 1] - g0;
    const int* prow = pos + (size_t)b * S;
    for (int k = threadIdx.x; k < nblk * seg; k += FWD_ROWS_THREADS) {
        const int s = n > 0 ? prow[k < n ? k : n - 1] : 0;
        rows[(size_t)g0 * seg + k] = make_int2(b * S + s, s);
    }
    for (int k = threadIdx.x; k < nblk; k += FWD_ROWS_THREADS)
        blk_meta[g0 + k] = b | (k == nblk - 1 ? FWD_META_LAST : 0) | (n == 0 ? FWD_META_EMPTY : 0) |
                           (k == 0 ? FWD_META_FIRST : 0);
}

// The three passes above in one launch of one workgroup, for batches of few sequences and tokens, where three
// dependent launches cost more than the work in them: up to PACK_MAX_TOKENS mask entries and 64 sequences, or
// PACK_MAX_B of at most 64 tokens (packing as a profiled slot of its own, three launches -> one: B=100 S=40 13.8 -> 9.4 us,
// B=128 S=64 11.2 -> 10.3, and the forward 28.9 -> 25.2 at |V|=1000; not B=256 S=32 11.2 -> 15.3).  Wave w serves sequences w, w + 16, ...: it compacts the
// mask row (ballot + popcount) into LDS, and after the prefix sum of the block counts writes the
// row table and block records of the same sequences.  What bounds it is latency, so PACK_U mask entries per lane are in
// flight at a time, every wave forms the prefix sum for itself by shuffles (one barrier), and positions stay in LDS (against one
// entry in flight, a prefix sum of 1024 partials and positions through memory: B=32 S=256 9.0 -> 4.9 us, B=8 S=512 7.4 -> 4.8).
constexpr int PACK_THREADS = 1024;
constexpr int PACK_MAX_B = 128;
constexpr int PACK_MAX_TOKENS = 16384;
constexpr int PACK_U = 8;

__global__ __launch_bounds__(PACK_THREADS) void fwd_pack_kernel(const uint8_t* __restrict__ mask, int* __restrict__ blk0,
                                                                 int2* __restrict__ rows, int* __restrict__ blk_meta,
                                                                 int B, int S, int seg) {
    __shared__ int s_len[PACK_MAX_B];
    __shared__ uint16_t s_pos[PACK_MAX_TOKENS];      // [B][S] valid positions, ascending
    constexpr int NW = PACK_THREADS / 64;
    __shared__ int s_first[NW][PACK_MAX_B];          // first segment of each sequence, a copy per wave
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // 1. compaction
    if (S <= 64) {
        // PACK_U sequences at a time
        for (int b0 = wave; b0 < B; b0 += NW * PACK_U) {
            uint8_t m[PACK_U];
#pragma unroll
            for (int u = 0; u < PACK_U; ++u) {
                const int b = b0 + u * NW;
                m[u] = b < B && lane < S ? mask[b * S + lane] : (uint8_t)0;
            }
#pragma unroll
            for (int u = 0; u < PACK_U; ++u) {
                const int b = b0 + u * NW;
                const unsigned long long bal = __ballot(m[u] != 0);
                if (m[u] != 0) s_pos[b * S + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)lane;
                if (lane == 0 && b < B) s_len[b] = __popcll(bal);
            }
        }
    }
    // PACK_U entries per lane of a sequence at a time
    for (int b = S <= 64 ? B : wave; b < B; b += NW) {
        const uint8_t* mrow = mask + (size_t)b * S;
        uint16_t* prow = s_pos + b * S;
        int base = 0;
        for (int s0 = 0; s0 < S; s0 += 64 * PACK_U) {
            uint8_t m[PACK_U];
#pragma unroll
            for (int u = 0; u < PACK_U; ++u) {
                const int s = s0 + u * 64 + lane;
                m[u] = s < S ? mrow[s] : (uint8_t)0;
            }
#pragma unroll
            for (int u = 0; u < PACK_U; ++u) {
                const unsigned long long bal = __ballot(m[u] != 0);
                if (m[u] != 0) prow[base + __popcll(bal & ((1ull << lane) - 1ull))] = (uint16_t)(s0 + u * 64 + lane);
                base += __popcll(bal);
            }
        }
        if (lane == 0) s_len[b] = base;
    }
    __syncthreads();
    // 2. exclusive prefix sum of the block counts: lane l holds sequences 2 l and 2 l + 1
    constexpr int PER = PACK_MAX_B / 64;
    int nb[PER], sum = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int b = lane * PER + j;
        nb[j] = b < B ? max(1, (s_len[b] + seg - 1) / seg) : 0;
        sum += nb[j];
    }
    int incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(incl, off);
        incl += lane >= off ? up : 0;
    }
    int run = incl - sum;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        const int b = lane * PER + j;
        // every wave writes the same values, and reads its own
        if (b < B) s_first[wave][b] = run;
        if (wave == 0 && b < B) blk0[b] = run;
        run += nb[j];
        if (wave == 0 && b == B - 1) blk0[B] = run;
    }
    __builtin_amdgcn_wave_barrier();                 // LDS operations of one wave execute in program order
    // 3. row table and block records
    for (int b = wave; b < B; b += NW) {
        const int n = s_len[b];
        const int g0 = s_first[wave][b];
        const int nblk = max(1, (n + seg - 1) / seg);
        const uint16_t* prow = s_pos + b * S;
        for (int k = lane; k < nblk * seg; k += 64) {
            const int s = n > 0 ? (int)prow[k < n ? k : n - 1] : 0;
            rows[(size_t)g0 * seg + k] = make_int2(b * S + s, s);
        }
        for (int k = lane; k < nblk; k += 64)
            blk_meta[g0 + k] = b | (k == nblk - 1 ? FWD_META_LAST : 0) | (n == 0 ? FWD_META_EMPTY : 0) |
                               (k == 0 ? FWD_META_FIRST : 0);
    }
}

// Joins the pieces of the sequences that a chunk boundary of the fused kernel cuts (see fwd_mfma.hpp).
// The workgroups of chunk c leave, for a sequence that runs on into chunk c+1, the raw (max, position)
// of its blocks inside chunk c in Y and I; the workgroups of every later chunk k the sequence reaches
// leave theirs in slot k of part_m / part_s.  One thread per (chunk, vocabulary entry) takes the
// pieces in order (later pieces hold higher positions, so an equal maximum keeps the earlier
// position), applies bias, ReLU and log1p (F4) and overwrites Y and I with the final values.
// grid (ceil(V/256), fwd_merge_rows): a workgroup walks the chunks y, y + gridDim.y, ... (most end
// with a whole sequence and cost one table read).  tpc = most tiles per chunk, spt = segments per tile
// (ChunkSplit); blk0 and blk_meta are the segment tables.
constexpr int FWD_MERGE_THREADS = 256;
// Rows of the grid: each chunk is a chain of dependent reads, so narrow vocabularies spread the chunks over more workgroups (4 ->
// 32 rows: B=32 S=256 |V|=30522 9.1 -> 7.5 us, B=256 S=512 12.4 -> 9.3); with a thousand workgroups per row four are enough (B=64
// S=512 |V|=250002 38.8 -> 46.5).
inline int fwd_merge_rows(int vgroups, int n_chunks) {
    int rows = 4096 / vgroups;
    rows = rows < 4 ? 4 : (rows > 32 ? 32 : rows);
    return n_chunks < rows ? n_chunks : rows;
}

template <bool ARG>
__global__ __launch_bounds__(FWD_MERGE_THREADS) void fwd_merge_kernel(const int* __restrict__ blk0,
                                                                       const int* __restrict__ blk_meta,
                                                                       const float* __restrict__ part_m,
                                                                       const int* __restrict__ part_s,
                                                                       const float* __restrict__ bias,
                                                                       float* __restrict__ Y, int* __restrict__ I,
                                                                       int B, int V, int tpc, int spt) {
    const int n_blocks = blk0[B];
    const ChunkSplit cs = chunk_split(n_blocks, tpc, spt);
    const int v = blockIdx.x * FWD_MERGE_THREADS + threadIdx.x;
    for (int c = blockIdx.y; c < cs.nc; c += gridDim.y) {
        const int c_lo = cs.first_tile(c) * spt;
        const int c_hi = min(n_blocks, cs.first_tile(c + 1) * spt);        // first segment behind the chunk
        const int meta = blk_meta[c_hi - 1];
        if (meta & FWD_META_LAST) continue;                                // the chunk ends with a sequence
        const int b = meta & FWD_META_SEQ;
        if (blk0[b] < c_lo) continue;                                      // began in an earlier chunk: joined from there
        const int k_end = cs.chunk_of_tile((blk0[b + 1] - 1) / spt);       // chunk that holds the sequence's last segment
        if (v >= V) continue;
        const size_t o = (size_t)b * V + v;
        float m = Y[o];
        int s = ARG ? I[o] : 0;
        for (int k = c + 1; k <= k_end; ++k) {
            const float pm = part_m[(size_t)k * V + v];
            if (pm > m) {
                m = pm;
                if (ARG) s = part_s[(size_t)k * V + v];
            }
        }
        Y[o] = log1pf(fmaxf(m + bias[v], 0.f));
        if (ARG) I[o] = s;
    }
}

// Register-only matrix-core probe: every wave issues `iters` rounds of four independent
// 32x32x16 bf16 MFMAs on operands it never reloads, so the time is the matrix pipes' alone at
// whatever clock the part sustains under that load.  The result is folded into one value per lane
// that is compared with a number it cannot take, so nothing is stored; `sink` only keeps the
// arithmetic alive.  Measurement aid: the denominator "what the matrix cores deliver on this box"
// beside the nominal peak.
constexpr int PROBE_THREADS = 256;
constexpr int PROBE_MFMA_PER_ITER = 4;

__global__ __launch_bounds__(PROBE_THREADS) void mfma_probe_kernel(int iters, float* sink) {
    const int lane = threadIdx.x & 63;
    bf16x8 a, b;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        a[i] = (__bf16)(0.001f * (float)((lane + i) & 7));
        b[i] = (__bf16)(0.002f * (float)((lane * 3 + i) & 7));
    }
    floatx16 acc[PROBE_MFMA_PER_ITER];
#pragma unroll
    for (int k = 0; k < PROBE_MFMA_PER_ITER; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[k][r] = 0.f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int k = 0; k < PROBE_MFMA_PER_ITER; ++k)
            acc[k] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc[k], 0, 0, 0);
    }
    float sum = 0.f;
#pragma unroll
    for (int k = 0; k < PROBE_MFMA_PER_ITER; ++k)
#pragma unroll
        for (int r = 0; r < 16; ++r) sum += acc[k][r];
    if (sum == -1.2345e30f) *sink = sum;      // sums of non-negative products: never taken
}

}  // namespace lsr
