// Backward of the sparse-lexical head (paper Sec. 3 "Backward Pass", Alg. 3).
//
// Per (b,v) the gradient is g = dY * exp(-Y) where Y > 0 (derivative of log(1+ReLU(x)) written
// with the saved output), routed to one hidden state H[b, I[b,v]] and one embedding row W[v]:
//     dW[v,:]   = sum_b g[b,v] * H[b, I[b,v], :]
//     dH[b,s,:] = sum_{v : I[b,v] = s} g[b,v] * W[v,:]
//     db[v]     = sum_b g[b,v]
// The paper accumulates with atomics across blocks.  Here every output row has one owner that
// gathers its contributions in a fixed order (no global atomics, reproducible sums):
//   dW/db : the owner of row v walks b = 0..B-1 and gathers rows of H.
//   dH    : the (b,v) pairs with g != 0 are first bucketed by position s with a stable counting
//           sort (count -> scan -> place); the owner of row (b,s) then walks its bucket in
//           ascending v and gathers rows of W.  Empty buckets write zeros, so dH needs no memset.
// Rows are read as 16-byte chunks: one thread owns chunk c (+128, +256, ...) of the row and keeps
// fp32 accumulators for it.  All of this is bandwidth-bound row gathering; the arithmetic is plain
// fp32 FMA.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "lds_dma.hpp"

namespace lsr {

constexpr int ROW_THREADS = 128;     // threads that share one row (16 bytes each per pass)

__device__ __forceinline__ float gate_grad(float dy, float y) { return y > 0.f ? dy * expf(-y) : 0.f; }
__device__ __forceinline__ int clamp_pos(int s, int S) { return s < 0 ? 0 : (s >= S ? S - 1 : s); }

template <typename T> struct RowChunk;
template <> struct RowChunk<float> {
    static constexpr int N = 4;
    static __device__ __forceinline__ void fma(const uint4& x, float g, float* acc) {
        acc[0] = fmaf(g, __uint_as_float(x.x), acc[0]);
        acc[1] = fmaf(g, __uint_as_float(x.y), acc[1]);
        acc[2] = fmaf(g, __uint_as_float(x.z), acc[2]);
        acc[3] = fmaf(g, __uint_as_float(x.w), acc[3]);
    }
};
template <> struct RowChunk<uint16_t> {       // bfloat16 storage
    static constexpr int N = 8;
    static __device__ __forceinline__ void fma(const uint4& x, float g, float* acc) {
        const uint32_t w[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[2 * i] = fmaf(g, __uint_as_float(w[i] << 16), acc[2 * i]);
            acc[2 * i + 1] = fmaf(g, __uint_as_float(w[i] & 0xffff0000u), acc[2 * i + 1]);
        }
    }
};

// Gradient outputs are float32 or bfloat16 (OT = float or uint16_t): sums are always formed in float32
// and rounded once, to nearest even, when the final value is stored.
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float x) {
    const uint32_t u = __float_as_uint(x);
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;        // finite inputs
}
template <typename OT> struct OutVec;
template <> struct OutVec<float> {
    // four consecutive elements
    static __device__ __forceinline__ float4 load4(const float* p) { return *reinterpret_cast<const float4*>(p); }
    static __device__ __forceinline__ void store4(float* p, float4 x) { *reinterpret_cast<float4*>(p) = x; }
};
template <> struct OutVec<uint16_t> {
    static __device__ __forceinline__ float4 load4(const uint16_t* p) {
        const uint2 u = *reinterpret_cast<const uint2*>(p);
        return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u),
                           __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u));
    }
    static __device__ __forceinline__ void store4(uint16_t* p, float4 x) {
        *reinterpret_cast<uint2*>(p) = make_uint2(f32_to_bf16_bits(x.x) | (f32_to_bf16_bits(x.y) << 16),
                                                  f32_to_bf16_bits(x.z) | (f32_to_bf16_bits(x.w) << 16));
    }
};
// 1, 2, 4 or 8 consecutive elements
template <int K> __device__ __forceinline__ void load_n(const float* p, float (&x)[K]) {
    if constexpr (K == 1) x[0] = *p;
    else if constexpr (K == 2) { const float2 t = *reinterpret_cast<const float2*>(p); x[0] = t.x; x[1] = t.y; }
    else
#pragma unroll
        for (int i = 0; i < K; i += 4) { const float4 t = *reinterpret_cast<const float4*>(p + i); x[i] = t.x; x[i + 1] = t.y; x[i + 2] = t.z; x[i + 3] = t.w; }
}
template <int K> __device__ __forceinline__ void load_n(const uint16_t* p, float (&x)[K]) {
    static_assert(K % 2 == 0, "pairs");
    if constexpr (K == 2) {
        const uint32_t t = *reinterpret_cast<const uint32_t*>(p);
        x[0] = __uint_as_float(t << 16);
        x[1] = __uint_as_float(t & 0xffff0000u);
    } else
#pragma unroll
        for (int i = 0; i < K; i += 4) { const float4 t = OutVec<uint16_t>::load4(p + i); x[i] = t.x; x[i + 1] = t.y; x[i + 2] = t.z; x[i + 3] = t.w; }
}
template <int K, int M> __device__ __forceinline__ void store_n(float* p, const float (&x)[M]) {
    if constexpr (K == 1) *p = x[0];
    else if constexpr (K == 2) *reinterpret_cast<float2*>(p) = make_float2(x[0], x[1]);
    else
#pragma unroll
        for (int i = 0; i < K; i += 4) OutVec<float>::store4(p + i, make_float4(x[i], x[i + 1], x[i + 2], x[i + 3]));
}
template <int K, int M> __device__ __forceinline__ void store_n(uint16_t* p, const float (&x)[M]) {
    static_assert(K % 2 == 0, "pairs");
    if constexpr (K == 2) *reinterpret_cast<uint32_t*>(p) = f32_to_bf16_bits(x[0]) | (f32_to_bf16_bits(x[1]) << 16);
    else
#pragma unroll
        for (int i = 0; i < K; i += 4) OutVec<uint16_t>::store4(p + i, make_float4(x[i], x[i + 1], x[i + 2], x[i + 3]));
}
__device__ __forceinline__ float4 add4(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }

// ---------------------------------------------------------------------------------------------
// Stable bucketing of the non-zero (b,v) pairs by position s.
// The vocabulary is cut into n_seg segments of seg_len entries; (b, segment) is the unit of work.
// ---------------------------------------------------------------------------------------------

// Exclusive prefix sum over the 64 * NW threads of a workgroup: shuffles within each wave, then the sums of the waves in
// front; *total is the sum of all.  s_wave: NW ints, free again after the next barrier.  (One thread that walks 256
// partial sums in LDS takes 7 us: it waits for LDS at every step.)
template <int NW>
__device__ __forceinline__ int exclusive_scan(int x, int* s_wave, int* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl = x;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(incl, off);
        incl += lane >= off ? up : 0;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int t = s_wave[w];
        before += w < wave ? t : 0;
        all += t;
    }
    *total = all;
    return before + incl - x;
}

// Rank of a lane among the lanes of its wave with the same key, and how many there are: one ballot per key bit.
// The rank keeps the order of the lanes, so a bucket filled step by step ends up sorted by v (stable).
struct LaneGroup { int rank, size; };
__device__ __forceinline__ LaneGroup same_key_lanes(int key, bool active, int key_bits) {
    unsigned long long same = __ballot(active);
    for (int bit = 0; bit < key_bits; ++bit) {
        const bool one = (key >> bit) & 1;
        const unsigned long long bm = __ballot(active && one);
        same &= one ? bm : ~bm;
    }
    return {(int)__popcll(same & ((1ull << (threadIdx.x & 63)) - 1ull)), (int)__popcll(same)};
}

// cnt[b][seg][s] = number of v in the segment with g != 0 and I[b,v] = s.
// Four triples in flight per thread, and 1024 threads where segments are few, as long sequences have them: such a launch
// waits for memory alone (B=32 S=8192 |V|=30522 137 -> 9 us; B=64 S=512 |V|=250002, 256 threads, 50 -> 36).
constexpr int SORT_MAX_THREADS = 1024;
__global__ __launch_bounds__(SORT_MAX_THREADS) void bwd_count_kernel(const float* __restrict__ dY,
                                                                     const float* __restrict__ Y,
                                                                     const int* __restrict__ I,
                                                                     int* __restrict__ cnt,
                                                                     int S, int V, int n_seg, int seg_len) {
    extern __shared__ int s_hist[];
    const int seg = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, nt = blockDim.x;
    for (int s = tid; s < S; s += nt) s_hist[s] = 0;
    __syncthreads();
    const int vbeg = seg * seg_len;
    const int vend = vbeg + min(V - vbeg, seg_len);
    const size_t row = (size_t)b * V;
    for (int v0 = vbeg + tid; v0 < vend; v0 += 4 * nt) {
        float dy[4], y[4];
        int ix[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int v = v0 + u * nt;
            const bool ok = v < vend;
            dy[u] = ok ? dY[row + v] : 0.f;
            y[u] = ok ? Y[row + v] : 0.f;
            ix[u] = ok ? I[row + v] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (gate_grad(dy[u], y[u]) != 0.f) atomicAdd(&s_hist[clamp_pos(ix[u], S)], 1);
    }
    __syncthreads();
    int* out = cnt + ((size_t)b * n_seg + seg) * S;
    for (int s = tid; s < S; s += nt) out[s] = s_hist[s];
}

// Per b: cnt[b][seg][s] becomes the number of earlier-segment entries of bucket s, and
// bstart[b][0..S] the exclusive prefix of the bucket sizes (bstart[b][S] = non-zero pairs of row b).
// A thread owns one bucket of every NT: its loads and stores are coalesced, and the prefix over the buckets goes
// NT at a time (B=2 S=16 4.5 -> 2.5 us, B=64 S=512 with 64 segments 15 -> 10; 1024 threads against 256: B=16 S=600 13.6 and 25, B=32
// S=8192 14.8 and 29, B=256 S=512 7.2 and 8.4).  Beside a dW kernel that fills the chip the launch waits for room whatever NT is:
// at B=32 S=8192 it takes 242 us there and ends when dW does, where the serial prefix took 122 behind a count that had waited 137
// (count, scan and placement together 489 before, 316 now).
template <int NT>
__global__ __launch_bounds__(NT) void bwd_scan_kernel(int* __restrict__ cnt, int* __restrict__ bstart,
                                                      int S, int n_seg) {
    __shared__ int s_wave[2][NT / 64];
    const int b = blockIdx.x, tid = threadIdx.x;
    int* out = bstart + (size_t)b * (S + 1);
    int base = 0;
    for (int s0 = 0, it = 0; s0 < S; s0 += NT, ++it) {
        const int s = s0 + tid;
        int run = 0;
        // eight segments at a time: the loads of a batch are all issued before the first store,
        // which the compiler cannot do by itself (loads and stores go to the same array)
        for (int seg0 = 0; s < S && seg0 < n_seg; seg0 += 8) {
            int c[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                c[u] = seg0 + u < n_seg ? cnt[((size_t)b * n_seg + seg0 + u) * S + s] : 0;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (seg0 + u < n_seg) cnt[((size_t)b * n_seg + seg0 + u) * S + s] = run;
                run += c[u];
            }
        }
        int total;
        const int before = exclusive_scan<NT / 64>(run, s_wave[it & 1], &total);
        if (s < S) out[s] = base + before;
        base += total;
    }
    if (tid == 0) out[S] = base;
}

// Placement: PLACE_WAVES waves per (b, segment), each with a consecutive piece of the segment.  A wave first counts its
// pairs per bucket (LDS atomics); the counts of the waves in front of it and of the segments in front then give it a slot
// of its own in every bucket, and it walks its piece in ascending v, 64 at a time, without looking at the other waves.
// Lanes holding the same position find each other by ballots (same_key_lanes), so every bucket ends up sorted by v
// and the later sums have a fixed order.  What bounds it are the ballots and dependent LDS accesses of each step, so steps must not
// wait for one another (waves that took turns behind a barrier per 64 pairs: with LDS staging B=2 S=16 |V|=1000 8.4 ->
// 5.0 us, B=13 S=197 |V|=31091 11.8 -> 8.8, B=256 S=512 |V|=30522 66 -> 53, B=64 S=512 |V|=250002 145 -> 119;
// without, from one wave per workgroup, B=32 S=8192 |V|=30522 221 -> 62, B=64 S=8192 |V|=250002 598 -> 474, but with one gradient
// in twenty 418 -> 437, B=64 S=4096 218 -> 241, where the count and the scan in front gain more).
// Beside dW a shorter sort lets the two gathers run together for longer, and some shapes pay for that.  Whole backward, 196 shapes
// of S > 1024: geometric mean 0.86, 13 above 1.02, the worst B=100 S=1025 D=128 |V|=26630 with one in twenty 105 -> 119 and B=200
// S=3000 D=768 |V|=15000 612 -> 671; 193 shapes of 128 <= S <= 512: 0.99, 12 above 1.02, the worst B=200 S=128 D=768
// |V|=26630 815 -> 875.  Fewer waves per segment leave that as it is (one 0.97, 21; two 0.89, 17), a dW that starts behind the scan or
// behind the placement makes it worse (0.86, 38 and 0.90, 61; 128 <= S <= 512 1.05, 119 and 1.09, 134).
constexpr int PLACE_WAVES = 4;

// Long sequences: every pair is stored straight to its bucket.   dynamic LDS: PLACE_WAVES * S ints
__global__ __launch_bounds__(64 * PLACE_WAVES) void bwd_place_kernel(const float* __restrict__ dY,
                                                                     const float* __restrict__ Y,
                                                                     const int* __restrict__ I,
                                                                     const int* __restrict__ cnt,
                                                                     const int* __restrict__ bstart,
                                                                     uint2* __restrict__ perm,
                                                                     int S, int V, int n_seg, int seg_len, int key_bits) {
    extern __shared__ int s_place[];        // [PLACE_WAVES][S] counts, then the next free slot of each bucket
    const int seg = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    int* const s_off = s_place + wave * S;
    const int* c0 = cnt + ((size_t)b * n_seg + seg) * S;
    const int* b0 = bstart + (size_t)b * (S + 1);
    for (int s = tid; s < PLACE_WAVES * S; s += 64 * PLACE_WAVES) s_place[s] = 0;
    __syncthreads();
    const int piece = (seg_len / 64 + PLACE_WAVES - 1) / PLACE_WAVES * 64;       // (seg_len is a multiple of 64)
    const int vseg = seg * seg_len, n = min(V - vseg, seg_len);
    const int vbeg = vseg + min(n, wave * piece), vend = vseg + min(n, (wave + 1) * piece);
    const size_t row = (size_t)b * V;
    float dy[4], y[4];
    int ix[4];
    auto request = [&](int base) {          // four steps of 64
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int v = base + u * 64 + lane;
            const bool ok = v < vend;
            dy[u] = ok ? dY[row + v] : 0.f;
            y[u] = ok ? Y[row + v] : 0.f;
            ix[u] = ok ? I[row + v] : 0;
        }
    };
    for (int base = vbeg; base < vend; base += 256) {
        request(base);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (gate_grad(dy[u], y[u]) != 0.f) atomicAdd(&s_off[clamp_pos(ix[u], S)], 1);
    }
    request(vbeg);
    __syncthreads();
    for (int s = tid; s < S; s += 64 * PLACE_WAVES) {
        int at = b0[s] + c0[s];
#pragma unroll
        for (int w = 0; w < PLACE_WAVES; ++w) {
            const int c = s_place[w * S + s];
            s_place[w * S + s] = at;
            at += c;
        }
    }
    __syncthreads();
    for (int base = vbeg; base < vend; base += 256) {
        float g[4];
        int key[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            g[u] = gate_grad(dy[u], y[u]);      // 0 for lanes past the end (dy = 0, y = 0)
            key[u] = clamp_pos(ix[u], S);
        }
        // the next four steps are requested before the current ones are ranked
        request(base + 256);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const bool active = g[u] != 0.f;
            const LaneGroup lg = same_key_lanes(key[u], active, key_bits);
            int dest = 0;
            if (active) {
                dest = s_off[key[u]] + lg.rank;
                perm[row + dest] = make_uint2((unsigned)(base + u * 64 + lane), __float_as_uint(g[u]));      // one 8-byte scattered store
            }
            // LDS instructions of one wave execute in program order for all lanes, so the read of s_off above precedes
            // this update and the update precedes the next step's read.  wave_barrier only pins that order for the compiler.
            __builtin_amdgcn_wave_barrier();
            if (active && lg.rank == lg.size - 1) s_off[key[u]] = dest + 1;
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// Placement through LDS (S <= PLACE_MAX_S, segments of at most PLACE_MAX_SEG entries).
// ONE: the sequence is one segment; then this is the whole sort, and the bucket starts are written here.  (A sequence that fits one segment
// always is one: backward B=23 S=88 D=256 |V|=2000 with one gradient in twenty 30.7 -> 19.7 us with dW in the same launch, B=4 S=640 D=64
// |V|=3500 float32 23.3 -> 21.1, B=245 S=48 D=128 |V|=3500 102.8 -> 102.9; none of 35 backwards of 1024 to 4096 entries slower.  dH alone: see NW; many sequences beside dW: see backward_impl.)
// The kernel above stores every (v, g) pair straight to its bucket: the 64 stores of a step go to some
// fifty buckets, and with thousands of (b, segment) waves in flight every bucket's line leaves L2
// between two stores to it (measured at C5: 0.48 GB written for 0.13 GB of pairs).  Here a workgroup
// first sorts its whole segment by bucket in LDS and then writes it out in sorted order:
// the pairs a bucket receives from this segment (about a dozen at C5) leave as one contiguous run.
//   1. every wave loads its piece of the segment, keeps (g, bucket) in registers and counts per bucket;
//   2. exclusive prefix over buckets and waves = first local slot of each (bucket, wave); delta = first global
//      slot of the bucket - its first local slot;
//   3. steps of 64 pairs per wave: ballot ranking, staging;
//   4. local slot k goes to global slot k + s_delta[bucket of k].
// A staged pair is (v - vbeg) | bucket << 12 and g.   dynamic LDS: NW / 2 * S ints + seg_len pairs.
// NW: waves per segment.  PLACE_WAVES, and PLACE_ONE_WAVES where a sequence is one segment and dW has launches of its own: a single workgroup has the whole
// sequence then, whose steps follow one another (dH alone, us, segments of 512 entries in three launches -> one of four waves -> of eight: B=1 S=163 D=256
// |V|=3856 20.1 -> 23.9 -> 17.9, one in twenty B=102 S=175 D=256 |V|=4016 20.0 -> 25.2 -> 18.6, B=62 S=4 D=1024 |V|=1032 19.3 -> 14.0 -> 13.4; 80 shapes of 1025
// to 4096 entries 0.92 with four, the worst 1.26, 0.77 with eight, the worst 0.93).
// STEPS: steps of 64 per wave, at least seg_len / (64 * NW); steps behind the end of a piece are left out.
// Counts and slots of two waves share an int (a segment has at most 4096), and the deltas take their place once all is
// staged, because the LDS decides how many workgroups a CU holds.  Against an int per wave, deltas of their own and every
// step taken: B=64 S=512 |V|=250002 158 -> 119 us, B=256 S=1024 |V|=33700 98 -> 72 and, with one gradient in twenty, 86 -> 53
// (nine steps of 16), B=64 S=128 |V|=135000 59 -> 49; 56 -> 43, B=2 S=16 |V|=1000 7.4 -> 7.5 for the barrier more.
// ---------------------------------------------------------------------------------------------
constexpr int PLACE_MAX_S = 1024;
constexpr int PLACE_MAX_SEG = 4096;
constexpr int PLACE_ONE_WAVES = 8;

template <int STEPS, int NW, bool ONE>
__device__ __forceinline__ void place_staged(const float* __restrict__ dY, const float* __restrict__ Y, const int* __restrict__ I,
                                             const int* __restrict__ cnt, int* bstart, uint2* __restrict__ perm,
                                             int S, int V, int n_seg, int seg_len, int key_bits, int seg, int b) {
    constexpr int NT = 64 * NW;
    extern __shared__ __attribute__((aligned(16))) int s_place[];
    uint2* s_stage = reinterpret_cast<uint2*>(s_place);             // [seg_len]
    unsigned* s_cnt = reinterpret_cast<unsigned*>(s_place + 2 * seg_len);      // [NW / 2][S]: counts of waves 2 i and 2 i + 1
    int* s_delta = s_place + 2 * seg_len;                           // [S] global slot - local slot, in the same place at the end
    __shared__ int s_wave[NW];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = wave & 1;
    unsigned* const s_count = s_cnt + (wave >> 1) * S;
    uint16_t* const s_next = reinterpret_cast<uint16_t*>(s_count) + half;      // next free local slot of bucket s at [2 s]
    const int* c0 = cnt + ((size_t)b * n_seg + seg) * S;
    int* const b0 = bstart + (size_t)b * (S + 1);

    // 1. this wave's piece
    const int piece = (seg_len / 64 + NW - 1) / NW * 64;       // (seg_len is a multiple of 64)
    const int vseg = seg * seg_len, n = min(V - vseg, seg_len);
    const int vbeg = vseg + min(n, wave * piece), vend = vseg + min(n, (wave + 1) * piece);
    const size_t row = (size_t)b * V;
    float g[STEPS];
    int key[STEPS];
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
        const int v = vbeg + i * 64 + lane;
        const bool ok = v < vend;
        const float dy = ok ? dY[row + v] : 0.f;
        const float y = ok ? Y[row + v] : 0.f;
        key[i] = ok ? clamp_pos(I[row + v], S) : 0;
        g[i] = gate_grad(dy, y);                // 0 for lanes past the end (dy = 0, y = 0)
    }
    for (int s = tid; s < NW / 2 * S; s += NT) s_cnt[s] = 0;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < STEPS; ++i)
        if (g[i] != 0.f) atomicAdd(&s_count[key[i]], 1u << (16 * half));
    __syncthreads();

    // 2. slots
    const int per = (S + NT - 1) / NT;
    const int lo = min(S, tid * per), hi = min(S, lo + per);
    int sum = 0;
    for (int s = lo; s < hi; ++s)
#pragma unroll
        for (int w = 0; w < NW / 2; ++w) {
            const unsigned c = s_cnt[w * S + s];
            sum += (int)((c & 0xffffu) + (c >> 16));
        }
    int total;
    int run = exclusive_scan<NW>(sum, s_wave, &total);
    int delta[PLACE_MAX_S / NT];
#pragma unroll
    for (int u = 0; u < PLACE_MAX_S / NT; ++u) {
        const int s = lo + u;
        if (s < hi) {
            if (ONE) b0[s] = run;
            delta[u] = ONE ? 0 : b0[s] + c0[s] - run;
#pragma unroll
            for (int w = 0; w < NW / 2; ++w) {
                const unsigned c = s_cnt[w * S + s];
                const int next = run + (int)(c & 0xffffu);
                s_cnt[w * S + s] = (unsigned)run | (unsigned)next << 16;
                run = next + (int)(c >> 16);
            }
        }
    }
    if (ONE && tid == 0) b0[S] = total;
    __syncthreads();

    // 3. rank and stage
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
        if (vbeg + i * 64 >= vend) continue;     // the same for the whole wave
        const bool active = g[i] != 0.f;
        const LaneGroup lg = same_key_lanes(key[i], active, key_bits);
        int slot = 0;
        if (active) {
            slot = s_next[2 * key[i]] + lg.rank;
            s_stage[slot] = make_uint2((unsigned)(vbeg - vseg + i * 64 + lane) | ((unsigned)key[i] << 12), __float_as_uint(g[i]));
        }
        __builtin_amdgcn_wave_barrier();         // LDS operations of one wave execute in program order
        if (active && lg.rank == lg.size - 1) s_next[2 * key[i]] = (uint16_t)(slot + 1);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();

    // 4. sorted write-out
#pragma unroll
    for (int u = 0; u < PLACE_MAX_S / NT; ++u)
        if (lo + u < hi) s_delta[lo + u] = delta[u];
    __syncthreads();
    for (int k = tid; k < total; k += NT) {
        const uint2 e = s_stage[k];
        perm[row + k + s_delta[e.x >> 12]] = make_uint2((unsigned)vseg + (e.x & 4095u), e.y);
    }
}
template <int STEPS, int NW, bool ONE>
__global__ __launch_bounds__(64 * NW) void bwd_place_staged_kernel(const float* __restrict__ dY,
                                                               const float* __restrict__ Y,
                                                               const int* __restrict__ I,
                                                               const int* __restrict__ cnt,
                                                               int* bstart,
                                                               uint2* __restrict__ perm,
                                                               int S, int V, int n_seg, int seg_len, int key_bits) {
    place_staged<STEPS, NW, ONE>(dY, Y, I, cnt, bstart, perm, S, V, n_seg, seg_len, key_bits, blockIdx.x, blockIdx.y);
}

// ---------------------------------------------------------------------------------------------
// dH, whole rows (D not a multiple of 64, see sliced_gathers in lsr_head.hip).
// dH[b,s,:] = sum over the bucket of (b,s), in ascending v, of g * W[v,:].   grid (B, S): b fastest,
// so that the empty buckets behind the ends of the sequences are spread evenly over the chip
// ---------------------------------------------------------------------------------------------
// accumulate: the sums are added to what dH holds
template <typename T, int CPT, typename OT>
__global__ __launch_bounds__(ROW_THREADS) void bwd_dh_kernel(const T* __restrict__ W,
                                                             const int* __restrict__ bstart,
                                                             const uint2* __restrict__ perm,
                                                             OT* __restrict__ dH,
                                                             int S, int D, int V, int accumulate) {
    constexpr int N = RowChunk<T>::N;
    __shared__ int s_v[ROW_THREADS];
    __shared__ float s_g[ROW_THREADS];
    const int b = blockIdx.x, s = blockIdx.y, tid = threadIdx.x;
    const int n_chunks = D / N;
    const int beg = bstart[(size_t)b * (S + 1) + s];
    const int end = bstart[(size_t)b * (S + 1) + s + 1];
    const size_t prow = (size_t)b * V;
    float acc[CPT][N];
#pragma unroll
    for (int cp = 0; cp < CPT; ++cp)
#pragma unroll
        for (int i = 0; i < N; ++i) acc[cp][i] = 0.f;

    for (int base = beg; base < end; base += ROW_THREADS) {
        const int n = min(ROW_THREADS, end - base);
        const uint2 ent = perm[prow + base + min(tid, n - 1)];      // padding: the last row of the list, weight 0
        s_v[tid] = (int)ent.x;
        s_g[tid] = tid < n ? __uint_as_float(ent.y) : 0.f;
        __syncthreads();
        for (int k = 0; k < n; k += 4) {
            uint4 x[4][CPT];
            float g[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                g[u] = s_g[k + u];
                const T* src = W + (size_t)s_v[k + u] * D;
#pragma unroll
                for (int cp = 0; cp < CPT; ++cp) {
                    const int c = tid + cp * ROW_THREADS;
                    x[u][cp] = c < n_chunks ? *reinterpret_cast<const uint4*>(src + c * N) : make_uint4(0, 0, 0, 0);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int cp = 0; cp < CPT; ++cp) RowChunk<T>::fma(x[u][cp], g[u], acc[cp]);
        }
        __syncthreads();
    }
    OT* out = dH + ((size_t)b * S + s) * D;
#pragma unroll
    for (int cp = 0; cp < CPT; ++cp) {
        const int c = tid + cp * ROW_THREADS;
        if (c < n_chunks) {
#pragma unroll
            for (int i = 0; i < N; i += 4) {
                float4 r = make_float4(acc[cp][i], acc[cp][i + 1], acc[cp][i + 2], acc[cp][i + 3]);
                if (accumulate) r = add4(OutVec<OT>::load4(out + c * N + i), r);
                OutVec<OT>::store4(out + c * N + i, r);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// dW/db, whole rows (D not a multiple of 64 or large batches, see plan_backward).
// dW[v,:] = sum_b g[b,v] * H[b, I[b,v], :],  db[v] = sum_b g[b,v].
// A workgroup owns VT consecutive vocabulary rows.  It first stages g and I for all B x VT pairs in
// LDS (coalesced along v), then walks the rows one by one, skipping pairs with g = 0.
// dynamic LDS: B*VT floats + B*VT ints.
// ---------------------------------------------------------------------------------------------
// accumulate: the sums are added to what dW and db hold
template <typename T, int CPT, typename OT>
__global__ __launch_bounds__(ROW_THREADS) void bwd_dw_kernel(const T* __restrict__ H,
                                                             const float* __restrict__ dY,
                                                             const float* __restrict__ Y,
                                                             const int* __restrict__ I,
                                                             OT* __restrict__ dW, float* __restrict__ db,
                                                             int B, int S, int D, int V, int VT, int accumulate) {
    constexpr int N = RowChunk<T>::N;
    extern __shared__ int s_dyn[];
    float* s_g = reinterpret_cast<float*>(s_dyn);          // [B][VT]
    int* s_i = s_dyn + (size_t)B * VT;                     // [B][VT]
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int v0 = blockIdx.x * VT;
    const int n_chunks = D / N;

    for (int e = tid; e < B * VT; e += ROW_THREADS) {
        const int bb = e / VT, vv = e - bb * VT;
        const int v = v0 + vv;
        float g = 0.f;
        int idx = 0;
        if (v < V) {
            const size_t o = (size_t)bb * V + v;
            g = gate_grad(dY[o], Y[o]);
            idx = clamp_pos(I[o], S);
        }
        s_g[e] = g;
        s_i[e] = idx;
    }
    __syncthreads();

    for (int vv = 0; vv < VT; ++vv) {
        const int v = v0 + vv;
        if (v >= V) break;
        float acc[CPT][N];
#pragma unroll
        for (int cp = 0; cp < CPT; ++cp)
#pragma unroll
            for (int i = 0; i < N; ++i) acc[cp][i] = 0.f;
        float gsum = 0.f;
        for (int bb0 = 0; bb0 < B; bb0 += 64) {
            const int bl = bb0 + lane;
            const float gl = bl < B ? s_g[bl * VT + vv] : 0.f;
            gsum += gl;
            unsigned long long nz = dW ? __ballot(gl != 0.f) : 0ull;       // same in both waves
            int bb = 0;
            while (nz) {
                uint4 x[4][CPT];
                float g[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    // take the next non-zero pair, or repeat the last one (a row that is used anyway) with weight 0
                    const bool have = nz != 0;
                    bb = have ? bb0 + __builtin_ctzll(nz) : bb;
                    nz &= nz - 1;
                    g[u] = have ? s_g[bb * VT + vv] : 0.f;
                    const T* src = H + ((size_t)bb * S + s_i[bb * VT + vv]) * D;
#pragma unroll
                    for (int cp = 0; cp < CPT; ++cp) {
                        const int c = tid + cp * ROW_THREADS;
                        x[u][cp] = c < n_chunks ? *reinterpret_cast<const uint4*>(src + c * N) : make_uint4(0, 0, 0, 0);
                    }
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int cp = 0; cp < CPT; ++cp) RowChunk<T>::fma(x[u][cp], g[u], acc[cp]);
            }
        }
        OT* out = dW + (size_t)v * D;
        if (dW) {
#pragma unroll
            for (int cp = 0; cp < CPT; ++cp) {
                const int c = tid + cp * ROW_THREADS;
                if (c < n_chunks) {
#pragma unroll
                    for (int i = 0; i < N; i += 4) {
                        float4 r = make_float4(acc[cp][i], acc[cp][i + 1], acc[cp][i + 2], acc[cp][i + 3]);
                        if (accumulate) r = add4(OutVec<OT>::load4(out + c * N + i), r);
                        OutVec<OT>::store4(out + c * N + i, r);
                    }
                }
            }
        }
        if (db && tid < 64) {                                    // fixed-order butterfly over b
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) gsum += __shfl_xor(gsum, o);
            if (tid == 0) db[v] = accumulate ? db[v] + gsum : gsum;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// dW/db, column-sliced variant.
// The gathers of the kernel above hit rows of H scattered over all of H (tens of MB), so they are
// served by the memory-side cache at a fraction of the L2 rate.  Here the work is cut into slices of
// 64 hidden-state columns and the grid is ordered slice-major: the workgroups resident at any time
// all gather from the same [tokens x 64] slice of H (a few MB at most), which stays in every XCD's
// L2 (the host sizes a group of NDC consecutive slices to at most 9 MiB of H and a workgroup walks the
// slices of its group, so that the (g, I) staging is not repeated more often than needed).
// A row piece is 64 elements = LPR lanes x 16 bytes; a wave therefore serves 64/LPR vocabulary
// rows at once, walks the sequences that have a gradient for them with eight gathers in flight per
// lane, and writes one 64-column piece of each dW row.  Summation order over b is fixed.
// (No LDS beside the tile: sixteen bytes for a count of the pairs cost B=250 S=60 D=1024 one of five workgroups per CU,
// dW 4114 -> 4525 us.)
// A tile is compacted after staging where few enough of its pairs have a gradient: each column of the (g, I)
// tile in place to its non-zero entries, in ascending b (one wave per column, ballot ranking), closed by a
// zero, so that sparse gradients cost what they hold; the sums are the same either way (same terms, same order).
// dW us, without / with compaction, by the share of pairs that have a gradient:
//   16-row tiles (below 31/32)       1.0             0.98            0.95            0.85            0.55            0.25
//     B=256 S=32 D=768 |V|=30522     1058 / 1063     1053 / 1043     1052 / 1017     1054 / 937      1038 / 662      989 / 368
//     B=384 S=32 D=768 |V|=30522     2055 / 2089     2080 / 2072     2051 / 2012     2063 / 1818     2055 / 1262     1932 / 683
//     B=250 S=64 D=1000 |V|=30000    1489 / 1534     1483 / 1490     1475 / 1459     1451 / 1339     1415 / 970      1350 / 564
//   wider tiles (below one half)     0.95            0.85            0.7             0.55            0.4             0.25
//     B=64 S=100 D=768 |V|=50000     282 / 305       281 / 293       295 / 272       274 / 226       266 / 189       258 / 147
//     B=167 S=62 D=648 |V|=66407     1005 / 1104     982 / 1033      958 / 901       931 / 758       911 / 612       881 / 453
//     B=100 S=40 D=768 |V|=50000     434 / 460       425 / 422       417 / 369       414 / 317       401 / 261       388 / 187
// SWZ (16-row tiles, of which a workgroup of a large batch compacts many narrow columns): element (b, vv) sits at
// word b*VT + (vv ^ (b % VT)), so that the compaction's column reads spread over the LDS banks (B=250 S=60 D=1024
// |V|=100000, one in twenty, 747 -> 717 us).  On wider tiles the address arithmetic costs more than the bank
// conflicts (about 1 us per workgroup), and a word of padding per row costs a workgroup per CU.   VT a power of two.
// When the H slice of the whole batch (B*S rows x 128 bytes) is larger than L2, the host launches
// the kernel once per chunk of consecutive sequences (b_first, B = sequences of the chunk); later
// launches add to dW and db, which keeps the order of the sums fixed.
// Where the partial sums come from and where the result goes is set per launch: `prev` (float32, may
// be null) is added to the sums of this launch, `add_dst` adds what dst already holds (accumulation into
// the caller's gradient), and dst is float32 or bfloat16 (OT).  A float32 result spread over several
// launches passes prev = dst; a bfloat16 result keeps its partial sums in a float32 staging array (dst of
// all launches but the last, prev of all but the first), so that it is rounded once.
// dynamic LDS: B*VT floats + B*VT ints.   256 threads, grid = (ceil(V/VT), ceil(ceil(D/64)/NDC)).
// ---------------------------------------------------------------------------------------------
constexpr int DWS_COLS = 64;
constexpr int DH_NLD = 4;                 // gathers in flight per lane of the sliced dH gather
// threads per workgroup: one bucket if WPB > 1 waves share it, else four waves of BPW buckets each
constexpr int dh_threads(int wpb) { return wpb > 1 ? 64 * wpb : 256; }
constexpr int PERM_SLACK = 256;           // entries the workspace keeps behind the sorted lists (see bwd_dh_sliced_kernel)

// column slices of a row (D a multiple of 8: the last one may be partly filled)
__host__ __device__ constexpr int n_slices(int D) { return (D + DWS_COLS - 1) / DWS_COLS; }

// Slices owned by XCDs.  Workgroup ids go round-robin over the chip's 8 XCDs (id & 7), each with an L2
// of its own.  With n_dc = 8 q + r column slices, XCD x owns slices x, x + 8, ..., x + 8 (q - 1): every
// gather from one of them goes through the same L2, which then holds one copy of the slice's window
// instead of each of the eight L2s fetching its own, and sees all of the window's reuse.  The r slices
// left over are shared: each is dealt out over all XCDs by item (item i goes to XCD i & 7).
// An item is what the kernel iterates within a slice (a group of buckets).  A workgroup of the owned part
// walks up to `walk` of its XCD's slices for one item; of the shared part, one slice.
// Index j = id >> 3 of the workgroup on its XCD: first the owned part, ceil(q / walk) * n_items
// workgroups, item fastest; then the shared part, r * ceil(n_items / 8).  The grid is 8 times the sum;
// ids that fall behind the end of the shared part are not valid.
struct XcdSliceUnit { bool valid, first_of_item; int item, dc_first, dc_step, dc_count; };
__host__ __device__ inline long long xcd_slice_grid(int n_dc, int n_items, int walk) {
    const int q = n_dc >> 3, r = n_dc & 7;
    return 8ll * ((long long)((q + walk - 1) / walk) * n_items + (long long)r * ((n_items + 7) >> 3));
}
__host__ __device__ inline XcdSliceUnit xcd_slice_unit(unsigned id, int n_dc, int n_items, int walk) {
    XcdSliceUnit u;
    const int x = id & 7, j = (int)(id >> 3);
    const int q = n_dc >> 3, r = n_dc & 7;
    const int owned = ((q + walk - 1) / walk) * n_items;
    if (j < owned) {
        const int wg = j / n_items;                         // group of `walk` owned slices
        u.item = j - wg * n_items;
        u.dc_first = wg * walk * 8 + x;
        u.dc_step = 8;
        u.dc_count = (q < (wg + 1) * walk ? q : (wg + 1) * walk) - wg * walk;
        u.first_of_item = x == 0 && wg == 0;
        u.valid = true;
    } else {
        const int per = (n_items + 7) >> 3;
        const int jj = j - owned;
        const int l = jj / per;
        u.item = (jj - l * per) * 8 + x;
        u.dc_first = 8 * q + l;
        u.dc_step = 1;
        u.dc_count = 1;
        u.first_of_item = q == 0 && l == 0;
        u.valid = l < r && u.item < n_items;
    }
    return u;
}

template <typename T, bool SWZ, typename OT>
__device__ __forceinline__ void dw_sliced(const T* __restrict__ H, const float* __restrict__ dY, const float* __restrict__ Y,
                                          const int* __restrict__ I, const float* prev, OT* dW, int add_dst,
                                          float* __restrict__ db, int add_db, int b_first, int B, int S, int D, int V, int VT, int NDC,
                                          int vtile, int dg) {
    // b_first, B: the sequences of this launch; prev / add_dst: see above; add_db: db already holds the
    // sums over the sequences before b_first (or the caller's accumulated gradient) and is added to
    constexpr int N = RowChunk<T>::N;          // elements per 16-byte chunk
    constexpr int LPR = DWS_COLS / N;          // lanes per row piece
    constexpr int VPG = 64 / LPR;              // vocabulary rows a wave serves at once
    extern __shared__ __attribute__((aligned(16))) int s_dyn[];
    float* s_g = reinterpret_cast<float*>(s_dyn);          // [B][VT]
    int* s_i = s_dyn + (size_t)B * VT;                     // [B][VT]  token row b*S + I[b,v]
    auto at = [VT](int b, int vv) { return b * VT + (SWZ ? vv ^ (b & (VT - 1)) : vv); };
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int n_waves = blockDim.x >> 6;
    const int v0 = vtile * VT;
    const int dc_begin = dg * NDC;
    const int dc_end = min(n_slices(D), dc_begin + NDC);

    // staging, four independent (dY, Y, I) triples in flight per thread
    for (int e0 = tid; e0 < B * VT; e0 += 4 * blockDim.x) {
        float dy[4], y[4];
        int ix[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * blockDim.x;
            const int bb = e / VT, vv = e - bb * VT;
            const bool ok = e < B * VT && v0 + vv < V;
            const size_t o = ok ? (size_t)(b_first + bb) * V + v0 + vv : 0;
            dy[u] = ok ? dY[o] : 0.f;
            y[u] = ok ? Y[o] : 0.f;
            ix[u] = ok ? I[o] : 0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * blockDim.x;
            if (e < B * VT) {
                const int bb = e / VT, vv = e - bb * VT;
                s_g[at(bb, vv)] = gate_grad(dy[u], y[u]);
                s_i[at(bb, vv)] = (b_first + bb) * S + clamp_pos(ix[u], S);
            }
        }
    }
    __syncthreads();
    // how many of 1024 pairs spread over the tile have a gradient (the same for all waves)
    int nz = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float4 q = reinterpret_cast<const float4*>(s_g)[((j * 64 + lane) * (B * VT / 4)) >> 8];
        nz += __popcll(__ballot(q.x != 0.f)) + __popcll(__ballot(q.y != 0.f)) + __popcll(__ballot(q.z != 0.f)) + __popcll(__ballot(q.w != 0.f));
    }
    const bool compact = nz < (SWZ ? 992 : 512);

    // db: every wave sums the columns that it compacts below (so it has read them before), 256 / VT lanes per
    // column, each every (256 / VT)-th sequence, in float64, rounded once per launch.  Against float64, in units of the norm of
    // db, a float32 loop over B = 13 / 64 / 256 sequences is off by 7.0e-8 / 1.5e-7 / 2.9e-7, the 64-lane butterfly of the
    // whole-row kernel by 5.2e-8 / 6.7e-8 / 7.8e-8, this by 2.5e-8, and by 4.0e-8 / 7.4e-8 where four / sixteen launches each
    // round the db they hand on.
    if (db && dg == 0) {
        const int cols = VT / n_waves;
        const int part = lane / cols;
        const int vv = wave + n_waves * (lane - part * cols);
        double sum = 0.0;
        for (int k = part; k < B; k += 64 / cols) sum += (double)s_g[at(k, vv)];
        for (int off = cols; off < 64; off <<= 1) sum += __shfl_xor(sum, off);
        if (part == 0 && v0 + vv < V) db[v0 + vv] = (float)(add_db ? (double)db[v0 + vv] + sum : sum);
    }

    // compaction: column vv keeps its non-zero entries, in ascending b, at rows 0..n-1, and a zero at
    // row n if n < B.  A chunk of 64 rows is read before any of it is written and lands at or below
    // where it was read, so this works in place.
    const unsigned long long lt = (1ull << lane) - 1ull;
    for (int vv = wave; compact && vv < VT; vv += n_waves) {
        int n = 0;
        for (int b0 = 0; b0 < B; b0 += 64) {
            const int b = b0 + lane;
            const float g = b < B ? s_g[at(b, vv)] : 0.f;
            const int r = b < B ? s_i[at(b, vv)] : 0;
            const unsigned long long nz = __ballot(g != 0.f);
            if (g != 0.f) {
                const int k = n + __popcll(nz & lt);
                s_g[at(k, vv)] = g;
                s_i[at(k, vv)] = r;
            }
            n += __popcll(nz);
        }
        if (lane == 0 && n < B) s_g[at(n, vv)] = 0.f;
    }
    if (compact) __syncthreads();
    if (!dW) return;

    for (int dc = dc_begin; dc < dc_end; ++dc) {
        const int col = dc * DWS_COLS + (lane % LPR) * N;
        const int col0 = col < D ? col : 0;                    // behind D: gathers column 0, stores nothing
        for (int grp = wave; grp * VPG < VT; grp += n_waves) {
            const int vv = grp * VPG + lane / LPR;
            const int v = v0 + vv;
            float acc[N];
#pragma unroll
            for (int i = 0; i < N; ++i) acc[i] = 0.f;
            auto gather = [&](auto compacted) {
                constexpr bool C = decltype(compacted)::value;
                for (int k0 = 0; k0 < B; k0 += 8) {
                    float g[8];
                    uint4 x[8];
                    bool open = true;                            // false behind the closing zero of a compacted column
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        const int k = k0 + u;
                        g[u] = (open && k < B) ? s_g[at(k, vv)] : 0.f;
                        if (C) open = g[u] != 0.f;
                        x[u] = make_uint4(0, 0, 0, 0);
                        if (g[u] != 0.f) x[u] = *reinterpret_cast<const uint4*>(H + (size_t)s_i[at(k, vv)] * D + col0);
                    }
#pragma unroll
                    for (int u = 0; u < 8; ++u) RowChunk<T>::fma(x[u], g[u], acc);
                    if (C && !open) break;
                }
            };
            if (compact) gather(std::true_type{});
            else gather(std::false_type{});
            if (v < V && col < D) {
                const size_t o = (size_t)v * D + col0;
#pragma unroll
                for (int i = 0; i < N; i += 4) {
                    float4 r = make_float4(acc[i], acc[i + 1], acc[i + 2], acc[i + 3]);
                    if (prev) r = add4(*reinterpret_cast<const float4*>(prev + o + i), r);
                    if (add_dst) r = add4(OutVec<OT>::load4(dW + o + i), r);
                    OutVec<OT>::store4(dW + o + i, r);
                }
            }
        }
    }
}

template <typename T, bool SWZ, typename OT>
__global__ __launch_bounds__(256) void bwd_dw_sliced_kernel(const T* __restrict__ H,
                                                            const float* __restrict__ dY,
                                                            const float* __restrict__ Y,
                                                            const int* __restrict__ I,
                                                            const float* prev, OT* dW, int add_dst,
                                                            float* __restrict__ db, int add_db,
                                                            int b_first, int B, int S, int D, int V, int VT, int NDC) {
    // slice-group-major order
    dw_sliced<T, SWZ, OT>(H, dY, Y, I, prev, dW, add_dst, db, add_db, b_first, B, S, D, V, VT, NDC, blockIdx.x, blockIdx.y);
}

// The placement and dW/db in one launch, neither of which needs the other: the first B * n_seg workgroups place a segment each, the
// others are those of bwd_dw_sliced_kernel.  Small problems are bound by the launches they wait for one after the other (count, scan, placement,
// dW, dH; the first two go where a sequence is one segment).  B=2 S=16 D=64 |V|=1000 float32, forward and backward, 27.7 -> 17.5 us; backward
// B=7 S=495 D=64 |V|=1100 24.2 -> 14.0, B=1 S=10 D=1024 |V|=1500 float32 67.9 -> 56.9, B=54 S=181 D=256 |V|=1100 91.5 -> 80.2.
// When: see share_dw in lsr_head.hip.
template <typename T, typename OT, int STEPS, bool ONE>
__global__ __launch_bounds__(256) void bwd_place_dw_kernel(const T* __restrict__ H, const float* __restrict__ dY,
                                                           const float* __restrict__ Y, const int* __restrict__ I,
                                                           const int* __restrict__ cnt, int* bstart,
                                                           uint2* __restrict__ perm, OT* dW, float* __restrict__ db, int accumulate,
                                                           int B, int S, int D, int V, int n_seg, int seg_len, int key_bits, int VT, int NDC,
                                                           int n_vtiles) {
    static_assert(64 * PLACE_WAVES == 256, "one workgroup size");
    const int i = (int)blockIdx.x - B * n_seg;
    if (i < 0) {
        const int b = (int)blockIdx.x / n_seg;
        place_staged<STEPS, PLACE_WAVES, ONE>(dY, Y, I, cnt, bstart, perm, S, V, n_seg, seg_len, key_bits, (int)blockIdx.x - b * n_seg, b);
    } else {
        dw_sliced<T, false, OT>(H, dY, Y, I, nullptr, dW, accumulate, db, accumulate, 0, B, S, D, V, VT, NDC, i % n_vtiles, i / n_vtiles);
    }
}

// ---------------------------------------------------------------------------------------------
// dH, column-sliced variant.
// One sub-group of a wave owns one bucket and one 64-column slice; the grid is ordered slice-major.
// A 64-column piece of a row is LPR lanes x 16 bytes, so a sub-group of G = 64/BPW lanes gathers
// G/LPR bucket entries per load, keeps four loads in flight per lane, and folds the per-entry
// partial sums with a fixed butterfly at the end (reproducible order).
//
// What decides the speed is whether the rows of W being gathered come from L2.  All buckets walk the
// vocabulary in ascending v but not in step, so the working set of one slice pass is the whole slice
// of W: |V| x 128 bytes.  Up to about 4 MB that lives in L2; beyond, the vocabulary is cut into n_vc
// chunks and the pass is launched once per chunk (`vc` = chunk index), each launch gathering only
// the entries of its chunk.  `bounds` then holds, per bucket, the n_vc+1 positions in the sorted
// entry list where the chunks begin (bwd_chunk_bounds_kernel); with n_vc = 1 it is the bucket start
// table itself.  Chunk 0 writes dH (zeros for empty buckets), later chunks add to it: one owner per
// element and launch, launches in stream order, so the sum keeps a fixed order.
// As in the dW gather, `prev` (float32, may be null) is added to the sums of this launch, `add_dst` adds
// what dst already holds, dst is float32 or bfloat16; `write_all` makes every bucket write (the launch
// that produces the final value of a fresh result), otherwise only buckets with entries in this chunk do.
// grid = (B, ceil(S / (4*BPW)), ceil(D/64)), 256 threads, or (B, S, ceil(D/64)), 64 * WPB threads, where the WPB waves of
// a workgroup share one bucket; xcd_slice_grid workgroups instead of either where XCDs own the slices.
// ---------------------------------------------------------------------------------------------
// tops[b], if asked for: positions of sequence b up to the last one that has entries (what bwd_dw_tile_kernel copies).
__global__ __launch_bounds__(256) void bwd_chunk_bounds_kernel(const int* __restrict__ bstart,
                                                               const uint2* __restrict__ perm,
                                                               int* __restrict__ bounds, int* __restrict__ tops,
                                                               int n_buckets, int S, int V, int n_vc, int vc_len) {
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (long long)n_buckets * (n_vc + 1)) return;
    const int bucket = (int)(idx / (n_vc + 1));
    const int c = (int)(idx - (long long)bucket * (n_vc + 1));
    const int b = bucket / S, s = bucket - b * S;
    int lo = bstart[(size_t)b * (S + 1) + s];
    int hi = bstart[(size_t)b * (S + 1) + s + 1];
    if (c == n_vc) {
        // the last bucket of the sequence that has entries; the first bucket, if none has
        const int all = bstart[(size_t)b * (S + 1) + S];
        if (tops && hi == all && (lo < hi || (s == 0 && all == 0))) tops[b] = lo < hi ? s + 1 : 0;
        lo = hi;
    }
    const unsigned target = (unsigned)c * (unsigned)vc_len;     // first v of chunk c
    const uint2* list = perm + (size_t)b * V;
    while (lo < hi) {                                           // first entry with v >= target
        const int mid = lo + ((hi - lo) >> 1);
        if (list[mid].x < target) lo = mid + 1; else hi = mid;
    }
    bounds[idx] = lo;
}

// x of the lane 8 places away in the row of 16, added to the lane's own (DPP: no LDS crossbar)
__device__ __forceinline__ float add_half_row(float x) {
    return x + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), 0x128, 0xf, 0xf, true));      // row_ror:8
}
// Sums over two neighbouring rows of 16 lanes (two halves of the wave) of a and b: the even rows (lower half) keep a's, the
// odd rows (upper half) b's.
__device__ __forceinline__ float fold_rows(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float fold_halves(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// dc, sg, b: column slice, workgroup within the sequence (its bucket, if several waves share one) and sequence
template <typename T, int BPW, int WPB, typename OT, bool OFF32>
__device__ __forceinline__ void dh_sliced(const T* __restrict__ W, const int* __restrict__ bounds, const uint2* __restrict__ perm,
                                          const float* prev_sum, OT* dH, int add_dst, int write_all, int S, int D, int V,
                                          int n_vc, int vc, int dc, int sg, int b) {
    constexpr int N = RowChunk<T>::N;
    constexpr int LPR = DWS_COLS / N;          // lanes per row piece
    constexpr int G = 64 / BPW;                // lanes per bucket
    constexpr int EPG = G / LPR;               // entries of one bucket gathered per load
    static_assert(EPG >= 1, "a bucket needs at least one row piece worth of lanes");
    constexpr int NLD = DH_NLD;                // gathers in flight per lane (8: more registers, fewer
                                               // waves; C5 2.83 -> 3.71 ms)
    static_assert(G <= PERM_SLACK, "entries read behind the end of a list stay inside the slack");
    static_assert(WPB == 1 || BPW == 1, "either several buckets per wave or several waves per bucket");
    constexpr int BLK = G * WPB;               // entries between a wave's consecutive blocks
    constexpr int E = WPB > 1 ? 1 : 4;         // blocks of entries requested at a time
    constexpr int NV = N >> ((G >= 32) + (G >= 64));      // columns of a sum that a lane ends up with
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int col0 = dc * DWS_COLS + (lane % LPR) * N;
    const bool col_ok = col0 < D;              // the last slice may be partly filled: the lanes behind D gather column 0
    const int li = lane % G;                   // lane within its bucket
    const int sub = li / LPR;
    // the columns this lane writes (see the folds at the end): NV of its N
    const int vcol = (G >= 32 && (lane & 16) ? N / 2 : 0) + (G >= 64 && (lane & 32) ? NV : 0);
    const bool w_lane = col_ok && (LPR == 8 && G >= 16 ? (lane & 8) == 0 : true) && (WPB == 1 || wave == 0);
    const char* const Wb = reinterpret_cast<const char*>(W);
    const uint2* const pl = perm + (size_t)b * V;                   // b: the same for the whole workgroup
    const uint32_t row_bytes = (uint32_t)D * (uint32_t)sizeof(T);
    const uint32_t col_bytes = (uint32_t)(col_ok ? col0 : 0) * (uint32_t)sizeof(T);
    const int src0 = (lane - li + sub) * 4;    // bpermute address of the lane holding entry `sub` of the block

    const int s = WPB > 1 ? sg : (sg * 4 + wave) * BPW + lane / G;
    const bool live = s < S;
    const int bq = live ? b * S + s : 0;
    const size_t bi = n_vc == 1 ? (size_t)b * (S + 1) + s : (size_t)bq * (n_vc + 1) + vc;
    const int beg = live ? bounds[bi] : 0;
    const int end = live ? bounds[bi + 1] : 0;
    if (!write_all && !__any(beg < end)) return;      // nothing of this chunk in any bucket of the wave (WPB > 1: of the workgroup)
    // A shared bucket of at most one block of entries is the first wave's alone: the others leave at once, and nobody
    // waits at the barrier below (all waves of the workgroup see the same list).
    const bool alone = WPB > 1 && end - beg <= G;
    if (alone && wave > 0) return;
    const bool writer = w_lane && live && (write_all || beg < end);
    const size_t o = (size_t)bq * D + col0 + vcol;
    float acc[N];
#pragma unroll
    for (int i = 0; i < N; ++i) acc[i] = 0.f;
    float prev[NV];                            // the sum of the earlier chunks, requested early
#pragma unroll
    for (int i = 0; i < NV; ++i) prev[i] = 0.f;
    if (writer) {
        if (prev_sum) load_n<NV>(prev_sum + o, prev);
        if (add_dst) {
            float old[NV];
            load_n<NV>(dH + o, old);
#pragma unroll
            for (int i = 0; i < NV; ++i) prev[i] += old[i];
        }
    }
    // What limits this loop is the number of vector-memory instructions a CU can issue and the time their data
    // takes, so the (v, g) entries are not fetched per gather slot.  The G lanes of a bucket load G consecutive entries
    // with one coalesced instruction, a block that feeds RPB rounds of NLD gathers per lane, and E blocks are
    // requested at a time: loads return in order, so every gather behind an entry load waits until the entry has come from
    // beyond L2 (a block at a time, requested a block ahead: C5 2348 -> 2228 us, B=256 S=512 |V|=30522 778 -> 733).  Waves that
    // share a bucket take a block at a time, the next one in flight (four: B=32 S=128 D=1024 156 -> 159, B=2 S=16 D=64 |V|=1000
    // forward and backward 27.5 -> 29.3).
    // The lane that loads an entry settles what it stands for, once: the byte offset of its row (32 bits where W allows it)
    // and its gradient, or, behind the end of the list, a zero gradient and the row of the block's first entry (a row
    // the bucket uses anyway, so nothing that could be non-finite is multiplied by that zero; the entry
    // read there belongs to a later bucket, to the next sequence, or to the PERM_SLACK entries the workspace
    // keeps behind the last list, and is not looked at).  A lane takes the entry of its slot from the lane that loaded
    // it (ds_bpermute, which goes through the LDS crossbar, not the memory path).  With that, and the folds below
    // instead of bpermute butterflies, C5 2392 -> 2348, B=64 S=100 |V|=50000 with one gradient in twenty 93 -> 85.
    constexpr int RPB = G / (NLD * EPG);       // rounds per block of entries
    static_assert(RPB * NLD * EPG == G && RPB >= 1, "a block is a whole number of rounds");
    int left = end - beg - (WPB > 1 ? wave * G : 0);                // entries from the block's start to the end of the list
    const uint2* pe = pl + beg + li + (WPB > 1 && left > 0 ? wave * G : 0);      // this lane's entry of the current block
    uint2 ahead = make_uint2(0u, 0u);
    if (WPB > 1) ahead = *pe;
    for (; left > 0; left -= E * BLK) {
        uint2 entries[E];
        if constexpr (WPB > 1) {
            entries[0] = ahead;
            pe += left > BLK ? BLK : 0;        // only a block that exists is requested (BLK entries may be more than the slack)
            ahead = *pe;
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (e == 0 || e * BLK < left) entries[e] = pe[e * BLK];
            pe += E * BLK;
        }
        __builtin_amdgcn_sched_barrier(0);                          // all of them are requested first
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int rest = left - e * BLK;                        // entries from this block's start
            if (e > 0 && rest <= 0) break;
            const uint2 ent = entries[e];
            const uint32_t v_first = G == 64 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)ent.x)      // the block's first entry: inside the list
                                             : (uint32_t)__builtin_amdgcn_ds_bpermute((lane - li) * 4, (int)ent.x);
            const bool inside = li < rest;
            const uint32_t v = inside ? ent.x : v_first;
            const int at = (int)(OFF32 ? __umul24(v, row_bytes) : v);
            const int gv = inside ? (int)ent.y : 0;
#pragma unroll
            for (int p = 0; p < RPB; ++p) {
                if (p * NLD * EPG < rest) {                         // the round has entries; the lanes of a bucket agree
                    // three phases, kept apart: the entries of all NLD slots, then all NLD gathers, then the FMAs
                    // (left to itself the compiler gathers two rows at a time)
                    uint32_t off[NLD];
                    float gq[NLD];
                    uint4 x[NLD];
#pragma unroll
                    for (int u = 0; u < NLD; ++u) {
                        const int from = src0 + (p * NLD * EPG + u * EPG) * 4;      // block offset of the slot of sub-group 0
                        off[u] = (uint32_t)__builtin_amdgcn_ds_bpermute(from, at);
                        gq[u] = __int_as_float(__builtin_amdgcn_ds_bpermute(from, gv));
                        if (OFF32) off[u] += col_bytes;
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < NLD; ++u) {
                        if constexpr (OFF32) x[u] = *reinterpret_cast<const uint4*>(Wb + off[u]);
                        else x[u] = *reinterpret_cast<const uint4*>(Wb + ((size_t)off[u] * row_bytes + col_bytes));
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int u = 0; u < NLD; ++u) RowChunk<T>::fma(x[u], gq[u], acc);
                }
            }
        }
    }
    // The sub-groups' sums: every fold halves the columns a lane holds (NV are left), in a fixed order.
    if (__any(beg < end)) {
        if (LPR == 8 && G >= 16) {
#pragma unroll
            for (int i = 0; i < N; ++i) acc[i] = add_half_row(acc[i]);
        }
        if (G >= 32) {
#pragma unroll
            for (int i = 0; i < N / 2; ++i) acc[i] = fold_rows(acc[i], acc[i + N / 2]);
        }
        if (G >= 64) {
#pragma unroll
            for (int i = 0; i < N / 4; ++i) acc[i] = fold_halves(acc[i], acc[i + N / 4]);
        }
    }
    if (WPB > 1 && !alone) {
        // the waves' sums, added in wave order (the exits above leave all waves of a bucket or the first one)
        __shared__ __attribute__((aligned(16))) float s_sum[WPB][DWS_COLS];
        if ((LPR == 16 || (lane & 8) == 0) && wave > 0) {
#pragma unroll
            for (int i = 0; i < NV; ++i) s_sum[wave][(lane % LPR) * N + vcol + i] = acc[i];
        }
        __syncthreads();
        if (!writer) return;
#pragma unroll
        for (int w = 1; w < WPB; ++w)
#pragma unroll
            for (int i = 0; i < NV; ++i) acc[i] += s_sum[w][(lane % LPR) * N + vcol + i];
    }
    if (writer) {
#pragma unroll
        for (int i = 0; i < NV; ++i) acc[i] = prev[i] + acc[i];
        store_n<NV>(dH + o, acc);
    }
}

template <typename T, int BPW, int WPB, typename OT, bool OFF32>
__global__ __launch_bounds__(dh_threads(WPB)) __attribute__((amdgpu_waves_per_eu(8, 8))) void bwd_dh_sliced_kernel(const T* __restrict__ W,
                                                            const int* __restrict__ bounds,
                                                            const uint2* __restrict__ perm,
                                                            const float* prev_sum, OT* dH, int add_dst, int write_all,
                                                            int B, int S, int D, int V, int n_groups,
                                                            int n_vc, int vc, int xcd_own) {
    // Within a slice, consecutive workgroups take the same positions of consecutive sequences
    // (b fastest).  Workgroups are dealt to the chip's shader engines in a fixed rotation; with s
    // fastest, the empty buckets behind the end of each sequence recur with a period that can leave
    // some engines with twice the work of others.
    int dc = blockIdx.z, sg = blockIdx.y, b = blockIdx.x;          // slice-major order
    if (xcd_own) {                                                 // slices owned by XCDs (see xcd_slice_unit)
        const XcdSliceUnit u = xcd_slice_unit(blockIdx.x, n_slices(D), n_groups, 1);
        if (!u.valid) return;
        dc = u.dc_first;
        sg = u.item / B;
        b = u.item - sg * B;
    }
    dh_sliced<T, BPW, WPB, OT, OFF32>(W, bounds, perm, prev_sum, dH, add_dst, write_all, S, D, V, n_vc, vc, dc, sg, b);
}

// dW/db and the (first) dH gather in one launch: the dW workgroups first, which run longer, and the dH gather fills the chip beside them.
// The overlap is that of the auxiliary stream without its fork and join (32 us of the host's time, and waits on the GPU): whole
// training step through autograd, bound by the host, B=14 S=38 D=512 |V|=29935 198 -> 138 us; backward B=5 S=34 D=384 |V|=22757 56 -> 34.
// All workgroups of the launch carry the LDS of a dW tile, hence the limit on it.  When, and both sides: see share_dw in lsr_head.hip.
struct DhDwArgs {
    const void* H;
    const void* W;
    const float* dY;
    const float* Y;
    const int* I;
    const int* bounds;
    const uint2* perm;
    void* dH;
    void* dW;
    float* db;
    int accumulate;
    int B, S, D, V;
    int n_groups, n_vc, xcd_own;             // dH: as above
    int VT, NDC, n_vtiles, n_dw, n_dw_pad;   // dW: as above; its workgroups, and the same as a multiple of 8
};
// (Workgroups of four waves only: dW wants four, and its db sums are the same as in a launch of its own.)
template <typename T, int BPW, int WPB, typename OT>
__global__ __launch_bounds__(dh_threads(WPB)) __attribute__((amdgpu_waves_per_eu(8, 8))) void bwd_dh_dw_kernel(DhDwArgs p) {
    static_assert(dh_threads(WPB) == 256, "workgroups of four waves");
    int id = blockIdx.x;
    if (id < p.n_dw_pad) {
        if (id >= p.n_dw) return;
        const int dg = id / p.n_vtiles;
        dw_sliced<T, false, OT>(static_cast<const T*>(p.H), p.dY, p.Y, p.I, nullptr, static_cast<OT*>(p.dW), p.accumulate, p.db, p.accumulate, 0, p.B,
                                p.S, p.D, p.V, p.VT, p.NDC, id - dg * p.n_vtiles, dg);
        return;
    }
    id -= p.n_dw_pad;
    int dc, sg, b;
    if (p.xcd_own) {
        const XcdSliceUnit u = xcd_slice_unit(id, n_slices(p.D), p.n_groups, 1);
        if (!u.valid) return;
        dc = u.dc_first;
        sg = u.item / p.B;
        b = u.item - sg * p.B;
    } else {
        const int q = id / p.B, per = p.n_groups / p.B;
        b = id - q * p.B;
        dc = q / per;
        sg = q - dc * per;
    }
    OT* const dH = static_cast<OT*>(p.dH);
    dh_sliced<T, BPW, WPB, OT, true>(static_cast<const T*>(p.W), p.bounds, p.perm, nullptr, dH, p.accumulate, !p.accumulate, p.S, p.D, p.V, p.n_vc, 0, dc,
                                     sg, b);
}

// ---------------------------------------------------------------------------------------------
// dW/db, LDS-tile variant (bfloat16 inputs, D a multiple of 64, DWT_MIN_S <= S <= DWT_MAX_S).
// A workgroup of 1024 threads owns 1024 consecutive vocabulary rows and one 64-column slice and walks
// the sequences b = 0 .. B-1 in order.  For each sequence the slice of its hidden states (up to S x 128
// bytes, at most 64 KiB; see `tops` below) is copied into LDS and every gather of the sequence is an LDS read.  The four lanes
// of a quad stage one vocabulary row each and sum all four, a quarter of the columns each (two chunks of 16 bytes, 64
// float accumulators per thread): a row's (g, tile row) goes from the staging lane to the others as an operand modifier (DPP)
// of the xor that forms the LDS address and of one move, so it needs neither LDS nor registers of its own.  A
// sequence costs one tile copy for 1024 gathers: the traffic out of L2 is the tile (S x 128 bytes)
// instead of the gathers (1024 x 128 bytes), the reads are coalesced, and what is left is the arithmetic
// of the gather itself, one unpack and one FMA per element, with the LDS reads one row ahead of it (the last row of a
// sequence is multiplied behind the barrier, while the first of the next is on its way).
// A half of a tile row is 64 bytes: rows with bit 1 set hold their halves exchanged, so that the four rows that sixteen lanes
// read spread over all banks where they differ modulo 4, which positions do in one case of eleven.  What is left of the conflicts costs little (dW, us,
// positions as they come; made to differ; all equal modulo 4: B=64 S=512 D=1024 |V|=250002 1714; 1707; 1723, B=16 S=256 |V|=250002 350; 346; 358, B=32
// S=128 D=1024 92.0; 91.6; 93.4, B=256 S=512 |V|=30522 894 each).
// What bounds a round (one sequence): the arithmetic, 1.25 us, or the copy, 0.9 + 0.17 per 16 KiB (36 bytes per clock and CU: the 32
// CUs of an XCD read the same lines).  So only the rows up to the last one with a gradient are copied where a launch in front has
// left their number (`tops`; it does where dW runs behind dH): B=64 S=512 D=1024 |V|=250002, lengths 128..512, backward 3947 ->
// 3806 us, one gradient in twenty 2582 -> 2344.  Eight lanes per row with the pairs in LDS took dW 1736 -> 1714 there,
// B=16 S=256 |V|=250002 352 -> 344, B=32 S=128 D=1024 93.5 -> 90.
// The sixteen waves take four fifths of a CU's registers, so waves of dH or of the sort would find room beside them.  Where dH takes several
// windows that helps (backward, against a kernel that takes all registers: B=64 S=128 D=512 |V|=60000 442 -> 407 us, one gradient in twenty 212 ->
// 185, B=16 S=256 |V|=250002 940 -> 927).  Where it has one, which it gathers all at once, it slows the gather of dW's first rounds down, which is worth it
// only if dH would otherwise have to wait for the end.  Workgroups that do not come out at full rounds of 256 CUs leave CUs to dH in the last one, so there the
// workgroup keeps its CU to itself: ALONE (128 registers by name: sixteen waves of them are all a CU has).  Backward, us, beside -> ALONE: 1.27
// rounds, B=200 S=128 |V|=26630, 910 -> 779, 1.41, B=128 S=256 |V|=30522, 728 -> 638, 1.06, B=171 S=151 D=1024 |V|=16875, 689 -> 548; 70 shapes
// 0.96 in the mean, 11 above 1.03, the worst B=88 S=485 D=2048 |V|=24738 (3.1, one in twenty) 786 -> 856.  Full rounds: one, B=200 S=128 D=512
// |V|=32000, 581 -> 627, one in twenty B=9 S=374 D=2048 |V|=7285 53 -> 59, two, B=4 S=438 D=1024 |V|=31989, 81 -> 90; 50
// shapes of one round 1.04 in the mean, 45 of two and three 1.03.
// Not kept: (dY, Y, I) two sequences ahead (1701; 354), L2 touched two sequences ahead (1790; 372), the rows counted here
// by ballots and LDS (1762; 410), 12 waves (2059; 441), two workgroups of 8 waves (-; 340, beside dH 923 -> 961 for the backward).
// The next sequence's tile travels global -> LDS directly (LDS-DMA, no staging registers) into the other
// buffer while the current one is multiplied; its (dY, Y, I) travel through registers and are turned into
// (g, tile row offset) pairs at the end of the round.  One barrier per sequence, behind a full vmcnt wait.
// Pairs without gradient point at a row of zeros behind the tile (hidden states of padded positions are
// never multiplied, whatever they hold), and a wave skips a row of its quads when none of the sixteen has a gradient.  The order of the sums over b is the same as in the kernels above.
// Not for sparse gradients (the cost hardly falls with the number of non-zero pairs, as it does in the
// compacting kernel above) or for few workgroups: the host takes it for shapes with at least one
// workgroup per CU.
// grid = ceil(V / 1024) * (D / 64), slice-major.  PASSES = ceil(S / 128) copy passes per tile.
// ---------------------------------------------------------------------------------------------
constexpr int DWT_ROWS = 1024;
constexpr int DWT_MAX_S = 512;
constexpr int DWT_MIN_S = 128;

// Value that lane K of a lane's quad holds (DPP).  All four lanes have to be active.
template <int K> __device__ __forceinline__ uint32_t quad_lane(uint32_t x) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, K * 0x55, 0xf, 0xf, true);       // quad_perm:[K, K, K, K]
}

template <typename OT, int PASSES, bool ALONE>
__global__ __launch_bounds__(DWT_ROWS) void bwd_dw_tile_kernel(const uint16_t* __restrict__ H,
                                                               const float* __restrict__ dY,
                                                               const float* __restrict__ Y,
                                                               const int* __restrict__ I,
                                                               OT* dW, int add_dst, float* db, int add_db,
                                                               const int* __restrict__ tops, int B, int S, int D, int V, int n_vtiles) {
    constexpr int ROW_B = DWS_COLS * 2;                    // bytes per tile row
    constexpr int RPT = 4;                                 // vocabulary rows per thread: those its quad of lanes stages
    constexpr int RPP = DWT_ROWS / 8;                      // tile rows per copy pass
    constexpr int TROWS = PASSES * RPP;                    // tile rows: S <= TROWS
    constexpr uint32_t TILE_B = (TROWS + 1) * ROW_B;       // two tiles, each followed by a row of zeros
    if (ALONE) asm volatile("" ::: "v127");                // 128 registers: sixteen waves take all of a CU's
    __shared__ __attribute__((aligned(1024))) uint8_t s_tile[2 * TILE_B];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int dc = blockIdx.x / n_vtiles;
    const int v0 = (blockIdx.x - dc * n_vtiles) * DWT_ROWS;
    const int vs = v0 + tid;                               // the row this thread stages
    const bool vs_ok = vs < V;
    const int vs_c = vs_ok ? vs : V - 1;

    float acc[RPT][16];
#pragma unroll
    for (int k = 0; k < RPT; ++k)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[k][i] = 0.f;
    const bool sum_db = db && dc == 0;
    double db_acc = (sum_db && add_db && vs_ok) ? (double)db[vs] : 0.0;      // rounded once, as in the kernel above

    // The loads of a sequence are straight-line code (clamped addresses instead of predicates) and nothing
    // looks at their results before stage(), so that they stay in flight while the sequence before is
    // multiplied.  Byte offsets within a sequence's hidden states (S * D * 2 bytes is far below 4 GiB) and
    // within a row of dY / Y / I are kept in 32 bits; the sequence's base is wave-uniform.
    float dy_r, y_r;
    int ix_r;
    const uint32_t voff = (uint32_t)vs_c * 4u;
    auto gload = [&](int b) {
        const size_t ro = (size_t)b * V * 4;
        dy_r = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(dY) + ro + voff);
        y_r = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(Y) + ro + voff);
        ix_r = *reinterpret_cast<const int*>(reinterpret_cast<const char*>(I) + ro + voff);
    };
    // the eight tile rows a wave copies per pass land in 1024 contiguous LDS bytes, lane l at + 16 l, so the lane picks
    // the chunk that belongs there (rows r with bit 1 set hold their two halves exchanged); rows
    // behind S - 1 (when S is not a multiple of 8) receive copies of row S - 1 and are never read
    uint32_t hoff[PASSES];
#pragma unroll
    for (int p = 0; p < PASSES; ++p)
        hoff[p] = (uint32_t)((min(p * RPP + (tid >> 3), S - 1) * D + dc * DWS_COLS + ((lane & 7) ^ ((lane >> 4 & 1) * 4)) * 8) * 2);
    const uint32_t tile0 = __builtin_amdgcn_readfirstlane(lds_addr(&s_tile[0]));
    auto tile_load = [&](int b, int buf, int rows) {
        const char* hb = reinterpret_cast<const char*>(H) + (size_t)b * S * D * 2;
        const uint32_t dst = tile0 + buf * TILE_B + (uint32_t)wave * 8u * ROW_B;
#pragma unroll
        for (int p = 0; p < PASSES; ++p)
            if (p * RPP + wave * 8 < rows) dma16_to_lds(hb, hoff[p], dst + p * RPP * ROW_B);
    };
    // what this lane's row of the vocabulary takes from a sequence: g, and the byte offset of its tile row
    struct Pair { float g; uint32_t off; };
    auto stage = [&](int buf, bool count) {
        const float g = vs_ok ? gate_grad(dy_r, y_r) : 0.f;
        if (sum_db) db_acc += count ? (double)g : 0.0;
        const uint32_t r = (uint32_t)(g != 0.f ? clamp_pos(ix_r, S) : TROWS);
        return Pair{g, buf * TILE_B + r * ROW_B + (r >> 1 & 1) * 64};
    };
    if (tid < 16) *reinterpret_cast<uint4*>(&s_tile[(tid >> 3) * TILE_B + TROWS * ROW_B + (tid & 7) * 16]) = make_uint4(0, 0, 0, 0);
    const uint32_t chunk0 = (lane & 3) * 16, chunk1 = chunk0 | 64;
    uint4 x[2][2];
    // the two chunks of the tile row of vocabulary row K of this quad
    auto fetch = [&](auto k, const Pair& e) {
        constexpr int K = decltype(k)::value;
        const uint32_t r = quad_lane<K>(e.off);
        x[K & 1][0] = *reinterpret_cast<const uint4*>(&s_tile[r ^ chunk0]);
        x[K & 1][1] = *reinterpret_cast<const uint4*>(&s_tile[r ^ chunk1]);
    };
    // nz: which lanes of the wave hold a pair with a gradient
    auto multiply = [&](auto k, const Pair& e, unsigned long long nz) {
        constexpr int K = decltype(k)::value;
        if (nz & (0x1111111111111111ull << K)) {
            const float g = __uint_as_float(quad_lane<K>(__float_as_uint(e.g)));
            RowChunk<uint16_t>::fma(x[K & 1][0], g, acc[K]);
            RowChunk<uint16_t>::fma(x[K & 1][1], g, acc[K] + 8);
        }
    };
    constexpr std::integral_constant<int, 0> r0{};
    constexpr std::integral_constant<int, 1> r1{};
    constexpr std::integral_constant<int, 2> r2{};
    constexpr std::integral_constant<int, 3> r3{};
    const int b_last = B - 1;
    auto rows_of = [&](int b) { return tops ? tops[b] : S; };
    gload(0);
    tile_load(0, 0, rows_of(0));
    int top = rows_of(min(1, b_last));
    Pair cur = stage(0, true), before{0.f, 0u};
    unsigned long long nz = __ballot(cur.g != 0.f), nz_before = 0;
    wait_vmcnt<0>();
    __syncthreads();
    for (int b = 0; b < B; ++b) {
        const int buf = b & 1;
        // the last round loads and stages the last sequence once more (into the buffer nobody reads again):
        // no branch around the loads
        const bool more = b + 1 < B;
        gload(more ? b + 1 : b);
        tile_load(more ? b + 1 : b, buf ^ 1, top);
        top = rows_of(min(b + 2, b_last));
        fetch(r0, cur);
        __builtin_amdgcn_sched_barrier(0);
        multiply(r3, before, nz_before);
        fetch(r1, cur);
        __builtin_amdgcn_sched_barrier(0);
        multiply(r0, cur, nz);
        fetch(r2, cur);
        __builtin_amdgcn_sched_barrier(0);
        multiply(r1, cur, nz);
        fetch(r3, cur);
        __builtin_amdgcn_sched_barrier(0);
        multiply(r2, cur, nz);
        before = cur;
        nz_before = nz;
        cur = stage(buf ^ 1, more);
        nz = __ballot(cur.g != 0.f);
        __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): this tile's last row is in registers
        wait_vmcnt<0>();                               // the next tile has landed
        __syncthreads();
    }
    multiply(r3, before, nz_before);
    if (sum_db && vs_ok) db[vs] = (float)db_acc;
    if (!dW) return;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int v = v0 + (tid & ~3) + k;
        if (v < V) {
            const size_t o = (size_t)v * D + dc * DWS_COLS + (lane & 3) * 8;
#pragma unroll
            for (int i = 0; i < 16; i += 4) {
                const size_t at = o + (i & 7) + (i >> 3) * 32;
                float4 r = make_float4(acc[k][i], acc[k][i + 1], acc[k][i + 2], acc[k][i + 3]);
                if (add_dst) r = add4(OutVec<OT>::load4(dW + at), r);
                OutVec<OT>::store4(dW + at, r);
            }
        }
    }
}

}  // namespace lsr
