// Forward for calls of few tokens (one query of a serving loop): mask compaction, GEMM, maximum and
// activation in one launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fwd_mfma.hpp"

namespace lsr {

// What bounds such a call is the latency of reading W once.  The tile kernel puts 256 vocabulary entries on a
// workgroup, half the CUs at |V| = 30522, streams W through a ring that holds two slabs, and waits for a packing
// launch in front.  Here a wave owns 32 vocabulary entries at a time (954 for 1024 SIMDs at |V| = 30522), takes their
// rows of W straight into registers as MFMA fragments, FEW_U k-steps requested while the FEW_U before them are
// multiplied, and requests the first of them before it looks at the mask, or at the sums of the entries before.
// The hidden states of the valid tokens (at most FEW_MAX_TOKENS) lie in LDS, compacted, in rows padded so that
// fragment reads are free of bank conflicts; rows behind the last valid token are never filled and their products
// never looked at.  Every logit is the same sequence of MFMAs as in the tile kernel, so the results are the same
// bits, which the tests hold it to.  The logits then go through an area of LDS that the wave has to itself to one pair of lanes per (sequence,
// column), half a sequence each.  Workgroups stay and walk the vocabulary, FEW_COLS entries at a time, without a barrier.
constexpr int FEW_THREADS = 256;
constexpr int FEW_COLS = 32 * FEW_THREADS / 64;      // vocabulary entries per workgroup
constexpr int FEW_MAX_TOKENS = 64;                   // B * S
constexpr int FEW_U = 16;                            // k-steps per batch of loads
constexpr int FEW_LDS = 156 * 1024;                  // (the fragments in flight take the registers for one workgroup per CU anyway)
// LDS bytes of a row of hidden states of row_bytes, and of a call: the hidden states and the logits
inline int few_stride(int row_bytes) { return (row_bytes + 255) / 256 * 256 + 16; }
inline long few_lds(int tokens, int row_bytes) {
    return (long)((tokens + 31) / 32 * 32) * (few_stride(row_bytes) + FEW_COLS * 4);
}

template <typename T, bool ARG>
__global__ __launch_bounds__(FEW_THREADS) void fwd_few_kernel(const T* __restrict__ H, const T* __restrict__ W,
                                                              const float* __restrict__ bias,
                                                              const uint8_t* __restrict__ mask, float* __restrict__ Y,
                                                              int* __restrict__ I, int B, int S, int D, int V, int stride,
                                                              int n_tiles) {
    typedef typename FwdFrag<T>::type Frag;
    __shared__ __attribute__((aligned(16))) uint8_t s_buf[FEW_LDS];
    __shared__ int s_tok[FEW_MAX_TOKENS];            // b * S + s of the valid tokens
    __shared__ int s_start[FEW_MAX_TOKENS + 1];      // first row of each sequence
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int row_bytes = D * (int)sizeof(T);
    const int nks = (row_bytes + 31) / 32;           // k-steps of two 16-byte chunks
    int tile = blockIdx.x;
    int v = tile * FEW_COLS + wave * 32 + l32;
    const char* wrow = nullptr;
    auto w_row = [&]() { wrow = reinterpret_cast<const char*>(W) + (size_t)(v < V ? v : V - 1) * row_bytes + half * 16; };
    w_row();

    auto load_w = [&](Frag (&w)[FEW_U], int k0) {
        if ((k0 + FEW_U) * 32 <= row_bytes) {
#pragma unroll
            for (int u = 0; u < FEW_U; ++u) w[u] = *reinterpret_cast<const Frag*>(wrow + (k0 + u) * 32);
        } else {
#pragma unroll
            for (int u = 0; u < FEW_U; ++u) {
                w[u] = Frag{};
                if ((k0 + u) * 32 + half * 16 < row_bytes) w[u] = *reinterpret_cast<const Frag*>(wrow + (k0 + u) * 32);
            }
        }
    };
    Frag w0[FEW_U], w1[FEW_U];
    load_w(w0, 0);

    // valid tokens in ascending order
    if (wave == 0) {
        const bool f = lane < B * S && mask[lane] != 0;
        const unsigned long long bal = __ballot(f);
        const int k = __popcll(bal & ((1ull << lane) - 1ull));
        if (f) s_tok[k] = lane;
        if (lane < B * S && lane % S == 0) s_start[lane / S] = k;
        if (lane == 0) s_start[B] = __popcll(bal);
    }
    __syncthreads();
    const int n_rows = s_start[B];
    // hidden states into LDS, four chunks in flight per thread; a chunk behind the end of a row (odd number of chunks) is zero
    const int cpr = nks * 2, n_ch = n_rows * cpr;
    for (int e0 = tid; e0 < n_ch; e0 += 4 * FEW_THREADS) {
        uint4 x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * FEW_THREADS;
            const int r = e / cpr, c = e - r * cpr;
            x[u] = make_uint4(0, 0, 0, 0);
            if (e < n_ch && c * 16 < row_bytes)
                x[u] = *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(H) + (size_t)s_tok[r] * row_bytes + c * 16);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * FEW_THREADS;
            const int r = e / cpr, c = e - r * cpr;
            if (e < n_ch) *reinterpret_cast<uint4*>(&s_buf[r * stride + c * 16]) = x[u];
        }
    }
    __syncthreads();

    float* const s_logit = reinterpret_cast<float*>(s_buf + (B * S + 31) / 32 * 32 * stride) + wave * 32;      // [row][FEW_COLS]
    // the next tile's first fragments, requested before this one's logits are looked at
    int v_next = v;
    auto next = [&]() {
        if (tile + (int)gridDim.x >= n_tiles) return;
        v_next = v + (int)gridDim.x * FEW_COLS;
        wrow = reinterpret_cast<const char*>(W) + (size_t)(v_next < V ? v_next : V - 1) * row_bytes + half * 16;
        load_w(w0, 0);
    };
    auto blocks = [&](auto nb_c) {
        constexpr int NB = decltype(nb_c)::value;
        floatx16 acc[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
        const uint8_t* const sa = s_buf + l32 * stride + half * 16;
        auto multiply = [&](const Frag (&w)[FEW_U], int k0) {
#pragma unroll
            for (int u = 0; u < FEW_U; ++u) {
                if (k0 + u < nks) {
                    const Frag b = in_k_order(w[u]);
#pragma unroll
                    for (int i = 0; i < NB; ++i)
                        acc[i] = mma_chunk(in_k_order(*reinterpret_cast<const Frag*>(sa + i * 32 * stride + (k0 + u) * 32)), b, acc[i]);
                }
            }
        };
        for (int k0 = 0; k0 < nks; k0 += 2 * FEW_U) {
            if (k0 + FEW_U < nks) load_w(w1, k0 + FEW_U);
            multiply(w0, k0);
            if (k0 + 2 * FEW_U < nks) load_w(w0, k0 + 2 * FEW_U);
            if (k0 + FEW_U < nks) multiply(w1, k0 + FEW_U);
        }
        next();
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) s_logit[acc_row(i, r, half) * FEW_COLS + l32] = acc[i][r];
    };
    for (; tile < n_tiles; tile += gridDim.x) {
        const float bias_v = v < V ? bias[v] : 0.f;
        if (n_rows > 32) blocks(std::integral_constant<int, 2>{});
        else if (n_rows > 0) blocks(std::integral_constant<int, 1>{});
        else next();
        __builtin_amdgcn_wave_barrier();             // a wave reads only what it wrote, in program order
        for (int b = 0; b < B; ++b) {
            const int r0 = s_start[b], r1 = s_start[b + 1];
            const int mid = (r0 + r1 + 1) >> 1;
            float m = -INFINITY;                     // never replaced by NaN
            int at = -1;
            const int e = half ? r1 : mid;
#pragma unroll 8
            for (int r = half ? mid : r0; r < e; ++r) {
                const float x = s_logit[r * FEW_COLS + l32];
                if (x > m) { m = x; at = r; }
            }
            const float m2 = __shfl_xor(m, 32);
            const int at2 = __shfl_xor(at, 32);
            if (half == 0 && v < V) {
                if (m2 > m) { m = m2; at = at2; }    // rows of the second half hold higher positions: strict
                const size_t o = (size_t)b * V + v;
                Y[o] = r1 > r0 ? log1pf(fmaxf(m + bias_v, 0.f)) : 0.f;
                if (ARG) I[o] = at >= 0 ? s_tok[at] - b * S : 0;
            }
        }
        __builtin_amdgcn_wave_barrier();
        v = v_next;
    }
}

}  // namespace lsr
