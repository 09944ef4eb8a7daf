// Second half of the gate: the entropy decision about an utterance and its collapsed greedy path, for the kernels that have the
// frames' statistics at hand in different forms (gate.hip: stored or just counted, ctc_head.hip: partial sums of symbol groups).
#pragma once
#include "device_utils.h"

namespace ssd {

// The decision about one utterance and its collapsed path, by WAVES wavefronts.  frame(t, H, arg) reads frame t's statistics,
// before(t, arg) the symbol of the frame before it (every lane of a wavefront asks, for consecutive frames; anything will do at t == lo).
// 1024 frames a trip, 256 threads times four or 1024 threads: every trip waits for memory once and for the other wavefronts twice (with
// 256 a trip, 1500 frames were six waits).
template <int WAVES, int AHEAD, class Frame, class Before>
__device__ __forceinline__ void gate_utterance(int b, int lo, int hi, int blank, float tau, float* __restrict__ max_entropy, uint8_t* __restrict__ gate_pass,
                                               int32_t* __restrict__ draft, int32_t* __restrict__ draft_len, Frame frame, Before before) {
    __shared__ int wave_cnt[AHEAD][WAVES];
    __shared__ float wave_max[WAVES];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64;
    float mx = -INFINITY;
    int written = 0;                                   // same value in every thread
    for (int t0 = lo; t0 < hi; t0 += 64 * WAVES * AHEAD) {
        int a[AHEAD], prev[AHEAD];
        float H[AHEAD];
        unsigned long long mask[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int t = min(t0 + u * 64 * WAVES + (int)threadIdx.x, hi - 1);
            frame(t, H[u], a[u]);
            prev[u] = before(t, a[u]);
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int t = t0 + u * 64 * WAVES + threadIdx.x;
            bool keep = false;
            if (t < hi) {
                mx = fmaxf(mx, H[u]);
                keep = (a[u] != blank) && (t == lo || a[u] != prev[u]);
            }
            mask[u] = __ballot(keep);
            if (lane == 0) wave_cnt[u][wave] = __popcll(mask[u]);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            int wave_off = 0, total = 0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                const int c = wave_cnt[u][w];
                if (w < wave) wave_off += c;
                total += c;
            }
            const unsigned long long below = (1ull << lane) - 1ull;
            if (mask[u] >> lane & 1) draft[lo + written + wave_off + __popcll(mask[u] & below)] = a[u];
            written += total;
        }
        __syncthreads();
    }
    mx = group_allreduce<64>(mx, OpMax());
    if (lane == 0) wave_max[wave] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
        float m = wave_max[0];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) m = fmaxf(m, wave_max[w]);
        max_entropy[b] = m;
        gate_pass[b] = (m < tau) ? 1 : 0;
        draft_len[b] = written;
    }
}

}  // namespace ssd
