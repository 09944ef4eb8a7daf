// CTC gate (Sec. 2.1): frame entropy (Eq. 3), greedy alignment (Eq. 2), collapse map B, decision.
//
// Kernel 1 (gate_frames_*): one CTC frame per group of LPR lanes.  The whole row of scores is
// loaded once with 16-byte loads and kept in registers; the row maximum, the lowest index that
// attains it, sum exp(z-m) and sum exp(z-m)(z-m) are reduced inside the lane group.
//     H = log S - W / S,   S = sum_a exp(z_a - m),   W = sum_a exp(z_a - m) (z_a - m)
// which equals -sum_a p_a log p_a for p = softmax(z).  The kernel streams the logits exactly once
// and is bound by HBM bandwidth (co-limited by vector ALU issue for bf16 input).
//
// Kernel 2 (gate_utterances): one workgroup per utterance: max_t H_t, threshold test, and a
// stable compaction of the frames kept by B (not blank, and different from the previous frame).
//
// Batches that do not fill the device take both steps in one launch (gate_fused).
#include <algorithm>
#include "device_utils.h"
#include "gate_utterance.h"
#include "ssd_internal.h"

namespace ssd {

template <typename T> struct Chunk;          // 16 bytes of scores
template <> struct Chunk<float> {
    static constexpr int N = 4;
    static constexpr uint32_t NEG_INF = 0xff800000u;
    static __device__ __forceinline__ void unpack(const uint4& c, float* z) {
        z[0] = __uint_as_float(c.x); z[1] = __uint_as_float(c.y);
        z[2] = __uint_as_float(c.z); z[3] = __uint_as_float(c.w);
    }
};
template <> struct Chunk<bf16_t> {
    static constexpr int N = 8;
    static constexpr uint32_t NEG_INF = 0xff80ff80u;
    static __device__ __forceinline__ void unpack(const uint4& c, float* z) {
        z[0] = bf16_lo(c.x); z[1] = bf16_hi(c.x); z[2] = bf16_lo(c.y); z[3] = bf16_hi(c.y);
        z[4] = bf16_lo(c.z); z[5] = bf16_hi(c.z); z[6] = bf16_lo(c.w); z[7] = bf16_hi(c.w);
    }
};

// Rows are V scores with V*sizeof(T) a multiple of 16; a row has n_chunks <= LPR*NCH chunks.
// Lane g of a group owns chunks g, g+LPR, g+2*LPR, ...
// out(row, H, arg) is called by one lane per row.
template <typename T, int LPR, int NCH, class Out>
__device__ __forceinline__ void frame_vec(const T* __restrict__ logits, int64_t row, int64_t n_rows, int V, Out out) {
    constexpr int EPC = Chunk<T>::N;
    const int g = threadIdx.x % LPR;
    const bool live = row < n_rows;
    if (!live) row = n_rows - 1;                      // keep the lane group whole for the reductions
    const int n_chunks = V / EPC;
    const uint4* src = reinterpret_cast<const uint4*>(logits + row * (int64_t)V);

    uint4 c[NCH];
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
        const int idx = g + k * LPR;
        if (idx < n_chunks) {
            typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
            const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(src + idx));
            c[k] = make_uint4(v.x, v.y, v.z, v.w);
        }
        else c[k] = make_uint4(Chunk<T>::NEG_INF, Chunk<T>::NEG_INF, Chunk<T>::NEG_INF, Chunk<T>::NEG_INF);
    }

    float m = -INFINITY;
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
        float z[EPC];
        Chunk<T>::unpack(c[k], z);
#pragma unroll
        for (int e = 0; e < EPC; e += 2) m = fmaxf(m, fmaxf(z[e], z[e + 1]));
    }
    m = group_allreduce<LPR>(m, OpMax());

    // Walk the lane's elements from the highest index down so the last match is the lowest index.
    float S = 0.f, W = 0.f;
    int arg = 0x7fffffff;
#pragma unroll
    for (int k = NCH - 1; k >= 0; --k) {
        float z[EPC];
        Chunk<T>::unpack(c[k], z);
        const int base = (g + k * LPR) * EPC;
#pragma unroll
        for (int e = EPC - 1; e >= 0; --e) {
            const float d = z[e] - m;
            const float ex = __expf(d);
            S += ex;
            W = fmaf(ex, d, W);
            arg = (z[e] == m) ? base + e : arg;
        }
    }
    if (W != W) {
        // a score of -inf gives 0 * -inf above; redo the weighted sum with such terms as 0
        W = 0.f;
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            float z[EPC];
            Chunk<T>::unpack(c[k], z);
#pragma unroll
            for (int e = 0; e < EPC; ++e) {
                const float d = fmaxf(z[e] - m, -1e30f);
                W = fmaf(__expf(d), d, W);
            }
        }
    }
    S = group_allreduce<LPR>(S, OpSum());
    W = group_allreduce<LPR>(W, OpSum());
    arg = group_allreduce_i<LPR>(arg, OpMinI());
    if (live && g == 0) out(row, __logf(S) - W / S, arg);
}
template <typename T, int LPR, int NCH>
__global__ void __launch_bounds__(256) gate_frames_vec(const T* __restrict__ logits, int64_t n_rows,
                                                       int V, float* __restrict__ H_out,
                                                       int32_t* __restrict__ arg_out) {
    frame_vec<T, LPR, NCH>(logits, (int64_t)blockIdx.x * (256 / LPR) + threadIdx.x / LPR, n_rows, V,
                           [&](int64_t row, float H, int arg) { H_out[row] = H; arg_out[row] = arg; });
}

// bf16 fast path.  A bf16 score widened to fp32 has 16 zero bits at the bottom; the complement of
// the element index is put there while widening (one v_lshl_or / v_and_or per element, the same
// cost as the plain widening), so that ONE float maximum over these keys yields both the row maximum
// (top 16 bits) and, among equal scores, the lowest index (largest complement) -- no per-element
// compare/select.  That holds for a positive, normal maximum; rows whose maximum is negative, zero,
// denormal or non-finite take the generic route (compare/select per element), chosen per
// wavefront.  The second sweep is one fma (z*log2e - m*log2e), one v_exp_f32, one add, one fma per
// element:  H = ln2 * (log2 S - W2/S) with S = sum 2^t, W2 = sum 2^t t, which is shift invariant
// in t, so the rounding of m*log2e cancels.
// The kernel is persistent (grid-stride over row blocks) so the per-lane index constants are built
// once, and the loads of the next row block are issued before the arithmetic of the current one.
__device__ __forceinline__ float max3_bits(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));   // returns an operand bit-exactly
    return r;
}
__device__ __forceinline__ float max_bits(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
template <int W>
__device__ __forceinline__ float group_max_bits(float v) {
    v = max_bits(v, dpp_f<DPP_XOR1>(v));
    v = max_bits(v, dpp_f<DPP_XOR2>(v));
    v = max_bits(v, dpp_f<DPP_HALF_MIRROR>(v));
    v = max_bits(v, dpp_f<DPP_MIRROR>(v));
    if (W > 16) {
        v = max_bits(v, __shfl_xor(v, 16));
        v = max_bits(v, __shfl_xor(v, 32));
    }
    return v;
}

// Row blocks first, first + stride, ... (ONE: the first alone, with no second set of registers); FULL: the row has exactly LPR*NCH chunks (no chunk predicate)
template <int LPR, int NCH, bool FULL, bool ONE, class Out>
__device__ __forceinline__ void frames_bf16_keyed(const bf16_t* __restrict__ logits, int64_t n_rows, int V, int64_t first, int64_t stride, Out out) {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int ROWS_PER_BLOCK = 256 / LPR;
    constexpr float LOG2E = 1.4426950408889634f, LN2 = 0.6931471805599453f;
    const int g = threadIdx.x % LPR;
    const int n_chunks = V / 8;
    const int64_t n_blocks = (n_rows + ROWS_PER_BLOCK - 1) / ROWS_PER_BLOCK;
    // (~index) & 0xffff of the eight elements of this lane's first chunk.  Chunk k lies 128 k elements
    // further; for the row lengths served here (at most 8 chunks of 16 lanes) that only clears bits
    // 7.. of the complement, so the key of chunk k is the key of chunk 0 xor (k << 7): applied once
    // per chunk to the chunk's maximum, not per element.  Eight constants instead of one per element
    // keep the kernel at 150 registers, i.e. three wavefronts per SIMD instead of two (5.2 -> 5.6 TB/s).
    uint32_t low0[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) low0[e] = (~(uint32_t)(g * 8 + e)) & 0xffffu;
    auto load_block = [&](int64_t blk, u32x4 (&c)[NCH]) {
        int64_t row = blk * ROWS_PER_BLOCK + threadIdx.x / LPR;
        if (row >= n_rows) row = n_rows - 1;
        const u32x4* src = reinterpret_cast<const u32x4*>(logits + row * (int64_t)V) + g;
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            if (FULL || g + k * LPR < n_chunks) c[k] = __builtin_nontemporal_load(src + k * LPR);
            else c[k] = (u32x4){0xf14af14au, 0xf14af14au, 0xf14af14au, 0xf14af14au};   // about -1e30: finite, exp -> 0
        }
    };

    u32x4 buf0[NCH], buf1[NCH];
    if (first < n_blocks) load_block(first, buf0);
    // two row blocks per trip so that the register sets swap roles without copies
    for (int64_t blk0 = first; blk0 < n_blocks; blk0 += 2 * stride) {
      #pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int64_t blk = blk0 + half * stride;
        if (blk >= n_blocks) break;
        u32x4 (&cur)[NCH] = half ? buf1 : buf0;
        u32x4 (&nxt)[NCH] = half ? buf0 : buf1;
        const int64_t nblk = blk + stride;
        if (!ONE && nblk < n_blocks) load_block(nblk, nxt);
        const int64_t row = blk * ROWS_PER_BLOCK + threadIdx.x / LPR;
        const bool live = row < n_rows;

        // ---- sweep 1: maximum of the keyed values
        float mk = __uint_as_float(0xff800000u);           // -inf
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            float mc = __uint_as_float(0xff800000u);
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const uint32_t x = cur[k][w];
                const float k_lo = __uint_as_float((x << 16) | low0[2 * w]);
                const float k_hi = __uint_as_float((x & 0xffff0000u) | low0[2 * w + 1]);
                mc = max3_bits(mc, k_lo, k_hi);
            }
            // (a chunk without any value above -inf turns into a non-number here, which the maximum ignores)
            mk = max_bits(mk, __uint_as_float(__float_as_uint(mc) ^ (uint32_t)(k * LPR * 8)));
        }
        mk = group_max_bits<LPR>(mk);
        const uint32_t mb = __float_as_uint(mk);
        const uint32_t expo = mb & 0x7f800000u;
        const bool easy = (mb >> 31) == 0 && expo != 0 && expo != 0x7f800000u;
        // generic route: plain maximum, then the lowest index that attains it by compare/select
        auto generic_max = [&](float& m, int& arg) {
            m = -INFINITY;
#pragma unroll
            for (int k = 0; k < NCH; ++k)
#pragma unroll
                for (int w = 0; w < 4; ++w) m = fmaxf(m, fmaxf(bf16_lo(cur[k][w]), bf16_hi(cur[k][w])));
            m = group_allreduce<LPR>(m, OpMax());
            arg = 0x7fffffff;
#pragma unroll
            for (int k = NCH - 1; k >= 0; --k)
#pragma unroll
                for (int w = 3; w >= 0; --w) {
                    const int base = (g + k * LPR) * 8 + 2 * w;
                    arg = (bf16_hi(cur[k][w]) == m) ? base + 1 : arg;
                    arg = (bf16_lo(cur[k][w]) == m) ? base : arg;
                }
            arg = group_allreduce_i<LPR>(arg, OpMinI());
        };
        float m, S = 0.f, W2 = 0.f;
        int arg;
        if (__all(easy)) {
            m = __uint_as_float(mb & 0xffff0000u);
            arg = (int)((~mb) & 0xffffu);
        } else {
            generic_max(m, arg);
        }
        // ---- sweep 2: S = sum 2^t, W2 = sum 2^t t,  t = (z - m) log2(e) up to a row constant
        float nml = -m * LOG2E;
#pragma unroll
        for (int k = 0; k < NCH; ++k)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float t0 = fmaf(bf16_lo(cur[k][w]), LOG2E, nml), t1 = fmaf(bf16_hi(cur[k][w]), LOG2E, nml);
                const float e0 = __builtin_amdgcn_exp2f(t0), e1 = __builtin_amdgcn_exp2f(t1);
                S += e0; W2 = fmaf(e0, t0, W2);
                S += e1; W2 = fmaf(e1, t1, W2);
            }
        if (__any(W2 != W2)) {
            // A score of -inf gives 0 * -inf above (and a non-number key in sweep 1): redo the rows of
            // this wavefront on the generic route, with such terms counted as 0.
            generic_max(m, arg);
            nml = -m * LOG2E;
            S = 0.f; W2 = 0.f;
#pragma unroll
            for (int k = 0; k < NCH; ++k)
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const float t0 = fmaxf(fmaf(bf16_lo(cur[k][w]), LOG2E, nml), -1e30f);
                    const float t1 = fmaxf(fmaf(bf16_hi(cur[k][w]), LOG2E, nml), -1e30f);
                    const float e0 = __builtin_amdgcn_exp2f(t0), e1 = __builtin_amdgcn_exp2f(t1);
                    S += e0; W2 = fmaf(e0, t0, W2);
                    S += e1; W2 = fmaf(e1, t1, W2);
                }
        }
        S = group_allreduce<LPR>(S, OpSum());
        W2 = group_allreduce<LPR>(W2, OpSum());
        if (live && g == 0) out(row, LN2 * (__builtin_amdgcn_logf(S) - W2 / S), arg);
        if (ONE) return;
      }
    }
}
template <int LPR, int NCH, bool FULL>
__global__ void __launch_bounds__(256) gate_frames_bf16_keyed(const bf16_t* __restrict__ logits, int64_t n_rows, int V,
                                                              float* __restrict__ H_out, int32_t* __restrict__ arg_out) {
    frames_bf16_keyed<LPR, NCH, FULL, false>(logits, n_rows, V, blockIdx.x, gridDim.x,
                                           [&](int64_t row, float H, int arg) { H_out[row] = H; arg_out[row] = arg; });
}

// Any V, any alignment: one wavefront per row, two passes over memory (second pass hits cache).
template <typename T>
__global__ void __launch_bounds__(256) gate_frames_generic(const T* __restrict__ logits, int64_t n_rows,
                                                           int V, float* __restrict__ H_out,
                                                           int32_t* __restrict__ arg_out) {
    const int lane = threadIdx.x % 64;
    int64_t row = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    const bool live = row < n_rows;
    if (!live) row = n_rows - 1;
    const T* src = logits + row * (int64_t)V;
    auto ld = [&](int i) -> float {
        if constexpr (sizeof(T) == 2) return bf16_to_f32(src[i]); else return src[i];
    };
    float m = -INFINITY;
    for (int i = lane; i < V; i += 64) m = fmaxf(m, ld(i));
    m = group_allreduce<64>(m, OpMax());
    float S = 0.f, W = 0.f;
    int arg = 0x7fffffff;
    for (int i = lane; i < V; i += 64) {
        const float z = ld(i);
        const float d = fmaxf(z - m, -1e30f);
        const float ex = __expf(d);
        S += ex;
        W = fmaf(ex, d, W);
        if (z == m && i < arg) arg = i;
    }
    S = group_allreduce<64>(S, OpSum());
    W = group_allreduce<64>(W, OpSum());
    arg = group_allreduce_i<64>(arg, OpMinI());
    if (live && lane == 0) {
        H_out[row] = __logf(S) - W / S;
        arg_out[row] = arg;
    }
}

// One workgroup (256 threads) per utterance.  The frame range of an utterance is clamped into
// [0, n_rows], so that prefix sums that were never seen by the host cannot lead outside H / arg / draft.
template <class CU>
__global__ void __launch_bounds__(256) gate_utterances(const float* __restrict__ H,
                                                       const int32_t* __restrict__ arg,
                                                       const CU cu_frames, int n_rows, int blank,
                                                       float tau, float* __restrict__ max_entropy,
                                                       uint8_t* __restrict__ gate_pass,
                                                       int32_t* __restrict__ draft, int32_t* __restrict__ draft_len) {
    const int b = blockIdx.x;
    const int lo = min(max(cu_frames(b), 0), n_rows), hi = min(max(cu_frames(b + 1), lo), n_rows);
    gate_utterance<4, 4>(b, lo, hi, blank, tau, max_entropy, gate_pass, draft, draft_len,
                        [&](int t, float& h, int& a) { a = arg[t]; h = H[t]; }, [&](int t, int) { return arg[max(t - 1, lo)]; });
}

// ---- Both steps in one launch: the workgroup whose rows complete an utterance finishes it.
// A small call is bound by the host's two launches (8.8 us; of one, 6.5), not by what they do.  Every workgroup does one block of
// rows, stores the frames' statistics write-through, waits for the stores, and adds the rows it did to a count per utterance; whoever
// brings a count to the utterance's length reads the statistics past L1 and L2, decides, compacts, and clears the count for the
// next call.  Nobody waits for anybody.  (No agent-scope fences: they write back and invalidate a whole L2.)
// us a call, two launches / one: one utterance of 250 frames of 512 bf16 scores 9.9 / 7.0, 64 of 100 10.3 / 7.1, 32 of 500 9.9 / 7.2,
// 64 of 250 frames of 348 fp32 scores 10.0 / 8.3.
// Where the one launch stays the faster: until the device takes longer for it than the host for two (9.8 us).  A row block pays for its stores
// and the count with waits, which add up with the scores (two / one launch in us, MiB of scores; 512 bf16, 64 utterances: 24 9.7 / 8.1,
// 28 9.9 / 9.1, 32 10.9 / 10.0, 40 even; 348 fp32: 24 10.1 / 9.1, 28 10.1 / 9.6, 32 10.2 / 10.6, at 256 utterances 24 10.0 / 9.9, 28 9.9 /
// 10.3, 32 10.2 / 11.8; 256 and 512 fp32: 28 9.8 / 8.0 and 10.1 / 7.6); and additions to one count go one after the other, so that
// the last block of a long utterance waits for all before it.  That shows where the device is late already: 4 utterances of 188 blocks,
// 16 MiB, 10.0 / 11.3; of 192, 12 MiB, 9.7 / 10.6; of 141, 12 MiB, 10.1 / 10.0; of 128, 8 MiB, 9.8 / 8.0; 16 of 96, 24 MiB, 9.8 / 10.1; 16 of
// 80, 20 MiB, 9.7 / 8.3; 2 of 188, 3 MiB, 9.8 / 7.3.  Of 209 calls measured these limits take 168, of which one is more than 2 % slower (4 %);
// they leave 12 to the two launches that the one would take 5 to 20 % less for.  And no more workgroups than have a place in the arguments.
constexpr int64_t GATE_FUSED_MAX_BYTES = (int64_t)28 << 20;
constexpr int64_t GATE_FUSED_MAX_UTT_BYTES = (int64_t)2000 << 20;     // blocks of the longest utterance times bytes of the call
constexpr int GATE_FUSED_MAX_BLOCKS = 2048, GATE_FUSED_MAX_UTT_BLOCKS = 192;
constexpr int ARRIVED_STRIDE = GATE_ARRIVED_BYTES / GATE_MAX_ARG_UTTS / 4;
struct GateTail {
    uint8_t first[GATE_FUSED_MAX_BLOCKS];      // the utterance of a workgroup's first row.  No utterance has fewer rows than a workgroup, which so has rows of two at most
    int32_t cu[GATE_MAX_ARG_UTTS + 1];
    int blank;
    float tau;
    float* max_entropy; uint8_t* gate_pass; int32_t* draft; int32_t* draft_len;
    unsigned* arrived;
};
template <class V> __device__ __forceinline__ void store_shared(V* p, V v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <class V> __device__ __forceinline__ V load_shared(const V* p) { return __hip_atomic_load(const_cast<V*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T, int LPR, int NCH>
__global__ void __launch_bounds__(256) gate_fused(const T* __restrict__ logits, int n_rows, int V, float* H, int32_t* arg, const GateTail g) {
    constexpr int ROWS = 256 / LPR;
    const int row0 = blockIdx.x * ROWS, end = min(row0 + ROWS, n_rows);
    const int b0 = g.first[blockIdx.x], lo = g.cu[b0], mid = g.cu[b0 + 1];
    auto out = [&](int64_t row, float h, int a) {
        store_shared(H + row, h);
        store_shared(arg + row, (int32_t)a);
    };
    if constexpr (sizeof(T) == 2) {
        if (V / 8 == LPR * NCH) frames_bf16_keyed<LPR, NCH, true, true>(logits, n_rows, V, blockIdx.x, gridDim.x, out);
        else frames_bf16_keyed<LPR, NCH, false, true>(logits, n_rows, V, blockIdx.x, gridDim.x, out);
    } else {
        frame_vec<T, LPR, NCH>(logits, row0 + threadIdx.x / LPR, n_rows, V, out);
    }

    __shared__ int complete_s[2];
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // stored
    __syncthreads();
    if (threadIdx.x < 2) {
        const bool second = threadIdx.x == 1;
        const int mine = second ? end - mid : min(mid, end) - row0;
        bool complete = false;
        if (mine > 0) {
            unsigned* n = g.arrived + (b0 + second) * ARRIVED_STRIDE;
            const int length = second ? g.cu[b0 + 2] - mid : mid - lo;
            complete = __hip_atomic_fetch_add(n, (unsigned)mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + mine == (unsigned)length;
            if (complete) store_shared(n, 0u);
        }
        complete_s[threadIdx.x] = complete;
    }
    __syncthreads();
#pragma unroll 1
    for (int u = 0; u < 2; ++u)
        if (__builtin_amdgcn_readfirstlane(complete_s[u]))
            gate_utterance<4, 4>(b0 + u, g.cu[b0 + u], g.cu[b0 + u + 1], g.blank, g.tau, g.max_entropy, g.gate_pass, g.draft, g.draft_len,
                           [&](int t, float& h, int& a) { a = load_shared(arg + t); h = load_shared(H + t); }, [&](int t, int) { return load_shared(arg + max(t - 1, g.cu[b0 + u])); });
}

void launch_gate_utterances(const float* H, const int32_t* arg, const int32_t* cu_frames_dev, int64_t n_rows, int B, int blank,
                            float tau, float* max_entropy, uint8_t* gate_pass, int32_t* draft, int32_t* draft_len,
                            hipStream_t st) {
    hipLaunchKernelGGL(gate_utterances<CuArray>, dim3(B), dim3(256), 0, st, H, arg, CuArray{cu_frames_dev}, (int)n_rows, blank, tau,
                       max_entropy, gate_pass, draft, draft_len);
}

static bool pairs_fit(const int32_t* cu, int B) {
    if (B > GATE_MAX_PAIR_UTTS) return false;
    for (int b = 0; b < B; b += 2)                           // the lengths before the odd sums
        if (cu[b + 1] - cu[b] > 0xffff) return false;
    return true;
}
bool gate_prefix_fits_arguments(const int32_t* cu, int B) { return B <= GATE_MAX_ARG_UTTS || pairs_fit(cu, B); }
bool make_cu_pairs(const int32_t* cu, int B, CuPairs& out) {
    if (!pairs_fit(cu, B)) return false;
    for (int b = 0; b <= B; b += 2) out.even[b / 2] = cu[b];
    for (int p = 0; 2 * p + 1 <= B; ++p) {
        const int len = cu[2 * p + 1] - cu[2 * p];
        uint32_t& w = out.odd[p / 2];
        w = p % 2 ? w | (uint32_t)len << 16 : (uint32_t)len;
    }
    return true;
}

bool launch_gate_utterances_host(const float* H, const int32_t* arg, const int32_t* cu_frames, int64_t n_rows, int B, int blank,
                                 float tau, float* max_entropy, uint8_t* gate_pass, int32_t* draft, int32_t* draft_len,
                                 hipStream_t st) {
    if (B <= GATE_MAX_ARG_UTTS) {
        CuArgs cu;
        for (int b = 0; b <= B; ++b) cu.cu[b] = cu_frames[b];
        hipLaunchKernelGGL(gate_utterances<CuArgs>, dim3(B), dim3(256), 0, st, H, arg, cu, (int)n_rows, blank, tau,
                           max_entropy, gate_pass, draft, draft_len);
        return true;
    }
    CuPairs cu;
    if (!make_cu_pairs(cu_frames, B, cu)) return false;
    hipLaunchKernelGGL(gate_utterances<CuPairs>, dim3(B), dim3(256), 0, st, H, arg, cu, (int)n_rows, blank, tau,
                       max_entropy, gate_pass, draft, draft_len);
    return true;
}

template <typename T, int LPR>
static void launch_vec(const T* logits, int64_t n_rows, int V, float* H, int32_t* arg, hipStream_t st) {
    const int n_chunks = V / Chunk<T>::N;
    const int nch = (n_chunks + LPR - 1) / LPR;
    const unsigned grid = (unsigned)((n_rows + (256 / LPR) - 1) / (256 / LPR));
    if constexpr (sizeof(T) == 2) {
        // persistent launch: enough workgroups to fill 256 CUs several times over, no more than there is work
        const unsigned pgrid = grid < 256u * 8u ? grid : 256u * 8u;
        const bf16_t* z = logits;
        const bool full = n_chunks == nch * LPR;
#define SSD_GATE_LAUNCH(NCH_)                                                                                          \
        if (full) hipLaunchKernelGGL((gate_frames_bf16_keyed<LPR, NCH_, true>), dim3(pgrid), dim3(256), 0, st, z, n_rows, V, H, arg); \
        else hipLaunchKernelGGL((gate_frames_bf16_keyed<LPR, NCH_, false>), dim3(pgrid), dim3(256), 0, st, z, n_rows, V, H, arg)
        if (nch <= 1) { SSD_GATE_LAUNCH(1); }
        else if (nch <= 2) { SSD_GATE_LAUNCH(2); }
        else if (nch <= 4) { SSD_GATE_LAUNCH(4); }
        else { SSD_GATE_LAUNCH(8); }
#undef SSD_GATE_LAUNCH
        return;
    }
    if (nch <= 1) hipLaunchKernelGGL((gate_frames_vec<T, LPR, 1>), dim3(grid), dim3(256), 0, st, logits, n_rows, V, H, arg);
    else if (nch <= 2) hipLaunchKernelGGL((gate_frames_vec<T, LPR, 2>), dim3(grid), dim3(256), 0, st, logits, n_rows, V, H, arg);
    else if (nch <= 4) hipLaunchKernelGGL((gate_frames_vec<T, LPR, 4>), dim3(grid), dim3(256), 0, st, logits, n_rows, V, H, arg);
    // (1028 / 1536 scores, 17.6 K frames, as eight chunks of 64 lanes and as six: 20.0 / 20.4 and 17.1 / 17.4 us)
    else if (nch <= 6) hipLaunchKernelGGL((gate_frames_vec<T, LPR, 6>), dim3(grid), dim3(256), 0, st, logits, n_rows, V, H, arg);
    else hipLaunchKernelGGL((gate_frames_vec<T, LPR, 8>), dim3(grid), dim3(256), 0, st, logits, n_rows, V, H, arg);
}

// Lanes that share a row in the vectorised kernels, 16 or 64; 0: the row length or the alignment takes the general one.
template <typename T>
static int vec_lanes(const T* logits, int64_t n_rows, int V) {
    constexpr int EPC = Chunk<T>::N;
    if (V <= 0 || V % EPC || (reinterpret_cast<uintptr_t>(logits) & 15) || V > 64 * 8 * EPC) return 0;
    if (V > 16 * 8 * EPC) return 64;
    // fp32 rows of 257 to 512 scores: as two chunks of 64 lanes up to half of the slots are empty and every reduction
    // crosses DPP rows, but a lane has little to do and the few rows of a small batch spread over more wavefronts; as six or
    // eight chunks of 16 lanes four rows share a wavefront.  64 / 16 lanes in us, 260, 348, 384 scores: 250 frames 2.9 / 3.2, 2.9 / 3.2,
    // 2.9 / 3.0; 2000 frames even; 4000 frames 4.1 / 3.6, 4.3 / 3.7, 4.2 / 3.5; 17.6 K 8.9 / 7.0, 8.9 / 7.3, 9.0 / 6.0; 200 K 62 / 37,
    // 62 / 42, 64 / 45.  388, 448, 512 scores: 250 frames 2.8 / 3.4, 2.8 / 3.4, 2.7 / 3.2; 8000 frames even; 17.6 K 8.8 / 8.4, 8.9 / 8.1,
    // 7.7 / 7.3; 200 K 66 / 54, 63 / 51, 60 / 61.
    const int64_t few = V <= 16 * 6 * EPC ? 2048 : 8192;
    return V <= 16 * 4 * EPC || (sizeof(T) == 4 && n_rows > few) ? 16 : 64;
}
template <typename T>
static void launch_frames(const T* logits, int64_t n_rows, int V, float* H, int32_t* arg, hipStream_t st) {
    const int lanes = vec_lanes(logits, n_rows, V);
    if (lanes == 16) launch_vec<T, 16>(logits, n_rows, V, H, arg, st);
    else if (lanes == 64) launch_vec<T, 64>(logits, n_rows, V, H, arg, st);
    else {
        const unsigned grid = (unsigned)((n_rows + 3) / 4);
        hipLaunchKernelGGL((gate_frames_generic<T>), dim3(grid), dim3(256), 0, st, logits, n_rows, V, H, arg);
    }
}

void launch_gate_frames(const void* logits, int dtype, int64_t n_rows, int V, float* H, int32_t* arg, hipStream_t st) {
    if (dtype == SSD_BF16) launch_frames<bf16_t>(static_cast<const bf16_t*>(logits), n_rows, V, H, arg, st);
    else launch_frames<float>(static_cast<const float*>(logits), n_rows, V, H, arg, st);
}

template <typename T, int LPR>
static void launch_fused(const T* logits, int64_t n_rows, int V, float* H, int32_t* arg, const GateTail& tail, hipStream_t st) {
    const int nch = (V / Chunk<T>::N + LPR - 1) / LPR;
    const unsigned grid = (unsigned)((n_rows + (256 / LPR) - 1) / (256 / LPR));
#define SSD_FUSED(NCH_) hipLaunchKernelGGL((gate_fused<T, LPR, NCH_>), dim3(grid), dim3(256), 0, st, logits, (int)n_rows, V, H, arg, tail)
    if (nch <= 1) SSD_FUSED(1);
    else if (nch <= 2) SSD_FUSED(2);
    else if (nch <= 4) SSD_FUSED(4);
    else {
        if constexpr (sizeof(T) == 4) {
            if (nch <= 6) { SSD_FUSED(6); return; }
        }
        SSD_FUSED(8);
    }
#undef SSD_FUSED
}
bool launch_gate_fused(const void* logits, int dtype, const int32_t* cu_frames, int64_t n_rows, int B, int V, int blank, float tau, float* H, int32_t* arg,
                       float* max_entropy, uint8_t* gate_pass, int32_t* draft, int32_t* draft_len, unsigned* arrived, hipStream_t st) {
    const int lanes = dtype == SSD_BF16 ? vec_lanes(static_cast<const bf16_t*>(logits), n_rows, V) : vec_lanes(static_cast<const float*>(logits), n_rows, V);
    if (!arrived || B > GATE_MAX_ARG_UTTS || !lanes) return false;
    const int rows = 256 / lanes;
    const int64_t bytes = n_rows * V * (dtype == SSD_BF16 ? 2 : 4);
    if (n_rows > (int64_t)rows * GATE_FUSED_MAX_BLOCKS || bytes > GATE_FUSED_MAX_BYTES) return false;
    const int longest = rows * (int)std::min<int64_t>(GATE_FUSED_MAX_UTT_BLOCKS, GATE_FUSED_MAX_UTT_BYTES / bytes);
    GateTail tail;
    int block = 0;
    tail.cu[0] = 0;
    for (int b = 0; b < B; ++b) {
        const int length = cu_frames[b + 1] - cu_frames[b];
        if (length < rows || length > longest) return false;
        tail.cu[b + 1] = cu_frames[b + 1];
        for (; block * rows < cu_frames[b + 1]; ++block) tail.first[block] = (uint8_t)b;
    }
    tail.blank = blank; tail.tau = tau;
    tail.max_entropy = max_entropy; tail.gate_pass = gate_pass; tail.draft = draft; tail.draft_len = draft_len; tail.arrived = arrived;
    if (dtype == SSD_BF16) {
        if (lanes == 16) launch_fused<bf16_t, 16>(static_cast<const bf16_t*>(logits), n_rows, V, H, arg, tail, st);
        else launch_fused<bf16_t, 64>(static_cast<const bf16_t*>(logits), n_rows, V, H, arg, tail, st);
    } else {
        if (lanes == 16) launch_fused<float, 16>(static_cast<const float*>(logits), n_rows, V, H, arg, tail, st);
        else launch_fused<float, 64>(static_cast<const float*>(logits), n_rows, V, H, arg, tail, st);
    }
    return true;
}

}  // namespace ssd
