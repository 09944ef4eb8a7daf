// Windowed cross-attention of the query-transformer projector (Sec. 3.1): every window of 15 consecutive encoder
// frames is summarised by 3 trainable queries, which turns the frame sequence into the 5 times shorter sequence
// of acoustic embeddings that the LLM is conditioned on (the g of Sec. 2.2).
//
// The queries are constants of the model, so the score of frame t for (query j, head h),
//     q_proj[j, h] . (w_k h_t)[h] / sqrt(d_head)  =  (w_k[h]^T q_proj[j, h] / sqrt(d_head)) . h_t,
// is a fixed linear function of the frame: the key projection folds into n_q * n_heads score rows.  Those rows and
// w_v form one weight matrix, and the path is
//   1. [scores | values] = enc_h w_cat^T                  one MFMA GEMM (gemm_mfma.hip): scores [frames, 64] fp32,
//                                                         values [frames, d_h] IEEE half
//   2. per window: softmax over its frames of each score column, weighted sum of the value columns   (here)
//   3. g [3 windows, d_out] = o w_o^T                      one MFMA GEMM, stored in the storage type of speech_emb
// Large batches of the usual shape skip the value columns of the product and project the values after the pooling instead
// (qformer_values.hip; the rule is values_after_pooling in api.hip).
// Windows never cross an utterance; the last window of an utterance may hold fewer frames.
#include "device_utils.h"
#include "ssd_internal.h"

namespace ssd {

int qformer_cat_rows(int d_h) { return (QF_SCORE_COLS + d_h + 255) / 256 * 256; }

// One workgroup per row of w_cat.
__global__ void __launch_bounds__(256) qformer_fold_kernel(const bf16_t* __restrict__ q_proj, const bf16_t* __restrict__ w_k,
                                                           const bf16_t* __restrict__ w_v, int n_q, int n_heads, int d_h,
                                                           int d_enc, bf16_t* __restrict__ w_cat) {
    const int r = blockIdx.x;
    bf16_t* dst = w_cat + (int64_t)r * d_enc;
    if (r < n_q * n_heads) {
        const int j = r / n_heads, h = r % n_heads, dh = d_h / n_heads;
        const float scale = 1.0f / sqrtf((float)dh);
        for (int e = threadIdx.x; e < d_enc; e += 256) {
            float acc = 0.f;
            for (int c = 0; c < dh; ++c)
                acc = fmaf(bf16_to_f32(q_proj[j * d_h + h * dh + c]), bf16_to_f32(w_k[(int64_t)(h * dh + c) * d_enc + e]), acc);
            dst[e] = f32_to_bf16(acc * scale);
        }
    } else if (r >= QF_SCORE_COLS && r < QF_SCORE_COLS + d_h) {
        const bf16_t* src = w_v + (int64_t)(r - QF_SCORE_COLS) * d_enc;
        for (int e = threadIdx.x; e < d_enc; e += 256) dst[e] = src[e];
    } else {
        for (int e = threadIdx.x; e < d_enc; e += 256) dst[e] = 0;
    }
}

void launch_qformer_fold(const uint16_t* q_proj, const uint16_t* w_k, const uint16_t* w_v, int n_q, int n_heads, int d_h,
                         int d_enc, uint16_t* w_cat, hipStream_t st) {
    hipLaunchKernelGGL(qformer_fold_kernel, dim3(qformer_cat_rows(d_h)), dim3(256), 0, st, q_proj, w_k, w_v, n_q, n_heads, d_h,
                       d_enc, w_cat);
}

// One workgroup per window.  Scores of the window's frames go through LDS, four threads normalise one
// (query, head) column over the frames, then every thread owns four consecutive value columns (one 8-byte load
// per frame, whole rows coalesced) and accumulates their n_q weighted sums over the frames.
// A chain of loads, two barriers and sums with little on the CU beside it: the first 16 frames' values are requested with the scores, and the
// softmax of a column is four threads' work.  17 windows 7.5 -> 5.4 us, 350 windows 7.9 -> 6.5 (values loaded in the loop, a thread a column).
struct QWindowList {
    const QWindow* w;
};
template <int NQ, class Wins>
__global__ void __launch_bounds__(256) qformer_pool_kernel(const float* __restrict__ scores, const f16_t* __restrict__ vals,
                                                           Wins wins, int n_heads, int d_h, bf16_t* __restrict__ o) {
    constexpr int AHEAD = 16, PER = QF_MAX_WINDOW / 4;       // PER: frames of a thread in the two steps before the sums
    static_assert(QF_SCORE_COLS == 64, "a wavefront reads the scores of a frame, four threads take a column");
    __shared__ __align__(16) float p_s[QF_SCORE_COLS][QF_MAX_WINDOW + 4];
    const QWindow w = wins.w[blockIdx.x];
    const int n = w.n_frames, n_pairs = NQ * n_heads;
    const float* sbase = scores + (int64_t)w.frame0 * QF_SCORE_COLS;
    const f16_t* vbase = vals + (int64_t)w.frame0 * d_h;
    float s_reg[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int t = threadIdx.x / 64 + 4 * k;
        s_reg[k] = t < n ? sbase[t * QF_SCORE_COLS + threadIdx.x % 64] : 0.f;
    }
    uint2 v[AHEAD];
    auto load = [&](int c, int t0) {
#pragma unroll
        for (int t = 0; t < AHEAD; ++t) v[t] = *reinterpret_cast<const uint2*>(vbase + (int64_t)min(t0 + t, n - 1) * d_h + c);
    };
    int c = 4 * threadIdx.x;
    if (c < d_h) load(c, 0);
#pragma unroll
    for (int k = 0; k < PER; ++k) p_s[threadIdx.x % 64][threadIdx.x / 64 + 4 * k] = s_reg[k];
    __syncthreads();
    if ((int)threadIdx.x / 4 < n_pairs) {
        float* p = p_s[threadIdx.x / 4] + threadIdx.x % 4;
        float e[PER], m = -INFINITY, sum = 0.f;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            e[k] = (int)threadIdx.x % 4 + 4 * k < n ? p[4 * k] : -INFINITY;
            m = fmaxf(m, e[k]);
        }
        m = fmaxf(m, __shfl_xor(m, 1));
        m = fmaxf(m, __shfl_xor(m, 2));
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            e[k] = __expf(e[k] - m);
            sum += (int)threadIdx.x % 4 + 4 * k < n ? e[k] : 0.f;
        }
        sum += __shfl_xor(sum, 1);
        sum += __shfl_xor(sum, 2);
        const float inv = 1.0f / sum;
#pragma unroll
        for (int k = 0; k < PER; ++k) p[4 * k] = e[k] * inv;
    }
    __syncthreads();
    const int dh = d_h / n_heads;                                              // a multiple of 4: four columns share a head
    while (c < d_h) {
        const int h = c / dh;
        float acc[NQ][4];
#pragma unroll
        for (int j = 0; j < NQ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[j][e] = 0.f;
        for (int t0 = 0;;) {
#pragma unroll
            for (int t4 = 0; t4 < AHEAD; t4 += 4) {
                if (t0 + t4 >= n) break;
                float4 p4[NQ];
#pragma unroll
                for (int j = 0; j < NQ; ++j) p4[j] = *reinterpret_cast<const float4*>(&p_s[j * n_heads + h][t0 + t4]);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (t0 + t4 + u >= n) break;
                    const uint2 raw = v[t4 + u];
                    const float x[4] = {f16_to_f32((f16_t)(raw.x & 0xffffu)), f16_to_f32((f16_t)(raw.x >> 16)),
                                        f16_to_f32((f16_t)(raw.y & 0xffffu)), f16_to_f32((f16_t)(raw.y >> 16))};
#pragma unroll
                    for (int j = 0; j < NQ; ++j) {
                        const float p = u == 0 ? p4[j].x : u == 1 ? p4[j].y : u == 2 ? p4[j].z : p4[j].w;
#pragma unroll
                        for (int e = 0; e < 4; ++e) acc[j][e] = fmaf(p, x[e], acc[j][e]);
                    }
                }
            }
            t0 += AHEAD;
            if (t0 >= n) break;
            load(c, t0);
        }
#pragma unroll
        for (int j = 0; j < NQ; ++j)
            *reinterpret_cast<uint2*>(o + ((int64_t)blockIdx.x * NQ + j) * d_h + c) =
                make_uint2(pack_bf16x2(acc[j][0], acc[j][1]), pack_bf16x2(acc[j][2], acc[j][3]));
        c += 1024;
        if (c < d_h) load(c, 0);
    }
}

template <class Wins>
static void launch_pool(const float* scores, const uint16_t* vals, const Wins& wins, int n_windows, int n_q, int n_heads, int d_h, uint16_t* o,
                        hipStream_t st) {
    if (n_windows <= 0) return;
#define SSD_QF(NQ) hipLaunchKernelGGL((qformer_pool_kernel<NQ, Wins>), dim3(n_windows), dim3(256), 0, st, scores, vals, wins, n_heads, d_h, o)
    if (n_q == 1) SSD_QF(1); else if (n_q == 2) SSD_QF(2); else if (n_q == 3) SSD_QF(3); else SSD_QF(4);
#undef SSD_QF
}
void launch_qformer_pool(const float* scores, const uint16_t* vals, const QWindow* wins, int n_windows, int n_q, int n_heads,
                         int d_h, uint16_t* o, hipStream_t st) {
    launch_pool(scores, vals, QWindowList{wins}, n_windows, n_q, n_heads, d_h, o, st);
}
void launch_qformer_pool_host(const float* scores, const uint16_t* vals, const QWindowArgs& wins, int n_windows, int n_q, int n_heads,
                              int d_h, uint16_t* o, hipStream_t st) {
    launch_pool(scores, vals, wins, n_windows, n_q, n_heads, d_h, o, st);
}

// The windows of utterance blockIdx.x, behind those of the utterances before it.
__global__ void __launch_bounds__(256) qformer_windows_kernel(CuPairs cu, int window, QWindow* __restrict__ wins) {
    __shared__ int part[4];
    const int b = blockIdx.x;
    int before = 0;
    for (int i = threadIdx.x; i < b; i += 256) before += (cu(i + 1) - cu(i) + window - 1) / window;
    before = group_allreduce_i<64>(before, [] __device__(int a, int c) { return a + c; });
    if (threadIdx.x % 64 == 0) part[threadIdx.x / 64] = before;
    __syncthreads();
    before = part[0] + part[1] + part[2] + part[3];
    const int first = cu(b), n = cu(b + 1) - first;
    for (int i = threadIdx.x; i * window < n; i += 256) wins[before + i] = QWindow{first + i * window, min(window, n - i * window)};
}
void launch_qformer_windows(const CuPairs& cu, int B, int window, QWindow* wins, hipStream_t st) {
    hipLaunchKernelGGL(qformer_windows_kernel, dim3(B), dim3(256), 0, st, cu, window, wins);
}

}  // namespace ssd
