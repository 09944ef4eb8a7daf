// All-fp32 decoder kernels (model dtype SSD_F32).  Everything contracts on v_mfma_f32_16x16x4_f32: fp32
// operands, fp32 products and sums, no rounding in between.
//
// What bounds this path is not arithmetic (a 285-row pass of the two-layer decoder is 0.94 GFLOP, 6 us of the
// matrix cores) but the number of dependent launches and the latency inside each of them, so a layer is five
// kernels (RMSNorm, rotary embedding, SiLU and the K/V-cache rows live in the GEMMs around them), and every
// kernel splits its reduction over the four wavefronts of a workgroup to keep the serial part short.
//
// Operand layout used throughout: an MFMA takes from lane (x = lane % 16, kq = lane / 16) ONE k of row / column x.
// Which k is free as long as both operands agree, so a lane loads the float4 at k = 16 t + 4 kq and feeds its four
// components to four MFMAs: 16 k per load, every load 16 rows x 64 contiguous bytes, no LDS staging.
// The instruction is issued with the weight (or key, or V^T) fragment as the row operand: a lane then holds one
// row x of the result and four consecutive columns 4 kq + r.
#include "device_utils.h"
#include "ssd_internal.h"

namespace ssd {

typedef float f32x4v_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4v_t mfma_f32_k16(const float4& w, const float4& a, f32x4v_t c) {
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(w.x, a.x, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(w.y, a.y, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x4f32(w.z, a.z, c, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(w.w, a.w, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------------------------
// C = A W^T for 16 RB rows x 16 PB column PAIRS per workgroup; the end of the tile gets both members of a pair in one thread:
//   F32_QKV      (i, i + head_dim/2) of a rotary head, or (c, c + d_kv/2) of v: rotation, store, K/V-cache row
//   F32_SWIGLU   gate and up of one hidden unit: h = silu(gate) * up
//   F32_RESIDUAL (no pairs: single columns) x += acc
// QKV and SWIGLU take RMSNorm(x) as A: the gain is applied to the fragments, the sum of squares of the row falls out
// of the same loads, and 1/rms multiplies the finished sums (out = inv * sum_k (x_k g_k) w_k).
// The NW wavefronts split K; their partial tiles are added through LDS in wavefront order.
// K % 16 == 0; M, the pair count and head_dim are arbitrary (rows and columns beyond the end are clamped on load).
// What the ends read (rotary entries, old residual values) is requested before the products.
enum F32Pairs { F32_QKV, F32_SWIGLU, F32_RESIDUAL };
struct F32GemmArgs {
    const float* A; const float* W; const float* gain; float* out;
    int M, K, ldo, n_pairs; float eps;
    const int32_t* a_rows; const int32_t* o_rows;                               // rows of A / of out that are taken (NULL: all in order)
    int half, d_rot, d_q, d_kv; const int32_t* pos; const float2* rope_tab;     // QKV only
    const int32_t* row_slot; float* kc; float* vc;
};
template <int EPI>
__device__ __forceinline__ void pair_columns(const F32GemmArgs& g, int p, int& c0, int& c1, int& i_rot) {
    i_rot = -1;
    if constexpr (EPI == F32_QKV) {
        const int rot = g.d_rot / 2;
        if (p < rot) {
            i_rot = p % g.half;
            c0 = (p / g.half) * 2 * g.half + i_rot;
            c1 = c0 + g.half;
        } else {
            c0 = g.d_rot + (p - rot);
            c1 = c0 + g.d_kv / 2;
        }
    } else if constexpr (EPI == F32_SWIGLU) {
        c0 = p;
        c1 = g.n_pairs + p;
    } else {
        c0 = c1 = p;
    }
}

template <int EPI, int NW, int RB, int PB>
__global__ void __launch_bounds__(64 * NW) gemm_f32_kernel(F32GemmArgs g) {
    constexpr bool NORM = EPI != F32_RESIDUAL;
    constexpr int MEM = EPI == F32_RESIDUAL ? 1 : 2;         // members of a pair
    constexpr int UNITS = 128 * RB * PB;                     // ends of the tile: two pairs of one row each
    constexpr int PER = (UNITS + 64 * NW - 1) / (64 * NW);   // per thread
    __shared__ float4 red[NW][RB][PB * MEM][64];             // [wavefront][row block][column block][lane]
    __shared__ float ssl[NW][16 * RB];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64, x = lane % 16, kq = lane / 16;
    const int m0 = blockIdx.y * 16 * RB, p0 = blockIdx.x * 16 * PB;
    // what the ends read is requested before the products
    struct End { int bi, bj, ln, part, r, row; };
    auto end_of = [&](int k) {
        const int u = (k * 64 * NW + threadIdx.x) % UNITS, slot = u / 2, blk = slot / 64;
        End e{blk / PB, blk % PB, slot % 64, u % 2, 0, 0};
        e.r = 16 * e.bi + e.ln % 16;
        e.row = m0 + e.r;
        return e;
    };
    float2 e_old[PER][2];                                    // QKV: (cos, sin); RESIDUAL: the old value
    int e_slot[PER], e_out[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const End e = end_of(k);
        const int e_row = min(e.row, g.M - 1);
        e_out[k] = e_row;
        if constexpr (EPI == F32_RESIDUAL)
            if (g.o_rows) e_out[k] = g.o_rows[e_row];
        int e_pos = 0;
        if constexpr (EPI == F32_QKV) {
            e_pos = g.pos[e_row];
            e_slot[k] = g.row_slot ? g.row_slot[e_row] : -1;
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            int c0, c1, rot;
            pair_columns<EPI>(g, min(p0 + 16 * e.bj + 4 * (e.ln / 16) + 2 * e.part + c, g.n_pairs - 1), c0, c1, rot);
            if constexpr (EPI == F32_QKV) e_old[k][c] = rot >= 0 ? g.rope_tab[(int64_t)e_pos * g.half + rot] : make_float2(1.f, 0.f);
            if constexpr (EPI == F32_RESIDUAL) e_old[k][c].x = g.out[(int64_t)e_out[k] * g.ldo + c0];
        }
    }
    const float* a_row[RB];
    const float* w_row[PB * MEM];
#pragma unroll
    for (int i = 0; i < RB; ++i) {
        const int row = min(m0 + 16 * i + x, g.M - 1);
        a_row[i] = g.A + (int64_t)(g.a_rows ? g.a_rows[row] : row) * g.K + 4 * kq;
    }
#pragma unroll
    for (int j = 0; j < PB; ++j) {
        int c[2], unused;
        pair_columns<EPI>(g, min(p0 + 16 * j + x, g.n_pairs - 1), c[0], c[1], unused);
#pragma unroll
        for (int q = 0; q < MEM; ++q) w_row[MEM * j + q] = g.W + (int64_t)c[q] * g.K + 4 * kq;
    }
    f32x4v_t acc[RB][PB * MEM] = {};
    float ss[RB] = {};
    const int KT = g.K / 16, t0 = KT * wave / NW, t1 = KT * (wave + 1) / NW;
    constexpr int U = RB + PB * MEM > 4 ? 2 : 4;             // K steps in flight
    for (int t = t0; t < t1; t += U) {
        float4 a[U][RB], w[U][PB * MEM], gn[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = 16 * min(t + u, t1 - 1);       // a step beyond the end is loaded and left out
#pragma unroll
            for (int i = 0; i < RB; ++i) a[u][i] = *reinterpret_cast<const float4*>(a_row[i] + k);
#pragma unroll
            for (int j = 0; j < PB * MEM; ++j) w[u][j] = *reinterpret_cast<const float4*>(w_row[j] + k);
            if constexpr (NORM) gn[u] = *reinterpret_cast<const float4*>(g.gain + k + 4 * kq);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (t + u >= t1) break;
#pragma unroll
            for (int i = 0; i < RB; ++i) {
                float4 v = a[u][i];
                if constexpr (NORM) {
                    ss[i] += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
                    v = make_float4(v.x * gn[u].x, v.y * gn[u].y, v.z * gn[u].z, v.w * gn[u].w);
                }
#pragma unroll
                for (int j = 0; j < PB * MEM; ++j) acc[i][j] = mfma_f32_k16(w[u][j], v, acc[i][j]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < RB; ++i) {
#pragma unroll
        for (int j = 0; j < PB * MEM; ++j) red[wave][i][j][lane] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
        if constexpr (NORM) {
            float s = ss[i];
            s += __shfl_xor(s, 16);
            s += __shfl_xor(s, 32);
            if (kq == 0) ssl[wave][16 * i + x] = s;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const End e = end_of(k);
        if (e.row >= g.M || k * 64 * NW + (int)threadIdx.x >= UNITS) continue;
        float v[2][2] = {};
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int q = 0; q < MEM; ++q) {
                const float2 t = reinterpret_cast<const float2*>(&red[w][e.bi][MEM * e.bj + q][e.ln])[e.part];
                v[q][0] += t.x;
                v[q][1] += t.y;
            }
        if constexpr (NORM) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < NW; ++w) s += ssl[w][e.r];
            const float inv = 1.0f / sqrtf(s / (float)g.K + g.eps);
#pragma unroll
            for (int q = 0; q < MEM; ++q) { v[q][0] *= inv; v[q][1] *= inv; }
        }
        float* o = g.out + (int64_t)e_out[k] * g.ldo;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int p = p0 + 16 * e.bj + 4 * (e.ln / 16) + 2 * e.part + c;
            if (p >= g.n_pairs) continue;
            const float a = v[0][c], b = v[1][c];
            int c0, c1, i_rot;
            pair_columns<EPI>(g, p, c0, c1, i_rot);
            if constexpr (EPI == F32_SWIGLU) {
                o[p] = a / (1.0f + expf(-a)) * b;
            } else if constexpr (EPI == F32_RESIDUAL) {
                o[p] = e_old[k][c].x + a;
            } else {
                const bool rot = i_rot >= 0;                 // (columns of v come with the identity rotation)
                const float2 cs = e_old[k][c];
                const float o0 = rot ? a * cs.x - b * cs.y : a, o1 = rot ? b * cs.x + a * cs.y : b;
                o[c0] = o0;
                o[c1] = o1;
                if (e_slot[k] >= 0 && c0 >= g.d_q) {         // a pair lies inside q, k or v
                    float* dst = (rot ? g.kc : g.vc) + (int64_t)e_slot[k] * g.d_kv;
                    const int first = rot ? g.d_q : g.d_rot;
                    dst[c0 - first] = o0;
                    dst[c1 - first] = o1;
                }
            }
        }
    }
}

// Tile (row blocks of 16 x blocks of 16 pairs, single columns for RESIDUAL).  A workgroup pulls its operand rows through one CU's load
// path, and that is what a small launch waits for: the smallest tile that still runs in one round.  Two-layer decoder (K 256 / 1024), us of
// a launch, tiles of 32 rows x 16 pairs / as chosen: 64 rows QKV 6.1 / 4.6, O 4.8 / 3.6, gate/up 5.6 / 4.1, down 10.4 / 6.0 (also at 256
// rows); K = 1024 / 4096 at 64 rows O 10.4 / 6.2, down 32 / 16.5.  Beyond one round larger tiles load less per product: for pairs
// 2 x 2 or 2 x 1 by rounds times a tile's loads and products (14 to 8): gate/up of 2000 rows 35 / 30, QKV of 1024 rows (384 of the
// 2 x 2 tiles, one and a half rounds) 11.1 as 2 x 1, 13.1 as 2 x 2.  Above K = 512 those that are left as 2 x 1, and the largest of
// RESIDUAL, have K over eight wavefronts (down of 500 rows, K = 2048: 18.4 / 20.4 with four).
template <int EPI, int NW, int RB, int PB>
static void launch_pairs_tile(const F32GemmArgs& g, hipStream_t st) {
    const dim3 grid((g.n_pairs + 16 * PB - 1) / (16 * PB), (g.M + 16 * RB - 1) / (16 * RB));
    hipLaunchKernelGGL((gemm_f32_kernel<EPI, NW, RB, PB>), grid, dim3(64 * NW), 0, st, g);
}
template <int EPI>
static void launch_pairs(const F32GemmArgs& g, hipStream_t st) {
    if (g.M <= 0) return;
    auto tiles = [&](int rb, int pb) { return (int64_t)((g.M + 16 * rb - 1) / (16 * rb)) * ((g.n_pairs + 16 * pb - 1) / (16 * pb)); };
    auto rounds = [&](int rb, int pb) { return (tiles(rb, pb) + 255) / 256; };
    if (tiles(1, 1) <= 256) { launch_pairs_tile<EPI, 4, 1, 1>(g, st); return; }
    if (tiles(1, 2) <= 256) { launch_pairs_tile<EPI, 4, 1, 2>(g, st); return; }
    if constexpr (EPI == F32_RESIDUAL) {
        if (g.K > 512) launch_pairs_tile<EPI, 8, 2, 2>(g, st);
        else launch_pairs_tile<EPI, 4, 2, 2>(g, st);
    } else {
        if (14 * rounds(2, 2) <= 8 * rounds(2, 1) && (g.K <= 512 || rounds(2, 2) >= 2)) launch_pairs_tile<EPI, 4, 2, 2>(g, st);
        else if (g.K > 512) launch_pairs_tile<EPI, 8, 2, 1>(g, st);
        else launch_pairs_tile<EPI, 4, 2, 1>(g, st);
    }
}
void launch_gemm_f32_qkv(const float* x, const float* gain, float eps, const float* Wqkv, float* qkv, const int32_t* pos,
                         const float* rope_tab, int M, int d_model, int d_q, int d_kv, int head_dim, const int32_t* row_slot,
                         float* kc, float* vc, hipStream_t st) {
    F32GemmArgs g{x, Wqkv, gain, qkv, M, d_model, d_q + 2 * d_kv, (d_q + 2 * d_kv) / 2, eps, nullptr, nullptr, head_dim / 2, d_q + d_kv,
                  d_q, d_kv, pos, reinterpret_cast<const float2*>(rope_tab), row_slot, kc, vc};
    launch_pairs<F32_QKV>(g, st);
}
void launch_gemm_f32_swiglu(const float* x, const float* gain, float eps, const float* Wgu, float* h, int M, int d_ff, int d_model,
                            const int32_t* x_rows, hipStream_t st) {
    F32GemmArgs g{x, Wgu, gain, h, M, d_model, d_ff, d_ff, eps, x_rows, nullptr, 1, 0, 0, 0, nullptr, nullptr, nullptr, nullptr, nullptr};
    launch_pairs<F32_SWIGLU>(g, st);
}
void launch_gemm_f32_residual(const float* A, const float* W, float* x, int M, int N, int K, const int32_t* a_rows, const int32_t* x_rows,
                              hipStream_t st) {
    F32GemmArgs g{A, W, nullptr, x, M, K, N, N, 0.f, a_rows, x_rows, 1, 0, 0, 0, nullptr, nullptr, nullptr, nullptr, nullptr};
    launch_pairs<F32_RESIDUAL>(g, st);
}

// ---------------------------------------------------------------------------------------------
// Causal attention: a workgroup owns 16 queries of one head, its four wavefronts take every fourth block of 16 keys
// (a context of 70-380 positions is then 2-6 blocks per wavefront) and merge through LDS.
// S^T = K Q^T leaves a lane with query x and keys 4 kq + r, which is the operand that O^T += V^T P^T wants: the
// probabilities go from one product to the next in registers.
// qkv rows: [q heads | k heads | v heads]; head_dim <= 16 NDB and a multiple of 4.
// 20.4 -> 6.8 us at 285 rows (a wavefront per query read each key row from one lane and the values one key at a time);
// the look at the diagonal block's values is 0.1 us of that launch.
template <int NDB>
__global__ void __launch_bounds__(256) attn_f32_kernel(const float* __restrict__ qkv, float* __restrict__ out,
                                                       const AttnTile* __restrict__ tiles, int n_q_heads,
                                                       int n_kv_heads, int head_dim) {
    __shared__ float4 o_s[4][NDB][64];
    __shared__ float m_s[4][16], l_s[4][16];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64, x = lane % 16, kq = lane / 16;
    const AttnTile t = tiles[blockIdx.x];
    const int h = blockIdx.y, kvh = h / (n_q_heads / n_kv_heads);
    const int d_q = n_q_heads * head_dim, d_kv = n_kv_heads * head_dim, stride = d_q + 2 * d_kv;
    const int n = t.seq_len, qpos = t.q_start + x;
    const float scale = 1.0f / sqrtf((float)head_dim);
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    const float* q = qkv + (int64_t)(t.seq_start + min(qpos, n - 1)) * stride + h * head_dim;
    const float* kbase = qkv + (int64_t)t.seq_start * stride + d_q + kvh * head_dim;
    const float* vbase = kbase + d_kv;
    float4 qf[NDB];
#pragma unroll
    for (int c = 0; c < NDB; ++c) qf[c] = 16 * c + 4 * kq < head_dim ? *reinterpret_cast<const float4*>(q + 16 * c + 4 * kq) : zero;
    float m = -INFINITY, l = 0.f;
    f32x4v_t o[NDB] = {};
    const int last = min(t.q_start + 15, n - 1);
    for (int kb = wave; kb * 16 <= last; kb += 4) {
        const float* kr = kbase + (int64_t)min(kb * 16 + x, n - 1) * stride;
        float4 kf[NDB];
        float vf[NDB][4];
#pragma unroll
        for (int c = 0; c < NDB; ++c) kf[c] = 16 * c + 4 * kq < head_dim ? *reinterpret_cast<const float4*>(kr + 16 * c + 4 * kq) : zero;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float* vr = vbase + (int64_t)min(kb * 16 + 4 * kq + r, n - 1) * stride;
#pragma unroll
            for (int c = 0; c < NDB; ++c) vf[c][r] = 16 * c + x < head_dim ? vr[16 * c + x] : 0.f;
        }
        f32x4v_t s = {};
#pragma unroll
        for (int c = 0; c < NDB; ++c) s = mfma_f32_k16(kf[c], qf[c], s);
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[r] = kb * 16 + 4 * kq + r <= qpos ? s[r] * scale : -INFINITY;
            mx = fmaxf(mx, s[r]);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m, mx);
        const float ref = m_new == -INFINITY ? 0.f : m_new;   // no key of this query in the blocks so far
        const float alpha = expf(m - ref);
        float p[4], ps = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) { p[r] = expf(s[r] - ref); ps += p[r]; }
        ps += __shfl_xor(ps, 16);
        ps += __shfl_xor(ps, 32);
        l = l * alpha + ps;
        m = m_new;
#pragma unroll
        for (int c = 0; c < NDB; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) o[c][r] *= alpha;
        // In the block of the diagonal the matrix product multiplies values a query must not see by probabilities of 0,
        // which is only nothing while they are finite.
        float zero_sum = 0.f;
        if (kb * 16 >= t.q_start) {
#pragma unroll
            for (int c = 0; c < NDB; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) zero_sum = fmaf(vf[c][r], 0.f, zero_sum);
        }
        if (__any(zero_sum != 0.f)) {                         // an infinite or NaN value: visible keys only, one at a time
            for (int j = 0; j < 16; ++j) {                    // in the order of the matrix product
                const int r = j / 4, q = j % 4, key = kb * 16 + 4 * q + r;
                const float pj = __shfl(r == 0 ? p[0] : r == 1 ? p[1] : r == 2 ? p[2] : p[3], 16 * q + x);
                if (key > qpos) continue;
                const float* vr = vbase + (int64_t)min(key, n - 1) * stride + 4 * kq;
#pragma unroll
                for (int c = 0; c < NDB; ++c) {
                    if (16 * c + 4 * kq >= head_dim) continue;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[c][e] = fmaf(pj, vr[16 * c + e], o[c][e]);
                }
            }
        } else {
#pragma unroll
            for (int c = 0; c < NDB; ++c)
#pragma unroll
                for (int r = 0; r < 4; ++r) o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[c][r], p[r], o[c], 0, 0, 0);
        }
    }
#pragma unroll
    for (int c = 0; c < NDB; ++c) o_s[wave][c][lane] = make_float4(o[c][0], o[c][1], o[c][2], o[c][3]);
    if (kq == 0) { m_s[wave][x] = m; l_s[wave][x] = l; }
    __syncthreads();
    if (qpos >= n) return;
    float mt = m_s[0][x];                                    // finite: key 0 is in block 0
#pragma unroll
    for (int w = 1; w < 4; ++w) mt = fmaxf(mt, m_s[w][x]);
    float f[4], lt = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        f[w] = expf(m_s[w][x] - mt);                         // 0 for a wavefront without a key
        lt = fmaf(l_s[w][x], f[w], lt);
    }
    const float inv = 1.0f / lt;
    for (int c = wave; c < NDB; c += 4) {
        const int d = 16 * c + 4 * kq;
        if (d >= head_dim) continue;
        float4 r = zero;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float4 v = o_s[w][c][lane];
            r.x = fmaf(v.x, f[w], r.x); r.y = fmaf(v.y, f[w], r.y); r.z = fmaf(v.z, f[w], r.z); r.w = fmaf(v.w, f[w], r.w);
        }
        *reinterpret_cast<float4*>(out + (int64_t)(t.seq_start + qpos) * d_q + h * head_dim + d) = make_float4(r.x * inv, r.y * inv, r.z * inv, r.w * inv);
    }
}

void launch_attn_f32(const float* qkv, float* out, const AttnTile* tiles, int n_tiles, int n_q_heads, int n_kv_heads,
                     int head_dim, hipStream_t st) {
    if (n_tiles <= 0) return;
    if (head_dim <= 64)
        hipLaunchKernelGGL(attn_f32_kernel<4>, dim3(n_tiles, n_q_heads), dim3(256), 0, st, qkv, out, tiles, n_q_heads, n_kv_heads, head_dim);
    else
        hipLaunchKernelGGL(attn_f32_kernel<8>, dim3(n_tiles, n_q_heads), dim3(256), 0, st, qkv, out, tiles, n_q_heads, n_kv_heads, head_dim);
}

// ---------------------------------------------------------------------------------------------
// One query row per utterance against its cached rows (the last of which is the query token's own).  A workgroup is
// one (utterance, head): sixteen groups of 16 lanes, each with an online softmax of its own over every sixteenth key
// (a lane holds four dims of a row, eight above head_dim 64; a group reads a key row as one contiguous piece), four
// keys in flight per group; the groups are merged through LDS at the end.  head_dim <= 128, a multiple of 4.
__global__ void __launch_bounds__(256) decode_attn_f32_kernel(const float* __restrict__ qkv, const float* __restrict__ kc,
                                                              const float* __restrict__ vc, const int32_t* __restrict__ kv_start,
                                                              const int32_t* __restrict__ n_ctx, int n_q_heads, int n_kv_heads,
                                                              int head_dim, float* __restrict__ out) {
    __shared__ float o_s[16][128];
    __shared__ float m_s[16], l_s[16];
    const int dc = threadIdx.x % 16, grp = threadIdx.x / 16;
    const int b = blockIdx.x, h = blockIdx.y, kvh = h / (n_q_heads / n_kv_heads);
    const int d_q = n_q_heads * head_dim, d_kv = n_kv_heads * head_dim;
    const int n = n_ctx[b];
    const float scale = 1.0f / sqrtf((float)head_dim);
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    const bool live[2] = {dc * 4 < head_dim, 64 + dc * 4 < head_dim};
    const float* q = qkv + (int64_t)b * (d_q + 2 * d_kv) + h * head_dim + dc * 4;
    const float* kbase = kc + (int64_t)kv_start[b] * d_kv + kvh * head_dim + dc * 4;
    const float* vbase = vc + (int64_t)kv_start[b] * d_kv + kvh * head_dim + dc * 4;
    float4 qf[2], o[2] = {zero, zero};
#pragma unroll
    for (int e = 0; e < 2; ++e) qf[e] = live[e] ? *reinterpret_cast<const float4*>(q + 64 * e) : zero;
    float m = -INFINITY, l = 0.f;
    constexpr int U = 4;
    for (int k0 = grp; k0 < n; k0 += 16 * U) {
        float4 kr[U][2], vr[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t off = (int64_t)min(k0 + 16 * u, n - 1) * d_kv;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                kr[u][e] = live[e] ? *reinterpret_cast<const float4*>(kbase + off + 64 * e) : zero;
                vr[u][e] = live[e] ? *reinterpret_cast<const float4*>(vbase + off + 64 * e) : zero;
            }
        }
        float s[U], m_new = m;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float acc = 0.f;
#pragma unroll
            for (int e = 0; e < 2; ++e)
                acc += qf[e].x * kr[u][e].x + qf[e].y * kr[u][e].y + qf[e].z * kr[u][e].z + qf[e].w * kr[u][e].w;
            acc = group_allreduce<16>(acc, OpSum()) * scale;
            s[u] = k0 + 16 * u < n ? acc : -INFINITY;
            m_new = fmaxf(m_new, s[u]);
        }
        const float alpha = expf(m - m_new);                  // 0 on the first trip
        l *= alpha;
#pragma unroll
        for (int e = 0; e < 2; ++e) o[e] = make_float4(o[e].x * alpha, o[e].y * alpha, o[e].z * alpha, o[e].w * alpha);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const float p = expf(s[u] - m_new);
            l += p;
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                o[e].x = fmaf(p, vr[u][e].x, o[e].x); o[e].y = fmaf(p, vr[u][e].y, o[e].y);
                o[e].z = fmaf(p, vr[u][e].z, o[e].z); o[e].w = fmaf(p, vr[u][e].w, o[e].w);
            }
        }
        m = m_new;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) *reinterpret_cast<float4*>(&o_s[grp][64 * e + dc * 4]) = o[e];
    if (dc == 0) { m_s[grp] = m; l_s[grp] = l; }
    __syncthreads();
    const int d = threadIdx.x;
    if (d >= head_dim) return;
    float mt = m_s[0];                                        // finite: key 0 belongs to group 0
#pragma unroll
    for (int w = 1; w < 16; ++w) mt = fmaxf(mt, m_s[w]);
    float lt = 0.f, r = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        const float f = expf(m_s[w] - mt);                    // 0 for a group without a key
        lt = fmaf(l_s[w], f, lt);
        r = fmaf(o_s[w][d], f, r);
    }
    out[(int64_t)b * d_q + h * head_dim + d] = r / lt;
}

void launch_decode_attn_f32(const float* qkv, const float* kc, const float* vc, const int32_t* kv_start, const int32_t* n_ctx, int Br,
                            int n_q_heads, int n_kv_heads, int head_dim, float* out, hipStream_t st) {
    if (Br <= 0) return;
    hipLaunchKernelGGL(decode_attn_f32_kernel, dim3(Br, n_q_heads), dim3(256), 0, st, qkv, kc, vc, kv_start, n_ctx, n_q_heads,
                       n_kv_heads, head_dim, out);
}

// ---------------------------------------------------------------------------------------------
// LM head (Eq. 5's likelihoods): a workgroup forms the logits of 32 rows x 64 vocabulary entries (K split over the
// wavefronts as above), reduces them to (max, sum exp) and the lowest index of the maximum per row, and writes the
// target's logit where it falls into its columns; launch_lmhead_finalize merges the column groups.  The logits stay
// in LDS.  Vocabulary and row count are arbitrary, d a multiple of 16.
// 1194 -> 9.0 us at 125 rows x 4096 entries: a workgroup per row walked the whole vocabulary with a six-step
// cross-lane sum per logit, i.e. 125 workgroups with 1024 dependent reductions each.
// Hidden rows and head are the caller's own buffers and may start at any float: 16-byte loads that are aligned to 4.
typedef float f32x4u_t __attribute__((ext_vector_type(4), aligned(4)));
__device__ __forceinline__ float4 load4_unaligned(const float* p) {
    const f32x4u_t v = *reinterpret_cast<const f32x4u_t*>(p);
    return make_float4(v.x, v.y, v.z, v.w);
}
int lmhead_f32_groups(int vocab) { return (vocab + 63) / 64; }
__global__ void __launch_bounds__(256) lmhead_f32_kernel(const float* __restrict__ hv, const float* __restrict__ w_lm,
                                                         const int32_t* __restrict__ targets, int Mv, int d, int vocab,
                                                         float2* __restrict__ part_ms, float* __restrict__ tgt_logit,
                                                         int2* __restrict__ part_arg) {
    __shared__ float4 red[4][8][64];
    __shared__ float z_s[32][64 + 4];
    const int lane = threadIdx.x % 64, wave = threadIdx.x / 64, x = lane % 16, kq = lane / 16;
    const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 64;
    const float *a_row[2], *w_row[4];
#pragma unroll
    for (int i = 0; i < 2; ++i) a_row[i] = hv + (int64_t)min(m0 + 16 * i + x, Mv - 1) * d + 4 * kq;
#pragma unroll
    for (int j = 0; j < 4; ++j) w_row[j] = w_lm + (int64_t)min(n0 + 16 * j + x, vocab - 1) * d + 4 * kq;
    f32x4v_t acc[2][4] = {};
    const int KT = d / 16, t0 = KT * wave / 4, t1 = KT * (wave + 1) / 4;
    constexpr int U = 4;
    for (int t = t0; t < t1; t += U) {
        float4 a[U][2], w[U][4];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t k = 16 * min(t + u, t1 - 1);
#pragma unroll
            for (int i = 0; i < 2; ++i) a[u][i] = load4_unaligned(a_row[i] + k);
#pragma unroll
            for (int j = 0; j < 4; ++j) w[u][j] = load4_unaligned(w_row[j] + k);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (t + u >= t1) break;
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = mfma_f32_k16(w[u][j], a[u][i], acc[i][j]);
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) red[wave][4 * i + j][lane] = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
    __syncthreads();
    for (int s = threadIdx.x; s < 512; s += 256) {
        const int blk = s / 64, ln = s % 64;
        float4 v = red[0][blk][ln];
#pragma unroll
        for (int w = 1; w < 4; ++w) {
            const float4 t = red[w][blk][ln];
            v.x += t.x; v.y += t.y; v.z += t.z; v.w += t.w;
        }
        *reinterpret_cast<float4*>(&z_s[16 * (blk / 4) + ln % 16][16 * (blk % 4) + 4 * (ln / 16)]) = v;
    }
    __syncthreads();
    // eight lanes per row, eight logits each (columns e * 8 + q: consecutive lanes read consecutive floats)
    const int r = threadIdx.x / 8, q = threadIdx.x % 8, row = m0 + r;
    const int n_cols = min(64, vocab - n0);
    float m = -INFINITY, z[8];
    int arg = 0x7fffffff;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        z[e] = 8 * e + q < n_cols ? z_s[r][8 * e + q] : -INFINITY;
        if (z[e] > m) { m = z[e]; arg = n0 + 8 * e + q; }
    }
    float mt = m;
#pragma unroll
    for (int o = 1; o < 8; o *= 2) mt = fmaxf(mt, __shfl_xor(mt, o));
    float sum = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) sum += expf(z[e] - mt);
    arg = m == mt ? arg : 0x7fffffff;
#pragma unroll
    for (int o = 1; o < 8; o *= 2) {
        sum += __shfl_xor(sum, o);
        arg = min(arg, __shfl_xor(arg, o));
    }
    if (row >= Mv || q != 0) return;
    const int64_t at = (int64_t)blockIdx.x * Mv + row;
    part_ms[at] = make_float2(mt, sum);
    part_arg[at] = make_int2(__float_as_int(mt), arg);
    const int tgt = min(max(targets[row], 0), vocab - 1) - n0;
    if (tgt >= 0 && tgt < 64) tgt_logit[row] = z_s[r][tgt];
}

void launch_lmhead_f32(const float* hv, const float* w_lm, const int32_t* targets, int Mv, int d, int vocab, float2* part_ms,
                       float* tgt_logit, int2* part_arg, hipStream_t st) {
    if (Mv <= 0) return;
    hipLaunchKernelGGL(lmhead_f32_kernel, dim3(lmhead_f32_groups(vocab), (Mv + 31) / 32), dim3(256), 0, st, hv, w_lm, targets, Mv, d,
                       vocab, part_ms, tgt_logit, part_arg);
}

}  // namespace ssd
