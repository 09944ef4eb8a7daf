// Auto-regressive fallback (Sec. 2.3, Eq. 6): kernels that exist only for the token-by-token
// continuation from the accepted prefix: attention of ONE new query row per utterance against its cached
// rows (16-bit models, head_dim 128; the fp32 model's is in f32_path.hip).
// Everything else of a decode step reuses the verification kernels on a batch of Br rows
// (RMSNorm, skinny weight-streaming GEMMs with split-K, LM head with argmax).
#include "device_utils.h"
#include "ssd_internal.h"

namespace ssd {

// eight 16-bit operand patterns (IEEE half or bfloat16) as fp32
template <bool BF>
__device__ __forceinline__ void unpack8(const uint4& w, float (&v)[8]) {
    if constexpr (BF) {
        v[0] = bf16_lo(w.x); v[1] = bf16_hi(w.x); v[2] = bf16_lo(w.y); v[3] = bf16_hi(w.y);
        v[4] = bf16_lo(w.z); v[5] = bf16_hi(w.z); v[6] = bf16_lo(w.w); v[7] = bf16_hi(w.w);
    } else {
        typedef _Float16 h8 __attribute__((ext_vector_type(8)));
        const h8 a = __builtin_bit_cast(h8, w);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = (float)a[e];
    }
}

// head_dim 128: a workgroup is DEC_WAVES wavefronts and serves one (utterance, G query heads of one K/V head): every
// cached row is read once for its G heads (one workgroup per query head read each row G times, from whichever XCD it
// ran on).  Per launch, before and after: 13.2 -> 9.8 us at 27 utterances of 16 heads over 8; at 70 utterances of 24 over 8
// 21.6 -> 20.7 us, the QKV splits now added here included (206 registers: two workgroups per CU, 560 of them).  Lane = (key group kg
// of 4, chunk dc of 8 dims).  A block of DEC_KEYS keys is 8 loads of K and 8 of V per lane (the rows are 256 bytes, a
// 16-lane group reads one row); a score is a 16-lane reduction, the softmax statistics are reduced over the four key
// groups, and P.V accumulates in the lane, reduced over the key groups at the end.  The wavefronts take the blocks of
// a context in turn and merge their (max, sum, output) triples through LDS: the blocks are loaded at once instead of
// one after the other, and the next block's keys are requested as soon as this block's scores are known.
constexpr int DEC_WAVES = 4;
constexpr int DEC_KEYS = 32;
constexpr int DEC_MAX_HEADS = 3;                             // one wavefront of the fused variant per head and one for the new k / v row

// Fused variant: the QKV projection of the step has been left as K-split partial sums
// part[split][row][packed column] (fp32, packed column order of the fused QKV weight: inside a head the
// rotary pairs (i, i+64) sit 32 columns apart in 64-column groups, V columns are in natural order).
// The kernel adds the splits, rotates q and the new k, appends the new k / v row to the cache (first query
// head of each K/V group) and treats that row as the last key without reading it back.
// a value as the cache / the next kernel will see it: rounded to the operand type, saturated for IEEE half
template <bool BF> __device__ __forceinline__ float round_like_stored(float v, bool& bad) {
    if constexpr (BF) return bf16_to_f32(f32_to_bf16(v));
    else return f16_to_f32(f32_to_f16_sat(v, bad));
}
template <bool BF> __device__ __forceinline__ uint32_t pack2_sat(float lo, float hi, bool& bad) {
    if constexpr (BF) return pack_bf16x2(lo, hi);
    else return pack_f16x2_sat(lo, hi, bad);
}

struct DecodeFused {
    const float* part; int n_splits; int64_t split_stride;    // split_stride = rows * (d_q + 2 d_kv)
    const float2* rope_tab;                                   // [position][64] (cos, sin)
    f16_t* kc_w; f16_t* vc_w;                                 // writable views of the cache
    int32_t* flags;                                           // sticky device flags (SSD_FLAG_ACT_OVERFLOW on a saturated store)
    // The new row's position is the number of rows its utterance has in the cache (cache row i of an
    // utterance is position i), and its slot is kv_start + that number: no further index arrays.
};
// Sum over the splits of eight consecutive packed columns starting at `col` of row b.  Key group kg adds splits kg and
// kg + 4 (SKINNY_MAX_SPLITS is 8), the groups are added over the wavefront: one round trip whatever the split count.
struct SplitSum { float v[8]; };
static_assert(SKINNY_MAX_SPLITS <= 8, "two splits per key group");
__device__ __forceinline__ void load_splits8(const DecodeFused& f, int64_t row_off, int col, int kg, float4 (&t)[2][2]) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int s = kg + 4 * k;
        t[k][0] = t[k][1] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (s < f.n_splits) {
            const float4* src = reinterpret_cast<const float4*>(f.part + s * f.split_stride + row_off + col);
            t[k][0] = src[0];
            t[k][1] = src[1];
        }
    }
}
__device__ __forceinline__ SplitSum add_splits8(const float4 (&t)[2][2]) {
    SplitSum r;
    r.v[0] = t[0][0].x + t[1][0].x; r.v[1] = t[0][0].y + t[1][0].y; r.v[2] = t[0][0].z + t[1][0].z; r.v[3] = t[0][0].w + t[1][0].w;
    r.v[4] = t[0][1].x + t[1][1].x; r.v[5] = t[0][1].y + t[1][1].y; r.v[6] = t[0][1].z + t[1][1].z; r.v[7] = t[0][1].w + t[1][1].w;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        r.v[e] += __shfl_xor(r.v[e], 16);
        r.v[e] += __shfl_xor(r.v[e], 32);
    }
    return r;
}
// dims 8 dc .. 8 dc + 7 of rotated head `head_col0` (packed column of the head's first dim) at position p
__device__ __forceinline__ SplitSum rotated_chunk(const DecodeFused& f, int64_t row_off, int head_col0, int dc, int kg, int p) {
    const int i0 = (dc % 8) * 8;                              // dim inside the first half of the head
    const int col_lo = head_col0 + (i0 / 32) * 64 + (i0 % 32);
    float4 tlo[2][2], thi[2][2];
    load_splits8(f, row_off, col_lo, kg, tlo);
    load_splits8(f, row_off, col_lo + 32, kg, thi);
    float2 cs[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) cs[e] = f.rope_tab[(int64_t)p * 64 + i0 + e];
    const SplitSum lo = add_splits8(tlo), hi = add_splits8(thi);
    SplitSum r;
#pragma unroll
    for (int e = 0; e < 8; ++e) r.v[e] = dc < 8 ? lo.v[e] * cs[e].x - hi.v[e] * cs[e].y : hi.v[e] * cs[e].x + lo.v[e] * cs[e].y;
    return r;
}

template <bool FUSED, bool BF, int G>
__global__ void __launch_bounds__(64 * DEC_WAVES) decode_attn_hd128_kernel(const f16_t* __restrict__ qkv, const f16_t* __restrict__ kc,
                                                               const f16_t* __restrict__ vc, const int32_t* __restrict__ kv_start,
                                                               const int32_t* __restrict__ n_ctx, int n_q_heads, int n_kv_heads,
                                                               f16_t* __restrict__ out, DecodeFused fu) {
    constexpr int HD = 128, ITS = DEC_KEYS / 4;
    static_assert(G <= DEC_MAX_HEADS && DEC_MAX_HEADS < DEC_WAVES, "wavefronts of the fused variant");
    __shared__ __align__(16) float new_rows[G + 2][HD];      // fused: the G scaled queries, the new k row, the new v row
    __shared__ float merge_o[DEC_WAVES][G][HD];
    __shared__ float merge_ml[DEC_WAVES][G][2];
    const int lane = threadIdx.x % 64, kg = lane / 16, dc = lane % 16;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int b = blockIdx.x, h0 = blockIdx.y * G;           // first query head
    const int kvh = h0 / (n_q_heads / n_kv_heads);
    const int d_q = n_q_heads * HD, d_kv = n_kv_heads * HD;
    const float sc = 0.08838834764831845f * 1.4426950408889634f;      // log2(e) / sqrt(128)
    float qf[G][8], m[G], l[G], o[G][8];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        m[g] = -INFINITY;
        l[g] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[g][e] = 0.f;
    }
    const int n = n_ctx[b] - (FUSED ? 1 : 0);                // rows to read from the cache
    const f16_t* kbase = kc + (int64_t)kv_start[b] * d_kv + kvh * HD + dc * 8;
    const f16_t* vbase = vc + (int64_t)kv_start[b] * d_kv + kvh * HD + dc * 8;
    uint4 kr[ITS], vr[ITS];
    auto load_rows = [&](const f16_t* base, int k0, uint4 (&r)[ITS]) {
#pragma unroll
        for (int it = 0; it < ITS; ++it) {
            const int key = min(k0 + it * 4 + kg, n - 1);
            r[it] = *reinterpret_cast<const uint4*>(base + (int64_t)key * d_kv);
        }
    };
    // the first block of keys and values is requested before q is put together
    if (wave * DEC_KEYS < n) {
        load_rows(kbase, wave * DEC_KEYS, kr);
        load_rows(vbase, wave * DEC_KEYS, vr);
    }
    if constexpr (FUSED) {
        // wavefront g < G finishes query head g, wavefront DEC_MAX_HEADS the new k / v row
        const int64_t row_off = (int64_t)b * (d_q + 2 * d_kv);
        const int p = n;                                     // position of the new token
        bool bad = false;
        if (wave < G) {
            const SplitSum q = rotated_chunk(fu, row_off, (h0 + wave) * HD, dc, kg, p);
            if (kg == 0) {
#pragma unroll
                for (int e = 0; e < 8; ++e) new_rows[wave][dc * 8 + e] = round_like_stored<BF>(q.v[e], bad) * sc;   // rounded (and saturated) like a stored row
            }
        } else if (wave == DEC_MAX_HEADS) {
            float4 tv[2][2];
            load_splits8(fu, row_off, d_q + d_kv + kvh * HD + dc * 8, kg, tv);
            const SplitSum kn = rotated_chunk(fu, row_off, d_q + kvh * HD, dc, kg, p);
            const SplitSum vn = add_splits8(tv);
            if (kg == 0) {
                // the cache holds 16 bits: the new row takes part in this step with the values later steps read
                uint4 kw, vw;
                kw.x = pack2_sat<BF>(kn.v[0], kn.v[1], bad); kw.y = pack2_sat<BF>(kn.v[2], kn.v[3], bad); kw.z = pack2_sat<BF>(kn.v[4], kn.v[5], bad); kw.w = pack2_sat<BF>(kn.v[6], kn.v[7], bad);
                vw.x = pack2_sat<BF>(vn.v[0], vn.v[1], bad); vw.y = pack2_sat<BF>(vn.v[2], vn.v[3], bad); vw.z = pack2_sat<BF>(vn.v[4], vn.v[5], bad); vw.w = pack2_sat<BF>(vn.v[6], vn.v[7], bad);
                if (h0 % (n_q_heads / n_kv_heads) == 0) {
                    const int64_t so = ((int64_t)kv_start[b] + n) * d_kv + kvh * HD + dc * 8;
                    *reinterpret_cast<uint4*>(fu.kc_w + so) = kw;
                    *reinterpret_cast<uint4*>(fu.vc_w + so) = vw;
                }
                float t[8];
                unpack8<BF>(kw, t);
#pragma unroll
                for (int e = 0; e < 8; ++e) new_rows[G][dc * 8 + e] = t[e];
                unpack8<BF>(vw, t);
#pragma unroll
                for (int e = 0; e < 8; ++e) new_rows[G + 1][dc * 8 + e] = t[e];
            }
        }
        if (bad) raise_flag(fu.flags, SSD_FLAG_ACT_OVERFLOW);
        __syncthreads();
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int e = 0; e < 8; ++e) qf[g][e] = new_rows[g][dc * 8 + e];
        if (wave == 0) {                                     // the new row is wavefront 0's first key
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float acc = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) acc = fmaf(qf[g][e], new_rows[G][dc * 8 + e], acc);
                m[g] = group_allreduce<16>(acc, OpSum());
                l[g] = 1.f;
                if (kg == 0) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[g][e] = new_rows[G + 1][dc * 8 + e];
                }
            }
        }
    } else {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            unpack8<BF>(*reinterpret_cast<const uint4*>(qkv + (int64_t)b * (d_q + 2 * d_kv) + (h0 + g) * HD + dc * 8), qf[g]);
#pragma unroll
            for (int e = 0; e < 8; ++e) qf[g][e] *= sc;
        }
    }
    for (int k0 = wave * DEC_KEYS; k0 < n; k0 += DEC_KEYS * DEC_WAVES) {
        const bool more = k0 + DEC_KEYS * DEC_WAVES < n;
        float s[G][ITS], alpha[G];
#pragma unroll
        for (int it = 0; it < ITS; ++it) {
            float kk[8];
            unpack8<BF>(kr[it], kk);
#pragma unroll
            for (int g = 0; g < G; ++g) {
                float acc = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) acc = fmaf(qf[g][e], kk[e], acc);
                acc = group_allreduce<16>(acc, OpSum());
                s[g][it] = (k0 + it * 4 + kg < n) ? acc : -INFINITY;
            }
        }
        if (more) load_rows(kbase, k0 + DEC_KEYS * DEC_WAVES, kr);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            float cm = s[g][0];
#pragma unroll
            for (int it = 1; it < ITS; ++it) cm = fmaxf(cm, s[g][it]);
            cm = fmaxf(cm, __shfl_xor(cm, 16));
            cm = fmaxf(cm, __shfl_xor(cm, 32));
            const float m_new = fmaxf(m[g], cm);             // finite: key k0 exists
            alpha[g] = __builtin_amdgcn_exp2f(m[g] - m_new);
            float ps = 0.f;
#pragma unroll
            for (int it = 0; it < ITS; ++it) {
                s[g][it] = __builtin_amdgcn_exp2f(s[g][it] - m_new);
                ps += s[g][it];
            }
            ps += __shfl_xor(ps, 16);
            ps += __shfl_xor(ps, 32);
            l[g] = l[g] * alpha[g] + ps;
            m[g] = m_new;
#pragma unroll
            for (int e = 0; e < 8; ++e) o[g][e] *= alpha[g];
        }
#pragma unroll
        for (int it = 0; it < ITS; ++it) {
            float vv[8];
            unpack8<BF>(vr[it], vv);
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int e = 0; e < 8; ++e) o[g][e] = fmaf(s[g][it], vv[e], o[g][e]);
        }
        if (more) load_rows(vbase, k0 + DEC_KEYS * DEC_WAVES, vr);
    }
    // merge the wavefronts: wave w's partial is (m, l, o) with o scaled by 2^-m; a wavefront without a block has l = 0
#pragma unroll
    for (int g = 0; g < G; ++g) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            o[g][e] += __shfl_xor(o[g][e], 16);
            o[g][e] += __shfl_xor(o[g][e], 32);
        }
        if (kg == 0) {
#pragma unroll
            for (int e = 0; e < 8; ++e) merge_o[wave][g][dc * 8 + e] = o[g][e];
            if (dc == 0) { merge_ml[wave][g][0] = m[g]; merge_ml[wave][g][1] = l[g]; }
        }
    }
    __syncthreads();
    if (wave < G && kg == 0) {                               // wavefront g finishes head g
        const int g = wave;
        float mt = -INFINITY;
#pragma unroll
        for (int w = 0; w < DEC_WAVES; ++w) mt = fmaxf(mt, merge_ml[w][g][0]);     // finite: wave 0 saw key 0
        float lt = 0.f, ot[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) ot[e] = 0.f;
#pragma unroll
        for (int w = 0; w < DEC_WAVES; ++w) {
            const float lw = merge_ml[w][g][1];
            const float f = lw > 0.f ? __builtin_amdgcn_exp2f(merge_ml[w][g][0] - mt) : 0.f;
            lt = fmaf(lw, f, lt);
#pragma unroll
            for (int e = 0; e < 8; ++e) ot[e] = fmaf(merge_o[w][g][dc * 8 + e], f, ot[e]);
        }
        const float inv = 1.0f / lt;
        uint4 w;
        w.x = op_pack2<BF>(ot[0] * inv, ot[1] * inv); w.y = op_pack2<BF>(ot[2] * inv, ot[3] * inv);
        w.z = op_pack2<BF>(ot[4] * inv, ot[5] * inv); w.w = op_pack2<BF>(ot[6] * inv, ot[7] * inv);
        *reinterpret_cast<uint4*>(out + (int64_t)b * d_q + (h0 + g) * HD + dc * 8) = w;
    }
}

template <bool FUSED>
static void launch_decode(const f16_t* qkv, const f16_t* kc, const f16_t* vc, const int32_t* kv_start, const int32_t* n_ctx, int Br,
                          int n_q_heads, int n_kv_heads, f16_t* out, const DecodeFused& fu, bool bf16_ops, hipStream_t st) {
    if (Br <= 0) return;
    // the most query heads of a K/V group that divide it evenly (four would take more than half of the registers)
    const int ratio = n_q_heads / n_kv_heads;
    const int G = ratio % 3 == 0 ? 3 : ratio % 2 == 0 ? 2 : 1;
#define SSD_DECODE(G_) \
    if (bf16_ops) hipLaunchKernelGGL((decode_attn_hd128_kernel<FUSED, true, G_>), dim3(Br, n_q_heads / G_), dim3(64 * DEC_WAVES), 0, st, qkv, kc, vc, kv_start, n_ctx, n_q_heads, n_kv_heads, out, fu); \
    else hipLaunchKernelGGL((decode_attn_hd128_kernel<FUSED, false, G_>), dim3(Br, n_q_heads / G_), dim3(64 * DEC_WAVES), 0, st, qkv, kc, vc, kv_start, n_ctx, n_q_heads, n_kv_heads, out, fu)
    if (G == 3) { SSD_DECODE(3); }
    else if (G == 2) { SSD_DECODE(2); }
    else { SSD_DECODE(1); }
#undef SSD_DECODE
}

void launch_decode_attn(const void* qkv, const void* kc, const void* vc, const int32_t* kv_start, const int32_t* n_ctx, int Br,
                        int n_q_heads, int n_kv_heads, void* out, bool bf16_ops, hipStream_t st) {
    launch_decode<false>((const f16_t*)qkv, (const f16_t*)kc, (const f16_t*)vc, kv_start, n_ctx, Br, n_q_heads, n_kv_heads, (f16_t*)out, DecodeFused{}, bf16_ops, st);
}

void launch_decode_attn_fused(const float* qkv_part, int n_splits, const float* rope_tab, void* kc, void* vc,
                              const int32_t* kv_start, const int32_t* n_ctx, int Br, int n_q_heads, int n_kv_heads,
                              void* out, int32_t* flags, bool bf16_ops, hipStream_t st) {
    const int64_t stride = (int64_t)Br * (n_q_heads + 2 * n_kv_heads) * 128;
    DecodeFused fu{qkv_part, n_splits, stride, reinterpret_cast<const float2*>(rope_tab), (f16_t*)kc, (f16_t*)vc, flags};
    launch_decode<true>(nullptr, (const f16_t*)kc, (const f16_t*)vc, kv_start, n_ctx, Br, n_q_heads, n_kv_heads, (f16_t*)out, fu, bf16_ops, st);
}

}  // namespace ssd
