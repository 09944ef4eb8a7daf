// Auto-regressive fallback (Sec. 2.3, Eq. 6): kernels that exist only for the token-by-token
// continuation from the accepted prefix: attention of ONE new query row per utterance against its cached
// rows (16-bit models, head_dim 128; the fp32 model's is in f32_path.hip).
// Everything else of a decode step reuses the verification kernels on a batch of Br rows
// (RMSNorm, skinny weight-streaming GEMMs with split-K, LM head with argmax).
#include "gemm_core.h"
#include "ssd_internal.h"

namespace ssd {

// head_dim 128: a workgroup is DEC_WAVES wavefronts and serves one (utterance, G query heads of one K/V head): every
// cached row is read once for its G heads.  The wavefronts take the blocks of DEC_KEYS keys of a context in turn and merge
// their (max, sum, output) triples through LDS.
// Both products are v_mfma_f32_16x16x32: S^T = K Q^T with the key rows straight from memory in operand registers, then
// O^T += V^T P^T with the values in LDS (global -> LDS loads, read back through the transposing ds_read_b64_tr_b16), whose
// key order is chosen so that a lane's scores are its operand of the second product.  Of the 16 columns of an operand G are
// needed; the columns hold the heads four times over (column c: head c % 4, part c / 4), and parts 0 to 2 carry the probabilities
// as a sum of three 16-bit pieces, which hold the 24 bits of an fp32 probability: the copies' outputs are added at the end.
// What bounds it is the chain of a launch: index, rows, score, output, with little else on the CU.  Scores and outputs on the vector
// ALU took 700 instructions a block and 206 registers (560 workgroups in two rounds); here 160 (three per CU).  The partial sums of
// the new row are requested before anything that waits for the context length and added lane by lane (loads return in order: behind
// the keys they cost a second round trip, and 32 cross-lane adds).  Per launch, traced: 27 utterances of 16 heads over 8 10.7 -> 7.7 us,
// 70 of 24 over 8 21.1 -> 14.6 us (0.4 and 0.5 of them for exact probabilities: third piece, scales, the sum of the parts; before it eight
// wavefronts instead of four 8.2 and 16.9 against 7.3 and 14.1, 128 registers, four per CU, 7.7 and 14.5).
constexpr int DEC_WAVES = 4;
constexpr int DEC_KEYS = 32;
constexpr int DEC_MAX_HEADS = 3;                             // one wavefront of the fused variant per head and one for the new k / v row

// Fused variant: the QKV projection of the step has been left as K-split partial sums
// part[split][row][packed column] (fp32, packed column order of the fused QKV weight: inside a head the
// rotary pairs (i, i+64) sit 32 columns apart in 64-column groups, V columns are in natural order).
// The kernel adds the splits, rotates q and the new k, appends the new k / v row to the cache (first query
// head of each K/V group) and treats that row as the last key without reading it back.
template <bool BF> __device__ __forceinline__ uint16_t round_sat(float v, bool& bad) {
    if constexpr (BF) return f32_to_bf16(v);
    else return f32_to_f16_sat(v, bad);
}
// The pieces of a probability p: piece 0 is p times P_SCALE, piece k + 1 what the operand type leaves of piece k, times PIECE_SCALE (a power
// of two below the first bit that is left, so that every piece keeps the magnitude of p: IEEE half would lose bits of a small one).
// P_SCALE is for half alone: with it all bits of a p down to 2^-37 are held, and of a smaller one those down to 2^-61; bfloat16 has fp32's
// range, and a scale would overflow its sums.  The exponent of p is formed without it: added there, the 14 took four bits of a p near 1.
template <bool BF> constexpr float P_SCALE = BF ? 1.f : 16384.f;
template <bool BF> constexpr float PIECE_SCALE = BF ? 256.f : 2048.f;
template <bool BF> __device__ __forceinline__ float piece_of(float p, int part) {
    const float r0 = p * P_SCALE<BF>;
    const float r1 = (r0 - Op16<BF>::to_f32(Op16<BF>::cvt(r0))) * PIECE_SCALE<BF>;
    const float r2 = (r1 - Op16<BF>::to_f32(Op16<BF>::cvt(r1))) * PIECE_SCALE<BF>;
    return part == 0 ? r0 : part == 1 ? r1 : r2;
}

// v and that of the lane the rotation names (with the bound control set, which no rotation needs, the two are one instruction)
template <int CTRL> __device__ __forceinline__ float add_rotated(float v) {
    return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
constexpr float F32_LARGEST = 3.4028234663852886e38f;

struct DecodeFused {
    const float* part; int n_splits; int64_t split_stride;    // split_stride = rows * (d_q + 2 d_kv)
    const float2* rope_tab;                                   // [position][64] (cos, sin)
    f16_t* kc_w; f16_t* vc_w;                                 // writable views of the cache
    int32_t* flags;                                           // sticky device flags (SSD_FLAG_ACT_OVERFLOW on a saturated store)
    // The new row's position is the number of rows its utterance has in the cache (cache row i of an
    // utterance is position i), and its slot is kv_start + that number: no further index arrays.
};
// Sums over the splits of two packed columns of a row, in split order.  All loads of a lane are requested at once (a split beyond
// the last is a second copy of it and left out), before anything that depends on the context length.
static_assert(SKINNY_MAX_SPLITS <= 8, "loads of a lane");
struct SplitPair { float a[SKINNY_MAX_SPLITS], b[SKINNY_MAX_SPLITS]; };
__device__ __forceinline__ void load_splits(const DecodeFused& f, int64_t off_a, int64_t off_b, SplitPair& t) {
#pragma unroll
    for (int s = 0; s < SKINNY_MAX_SPLITS; ++s) {
        const float* src = f.part + min(s, f.n_splits - 1) * f.split_stride;
        t.a[s] = src[off_a];
        t.b[s] = src[off_b];
    }
}
__device__ __forceinline__ float2 add_splits(const DecodeFused& f, const SplitPair& t) {
    float2 r = make_float2(t.a[0], t.b[0]);
#pragma unroll
    for (int s = 1; s < SKINNY_MAX_SPLITS; ++s) {
        r.x += s < f.n_splits ? t.a[s] : 0.f;
        r.y += s < f.n_splits ? t.b[s] : 0.f;
    }
    return r;
}

template <bool FUSED, bool BF, int G>
__global__ void __launch_bounds__(64 * DEC_WAVES, 3) decode_attn_hd128_kernel(const f16_t* __restrict__ qkv, const f16_t* __restrict__ kc,
                                                               const f16_t* __restrict__ vc, const int32_t* __restrict__ kv_start,
                                                               const int32_t* __restrict__ n_ctx, int n_q_heads, int n_kv_heads,
                                                               f16_t* __restrict__ out, DecodeFused fu) {
    constexpr int HD = 128, ROW = HD * 2, STEP = DEC_KEYS * DEC_WAVES;
    static_assert(G <= DEC_MAX_HEADS && DEC_MAX_HEADS < DEC_WAVES, "wavefronts of the fused variant");
    static_assert(G * HD * 4 <= DEC_KEYS * ROW, "a wavefront's output fits its block of values");
    __shared__ __align__(1024) unsigned char v_s[DEC_WAVES][DEC_KEYS * ROW];   // a wavefront's block of values, later its output [G][HD] fp32
    __shared__ uint4 new_rows[G + 2][HD / 8];                // fused: the G queries, the new k row, the new v row (operand type)
    __shared__ float merge_ml[DEC_WAVES][G][2];
    const int lane = threadIdx.x % 64, kg = lane / 16, dc = lane % 16;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int b = blockIdx.x, h0 = blockIdx.y * G;           // first query head
    const int kvh = h0 / (n_q_heads / n_kv_heads);
    const int d_q = n_q_heads * HD, d_kv = n_kv_heads * HD;
    const float sc = 0.08838834764831845f * 1.4426950408889634f;      // log2(e) / sqrt(128)
    const int head = min(dc % 4, G - 1), part = dc / 4;      // of this lane's column
    const int n_rows = n_ctx[b], slot0 = kv_start[b];
    // fused: wavefront g < G finishes query head g, wavefront DEC_MAX_HEADS the new k / v row; lane i has rotary pair (i, i + 64).
    // (Wavefronts in between repeat the last head: with a branch around these loads the rotary entries are fetched behind it.)
    const int job = wave == DEC_MAX_HEADS ? G : min(wave, G - 1);
    SplitPair tq, tv;
    if constexpr (FUSED) {
        const int64_t row_off = (int64_t)b * (d_q + 2 * d_kv);
        const int64_t col = row_off + (job < G ? (h0 + job) * HD : d_q + kvh * HD) + (lane / 32) * 64 + lane % 32;
        load_splits(fu, col, col + 32, tq);
        if (wave == DEC_MAX_HEADS) load_splits(fu, row_off + d_q + d_kv + kvh * HD + lane, row_off + d_q + d_kv + kvh * HD + lane + 64, tv);
        __builtin_amdgcn_sched_barrier(0);
    }
    const int n = n_rows - (FUSED ? 1 : 0);                  // rows to read from the cache; the position of the new token
    const int64_t first = (int64_t)slot0 * d_kv + kvh * HD;
    float2 cs = make_float2(1.f, 0.f);
    if constexpr (FUSED) cs = fu.rope_tab[(int64_t)n * 64 + lane];
    const int d_kv2 = d_kv * 2, last = max(n - 1, 0);
    u32x4_t kr[2][4];
    // Keys k0 .. k0 + 31: lane (row dc of a half of 16, dims 8 kg + 32 s) in registers.  Values: four rows of 256 bytes per
    // instruction, the sixteen 16-byte chunks of row r at chunk ^ 4 (r & 3) ^ 2 (r >> 2 & 1), which spreads the eight 32-byte
    // pieces that half a wavefront reads over all LDS banks.  Rows beyond the context are copies of the last one.
    // (32-bit offsets from the block's first row: a context may be longer than 4 GiB.)
    auto load_keys = [&](int k0) {
        const int r0 = min(k0, last), beyond = last - r0;
        const __amdgpu_buffer_rsrc_t k_rsrc = make_rsrc(kc + first + (int64_t)r0 * d_kv);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int off = min(16 * c + dc, beyond) * d_kv2 + kg * 16;
#pragma unroll
            for (int s = 0; s < 4; ++s) kr[c][s] = __builtin_amdgcn_raw_buffer_load_b128(k_rsrc, off + 64 * s, 0, 0);
        }
    };
    auto load_values = [&](int k0) {
        const int r0 = min(k0, last), beyond = last - r0;
        const __amdgpu_buffer_rsrc_t v_rsrc = make_rsrc(vc + first + (int64_t)r0 * d_kv);
#pragma unroll
        for (int i = 0; i < DEC_KEYS / 4; ++i) {
            const int off = min(4 * i + kg, beyond) * d_kv2 + (dc ^ (4 * kg + 2 * (i & 1))) * 16;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(v_rsrc, (lds_void_t*)(v_s[wave] + i * 1024), 16, off, 0, 0, 0);
        }
    };
    // The first block is requested before q is put together, by every wavefront: a branch here would make the wait for the partial
    // sums one for everything.
    load_keys(wave * DEC_KEYS);
    load_values(wave * DEC_KEYS);
    f16x8_t qf[4];
    float m = -INFINITY, l = 0.f;
    f32x4_t o[HD / 16];
#pragma unroll
    for (int i = 0; i < HD / 16; ++i) o[i] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
    if constexpr (FUSED) {
        bool bad = false;
        // as later steps and the next kernel read them: rounded to the operand type, saturated for IEEE half
        const float2 t = add_splits(fu, tq);
        const uint16_t lo = round_sat<BF>(t.x * cs.x - t.y * cs.y, bad), hi = round_sat<BF>(t.y * cs.x + t.x * cs.y, bad);
        uint16_t* row = reinterpret_cast<uint16_t*>(new_rows[job]);
        row[lane] = lo;
        row[lane + 64] = hi;
        if (wave == DEC_MAX_HEADS) {
            const float2 v = add_splits(fu, tv);
            const uint16_t v0 = round_sat<BF>(v.x, bad), v1 = round_sat<BF>(v.y, bad);
            uint16_t* vrow = reinterpret_cast<uint16_t*>(new_rows[G + 1]);
            vrow[lane] = v0;
            vrow[lane + 64] = v1;
            if (h0 % (n_q_heads / n_kv_heads) == 0) {
                f16_t* kd = fu.kc_w + first + (int64_t)n * d_kv + lane;
                f16_t* vd = fu.vc_w + first + (int64_t)n * d_kv + lane;
                kd[0] = lo; kd[64] = hi;
                vd[0] = v0; vd[64] = v1;
            }
        }
        if (bad) raise_flag(fu.flags, SSD_FLAG_ACT_OVERFLOW);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xC07F);                  // the LDS stores above; a barrier with a fence would wait for the values as well
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int s = 0; s < 4; ++s) qf[s] = as_f16x8(new_rows[head][4 * s + kg]);
        if (wave == 0) {                                     // the new row is wavefront 0's first key: every row of the operand
            f32x4_t s_new = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < 4; ++s) s_new = mfma_16x16x32<BF>(as_f16x8(new_rows[G][4 * s + kg]), qf[s], s_new);
            m = s_new[0] * sc;
            l = 1.f;
            const uint2* vn = reinterpret_cast<const uint2*>(new_rows[G + 1]);
#pragma unroll
            for (int i = 0; i < HD / 16; ++i) {
                const uint2 w = vn[4 * i + kg];              // dims 16 i + 4 kg .. + 3
                o[i] = (f32x4_t){Op16<BF>::to_f32((uint16_t)w.x), Op16<BF>::to_f32((uint16_t)(w.x >> 16)),
                                 Op16<BF>::to_f32((uint16_t)w.y), Op16<BF>::to_f32((uint16_t)(w.y >> 16))};
                o[i] = part == 0 ? o[i] * P_SCALE<BF> : (f32x4_t){0.f, 0.f, 0.f, 0.f};
            }
        }
    } else {
        const f16_t* q = qkv + (int64_t)b * (d_q + 2 * d_kv) + (h0 + head) * HD + kg * 8;
#pragma unroll
        for (int s = 0; s < 4; ++s) qf[s] = as_f16x8(*reinterpret_cast<const uint4*>(q + 32 * s));
    }
    // transposing read: lane i of 16 passes row i / 4 and dims 4 (i % 4) .. + 3 of a 16-dim block, lane j receives dim j of four rows
    const int v_row = 4 * kg + dc / 4, v_low = (dc % 4) / 2, v_sub = (dc % 2) * 8;
    const int v_swz = 4 * (v_row & 3) + 2 * ((v_row >> 2) & 1);           // the same for row v_row + 16
    auto block = [&](auto more_c, int k0) {                  // more: another block follows, its keys are requested as soon as these are used
        constexpr bool MORE = decltype(more_c)::value;
        f32x4_t s[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            s[c] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 4; ++t) s[c] = mfma_16x16x32<BF>(__builtin_bit_cast(f16x8_t, kr[c][t]), qf[t], s[c]);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MORE) load_keys(k0 + STEP);
        __builtin_amdgcn_sched_barrier(0);
        float mx = -INFINITY;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[c][r] = k0 + 16 * c + 4 * kg + r < n ? s[c][r] * sc : -INFINITY;
                mx = fmaxf(mx, s[c][r]);
            }
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float m_new = fmaxf(m, mx);                    // finite: key k0 exists
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        float ps = 0.f;
        uint32_t pw[4];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float pr = __builtin_amdgcn_exp2f(s[c][r] - m_new);
                ps += pr;
                v[r] = piece_of<BF>(pr, part);
            }
            pw[2 * c] = op_pack2<BF>(v[0], v[1]);
            pw[2 * c + 1] = op_pack2<BF>(v[2], v[3]);
        }
        ps += __shfl_xor(ps, 16);
        ps += __shfl_xor(ps, 32);
        l = l * alpha + ps;
        m = m_new;
        const f16x8_t pf = as_f16x8(make_uint4(pw[0], pw[1], pw[2], pw[3]));
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_waitcnt(0x0F70 | (MORE ? 8 : 0));  // the values of this block have landed (a wavefront reads its own only)
        __builtin_amdgcn_sched_barrier(0);
        tr_v4i16 vf[HD / 16][2];                             // all reads first: one LDS latency, not eight
#pragma unroll
        for (int i = 0; i < HD / 16; ++i) {
            const unsigned char* a = v_s[wave] + v_row * ROW + (((2 * i) | v_low) ^ v_swz) * 16 + v_sub;
            vf[i][0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr_v4i16*)a);
            vf[i][1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_tr_v4i16*)(a + 16 * ROW));
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < HD / 16; ++i) {
            o[i] *= alpha;
            o[i] = mfma_16x16x32<BF>(__builtin_bit_cast(f16x8_t, __builtin_shufflevector(vf[i][0], vf[i][1], 0, 1, 2, 3, 4, 5, 6, 7)), pf, o[i]);
        }
        if constexpr (MORE) {
            __builtin_amdgcn_s_waitcnt(0xC07F);              // the reads of this block are done
            __builtin_amdgcn_sched_barrier(0);
            load_values(k0 + STEP);
        }
    };
    int k0 = wave * DEC_KEYS;
    for (; k0 + STEP < n; k0 += STEP) block(std::true_type(), k0);
    if (k0 < n) block(std::false_type(), k0);
    // merge the wavefronts: wave w's partial is (m, l, o) with o scaled by 2^-m and P_SCALE; a wavefront without a block has l = 0
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);                      // the values of a wavefront without a block: they land where its output goes
    __builtin_amdgcn_sched_barrier(0);
    float* mine = reinterpret_cast<float*>(v_s[wave]);
    const float lower = part == 1 ? 1.f / PIECE_SCALE<BF> : part == 2 ? 1.f / (PIECE_SCALE<BF> * PIECE_SCALE<BF>) : 0.f;
#pragma unroll
    for (int i = 0; i < HD / 16; ++i) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {                        // the parts of a column lie 4 lanes apart
            // part 3 is a copy of part 2.  An infinite value times a lower piece of 0 is NaN, which the clamp makes finite: the infinite sum of part 0 stays
            const float rest = add_rotated<DPP_ROW_ROR4>(add_rotated<DPP_ROW_ROR8>(o[i][r] * lower));
            o[i][r] += __builtin_amdgcn_fmed3f(rest, -F32_LARGEST, F32_LARGEST);
        }
        if (dc < G) *reinterpret_cast<f32x4_t*>(mine + dc * HD + 16 * i + 4 * kg) = o[i];
    }
    if (lane < G) { merge_ml[wave][lane][0] = m; merge_ml[wave][lane][1] = l; }
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
            const float* src = reinterpret_cast<const float*>(v_s[w]) + g * HD + dc * 8;
#pragma unroll
            for (int e = 0; e < 8; ++e) ot[e] = fmaf(src[e], f, ot[e]);
        }
        const float inv = 1.0f / P_SCALE<BF> / lt;
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
