// The three projection GEMMs of a decoder layer (Eq. 4's network), 16-bit MFMA (IEEE half or bfloat16 operands,
// a template parameter of every kernel here) with fused epilogues:
//   QKV      : a[M,d] x Wqkv^T  -> rotary embedding on q,k in fp32 -> f16 qkv[M, d_q + 2 d_kv]
//   residual : o[M,K] x W^T     -> x[M,N] += acc                (attention output and MLP down projection)
//   SwiGLU   : b[M,d] x Wgu^T   -> h[M,d_ff] = silu(gate) * up  (f16)
// Every epilogue first multiplies the accumulator by `descale`, the inverse of the power of two the
// weight tensor was scaled by when it was converted to f16.
// The fused weight layouts are produced by pack_qkv_kernel / pack_gate_up_kernel: a column and the
// column it must be combined with sit 32 packed columns apart inside a group of 64, i.e. in two
// accumulator blocks of the same lane.
// Four main loops feed these epilogues: big tiles on v_mfma_f32_16x16x32_f16 (gemm_core16.h), skinny
// LDS-ring tiles from 33 rows on (gemm_core.h) and, from the stream layout of the weights, the
// register-streaming kernels for at most 32 and for 33..128 rows (gemm_stream.h).
#include <algorithm>
#include <type_traits>

#include "gemm_core.h"
#include "gemm_core16.h"
#include "gemm_stream.h"
#include "ssd_internal.h"

namespace ssd {

// Workgroup id -> tile: one XCD walks a contiguous run of tiles, and tiles are ordered in bands of
// GROUP_M row-tiles so that the run reuses few A and W panels.
__device__ __forceinline__ void tile_of_workgroup(int pid, int total, int tiles_m, int tiles_n, int& tm, int& tn) {
    constexpr int GROUP_M = 4;
    const int v = xcd_contiguous_index(pid, total);
    const int band = v / (GROUP_M * tiles_n);
    const int first_m = band * GROUP_M;
    const int rows = min(tiles_m - first_m, GROUP_M);
    const int in = v % (GROUP_M * tiles_n);
    tm = first_m + in % rows;
    tn = in / rows;
}

// The epilogues below read first and write afterwards, block by block: a load placed after a store
// through an unrelated pointer cannot be moved ahead of it by the compiler, and a read-modify-write
// written element by element degenerates into one exposed memory round trip per element.
// They are written against an accumulator layout L (Layout32: 32x32 blocks of v_mfma_f32_32x32x16,
// Layout16: 16x16 blocks of v_mfma_f32_16x16x32): L::row / L::col give the element a register holds and
// L::PAIR the distance, in blocks, to the block 32 columns further (where the fused weight layouts put
// the partner column).
constexpr int residual_batch(int tm, int g0) {             // largest divisor of tm that is at most g0 (at least 1)
    int g = 1;
    for (int c = 1; c <= tm; ++c)
        if (tm % c == 0 && c <= g0) g = c;
    return g;
}
template <bool BF_>
struct EpiResidual {
    // (not transposed: the fp32 read-modify-write measured 3-8 % slower with 16-byte accesses whose lanes of one
    // row segment are 16 lane ids apart, O projection 8.77 -> 8.95 ms per step at 15214 rows)
    static constexpr bool WANTS_SPLIT = false, BF = BF_, TRANSPOSE = false, USES_LDS = false;
    float* x; int ldx; float descale;
    template <int TM, int TN, class L = Layout32>
    __device__ __forceinline__ void operator()(typename L::vec_t (&acc)[TM][TN], int row0, int col0, int M, int lane) const {
        if constexpr (L::TRANSPOSED) {
            // a lane holds four consecutive columns of one row per block: 16-byte loads and stores
            constexpr int GT = residual_batch(TM, 96 / (4 * TN));
#pragma unroll
            for (int i0 = 0; i0 < TM; i0 += GT) {
                float4 old[GT][TN];
#pragma unroll
                for (int g = 0; g < GT; ++g) {
                    const int row = min(row0 + L::row(i0 + g, lane), M - 1);
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        old[g][j] = *reinterpret_cast<const float4*>(x + (int64_t)row * ldx + col0 + L::col4(j, lane));
                }
#pragma unroll
                for (int g = 0; g < GT; ++g) {
                    const int row = row0 + L::row(i0 + g, lane);
                    if (row >= M) continue;
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const f32x4_t a = acc[i0 + g][j];
                        *reinterpret_cast<float4*>(x + (int64_t)row * ldx + col0 + L::col4(j, lane)) =
                            make_float4(old[g][j].x + a[0] * descale, old[g][j].y + a[1] * descale, old[g][j].z + a[2] * descale,
                                        old[g][j].w + a[3] * descale);
                    }
                }
            }
            return;
        } else {
        // Row blocks per batch: all loads of a batch are in flight together, so a tile pays one memory
        // latency per batch.  Up to 96 registers of old values (the fragment registers are dead by now).
        constexpr int G0 = 96 / (L::REGS * TN);
        constexpr int G = residual_batch(TM, G0);
#pragma unroll
        for (int i0 = 0; i0 < TM; i0 += G) {
            float old[G][L::REGS][TN];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int r = 0; r < L::REGS; ++r) {
                    const int row = min(row0 + L::row(i0 + g, r, lane), M - 1);
#pragma unroll
                    for (int j = 0; j < TN; ++j) old[g][r][j] = x[(int64_t)row * ldx + col0 + L::col(j, lane)];
                }
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int r = 0; r < L::REGS; ++r) {
                    const int row = row0 + L::row(i0 + g, r, lane);
                    if (row >= M) continue;
#pragma unroll
                    for (int j = 0; j < TN; ++j)
                        x[(int64_t)row * ldx + col0 + L::col(j, lane)] = old[g][r][j] + acc[i0 + g][j][r] * descale;
                }
        }
        }
    }
};

// The residual epilogue of the big tiles: x[M,N] += acc through the workgroup's LDS (free after the K loop).  With
// transposed accumulator blocks a lane writes its four consecutive columns of a row as one 16-byte LDS store; the
// wavefront's 64 x 64 half tile is then read back row by row, 16 lanes per 256-byte row, so that the old values of x
// are loaded and the sums stored with fully coalesced 16-byte accesses: 32 + 32 global instructions per wavefront
// instead of 128 + 128 four-byte ones that touch 64-byte pieces of four rows each.
constexpr int RES_LDS_STRIDE = 68;                           // floats per staged row: 64 + 4 (16-byte columns stay spread)
template <bool BF_>
struct EpiResidualLds {
    static constexpr bool WANTS_SPLIT = false, BF = BF_, TRANSPOSE = true, USES_LDS = true;
    float* x; int ldx; float descale;
    template <int TM> static constexpr int wave_lds_bytes() { return ((TM + 1) / 2) * 16 * RES_LDS_STRIDE * 4; }
    template <int TM, int TN>
    __device__ __forceinline__ void run_lds(f32x4_t (&acc)[TM][TN], int row0, int col0, int M, int lane, float* stage) const {
        static_assert(TN == 4, "a wavefront tile of 64 columns");
        constexpr int H0 = (TM + 1) / 2;                     // row blocks of the first half; the second has TM - H0
        constexpr int ROWS = H0 * 16;
        const int m = lane % 16, g = lane / 16;
        const int rr = lane / 16, cc = (lane % 16) * 4;      // read-back: row 4 it + rr of the half, columns cc .. cc + 3
        auto do_half = [&](auto half) {
            constexpr int HB = half ? TM - H0 : H0;          // row blocks
            constexpr int NI = HB * 4;                       // instructions: 4 rows x 256 bytes each
            // old values first: their round trip overlaps the LDS exchange
            float4 old[NI];
#pragma unroll
            for (int it = 0; it < NI; ++it) {
                const int row = min(row0 + half * ROWS + 4 * it + rr, M - 1);
                typedef float f32x4v __attribute__((ext_vector_type(4)));
                const f32x4v t = __builtin_nontemporal_load(reinterpret_cast<const f32x4v*>(x + (int64_t)row * ldx + col0 + cc));
                old[it] = make_float4(t[0], t[1], t[2], t[3]);
            }
            if (half) __builtin_amdgcn_wave_barrier();       // the reads of the first half are done (waited for below)
#pragma unroll
            for (int i = 0; i < HB; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const f32x4_t a = acc[half * H0 + i][j];
                    *reinterpret_cast<float4*>(stage + (i * 16 + m) * RES_LDS_STRIDE + j * 16 + 4 * g) =
                        make_float4(a[0] * descale, a[1] * descale, a[2] * descale, a[3] * descale);
                }
            __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0): the stores have landed
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < NI; ++it) {
                const int row = row0 + half * ROWS + 4 * it + rr;
                const float4 v = *reinterpret_cast<const float4*>(stage + (4 * it + rr) * RES_LDS_STRIDE + cc);
                if (row < M)
                    *reinterpret_cast<float4*>(x + (int64_t)row * ldx + col0 + cc) =
                        make_float4(old[it].x + v.x, old[it].y + v.y, old[it].z + v.z, old[it].w + v.w);
            }
            __builtin_amdgcn_s_waitcnt(0xC07F);
        };
        do_half(std::integral_constant<int, 0>());
        do_half(std::integral_constant<int, 1>());
    }
};

template <bool BF_>
struct EpiQkvRope {
    static constexpr bool WANTS_SPLIT = false, BF = BF_, TRANSPOSE = true, USES_LDS = false;     // big tiles: transposed accumulator blocks
    f16_t* qkv; int ldq; int d_rot; float descale;            // d_rot = d_q + d_kv: columns that get rotated
    const int32_t* pos; const float2* rope_tab; // rope_tab[pos][i] = (cos, sin), i < 64
    // optional K/V cache: rows with row_slot[row] >= 0 also store their k and v parts at that slot
    const int32_t* row_slot; f16_t* kc; f16_t* vc; int d_q;
    // optional: the table rows already gathered per decoder row (rope_rows[row][i] = rope_tab[pos[row]][i]),
    // which takes the position lookup out of the dependency chain
    const float2* rope_rows;
    int32_t* flags;                             // sticky device flags: a saturated store raises SSD_FLAG_ACT_OVERFLOW
    template <int TM, int TN, class L = Layout32>
    __device__ __forceinline__ void operator()(typename L::vec_t (&acc)[TM][TN], int row0, int col0, int M, int lane) const {
        static_assert((TN * L::BLOCK) % 64 == 0, "rotation partners live 32 packed columns apart in groups of 64");
        if constexpr (L::TRANSPOSED) {
            // A lane holds one row and four consecutive packed columns per block: the four rotary entries are one
            // 32-byte read, the outputs two 8-byte stores (and two more into the K/V cache).
            const float2* tabT = rope_rows ? rope_rows : rope_tab;
            const int d_kvT = d_rot - d_q;
            float peak = 0.f;
            constexpr int NJT = TN / 2;
            constexpr int MOST = 64 / (NJT * 8) > 0 ? 64 / (NJT * 8) : 1, NB = (TM + MOST - 1) / MOST;
            constexpr int GT = (TM + NB - 1) / NB;          // row blocks of a batch; the last may be one short
#pragma unroll
            for (int i0 = 0; i0 < TM; i0 += GT) {
                int t_row[GT], slot[GT];
#pragma unroll
                for (int g = 0; g < GT; ++g) {
                    if (i0 + g >= TM) continue;
                    const int row = min(row0 + L::row(i0 + g, lane), M - 1);
                    t_row[g] = rope_rows ? row : pos[row];
                    slot[g] = row_slot ? row_slot[row] : -1;
                }
                float4 cs[GT][NJT][2];                      // (cos, sin) of four consecutive rotary indices
#pragma unroll
                for (int g = 0; g < GT; ++g)
#pragma unroll
                    for (int jj = 0; jj < NJT; ++jj) {
                        if (i0 + g >= TM) continue;
                        const int j = (jj / L::PAIR) * 2 * L::PAIR + jj % L::PAIR;
                        const int p = col0 + j * L::BLOCK;
                        const int i_rot = ((p % 128) / 64) * 32 + p % 32 + 4 * (lane / 16);
                        if (p < d_rot) {
                            const float4* src = reinterpret_cast<const float4*>(tabT + (int64_t)t_row[g] * 64 + i_rot);
                            cs[g][jj][0] = src[0];
                            cs[g][jj][1] = src[1];
                        } else {
                            cs[g][jj][0] = cs[g][jj][1] = make_float4(1.f, 0.f, 1.f, 0.f);
                        }
                    }
                auto store_batch = [&](auto clamp_c) {
                    constexpr bool CLAMP = decltype(clamp_c)::value;
#pragma unroll
                    for (int g = 0; g < GT; ++g) {
                        if (i0 + g >= TM) continue;
                        const int row = row0 + L::row(i0 + g, lane);
                        if (row >= M) continue;
#pragma unroll
                        for (int jj = 0; jj < NJT; ++jj) {
                            const int j = (jj / L::PAIR) * 2 * L::PAIR + jj % L::PAIR;
                            const int p = col0 + j * L::BLOCK;
                            const bool rot = p < d_rot;
                            const int head = p / 128, i_rot = ((p % 128) / 64) * 32 + p % 32 + 4 * (lane / 16);
                            const int c0 = rot ? head * 128 + i_rot : p + 4 * (lane / 16);
                            const int c1 = rot ? c0 + 64 : c0 + 32;
                            const f32x4_t a = acc[i0 + g][j], b = acc[i0 + g][j + L::PAIR];
                            const float cx[4] = {cs[g][jj][0].x, cs[g][jj][0].z, cs[g][jj][1].x, cs[g][jj][1].z};
                            const float sy[4] = {cs[g][jj][0].y, cs[g][jj][0].w, cs[g][jj][1].y, cs[g][jj][1].w};
                            uint16_t v0[4], v1[4];
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                const float av = a[r] * descale, bv = b[r] * descale;
                                v0[r] = Op16<BF>::template store<CLAMP>(av * cx[r] - bv * sy[r], peak);
                                v1[r] = Op16<BF>::template store<CLAMP>(bv * cx[r] + av * sy[r], peak);
                            }
                            const uint2 w0 = make_uint2((uint32_t)v0[0] | ((uint32_t)v0[1] << 16), (uint32_t)v0[2] | ((uint32_t)v0[3] << 16));
                            const uint2 w1 = make_uint2((uint32_t)v1[0] | ((uint32_t)v1[1] << 16), (uint32_t)v1[2] | ((uint32_t)v1[3] << 16));
                            f16_t* o = qkv + (int64_t)row * ldq;
                            *reinterpret_cast<uint2*>(o + c0) = w0;
                            *reinterpret_cast<uint2*>(o + c1) = w1;
                            if (slot[g] >= 0 && c0 >= d_q) {
                                f16_t* dst = (rot ? kc : vc) + (int64_t)slot[g] * d_kvT - (rot ? d_q : d_rot);
                                *reinterpret_cast<uint2*>(dst + c0) = w0;
                                *reinterpret_cast<uint2*>(dst + c1) = w1;
                            }
                        }
                    }
                };
                const float before = peak;
                store_batch(std::false_type());
                if (!(peak <= F16_MAX)) {
                    peak = before;
                    store_batch(std::true_type());
                    raise_flag(flags, SSD_FLAG_ACT_OVERFLOW);
                }
            }
        } else {
        // Column blocks come in groups of 64 packed columns: the first half holds x[i], the second x[i+64]
        // of 32 rotation pairs (or 64 plain columns of v); block j is handled with its partner j + PAIR.
        constexpr int NJ = TN / 2;
        // All table loads of a batch of row blocks are issued before the first store of the batch (the
        // compiler cannot move a load above a store that might alias it), so a batch costs one memory
        // latency, not one per block: up to 32 (cos, sin) pairs, 64 registers, are held per lane.
        constexpr int G = residual_batch(TM, 32 / (NJ * L::REGS) > 0 ? 32 / (NJ * L::REGS) : 1);
        const float2* tab = rope_rows ? rope_rows : rope_tab;
        const int d_kv = d_rot - d_q;
        float peak = 0.f;                                   // largest magnitude stored by this lane
#pragma unroll
        for (int i0 = 0; i0 < TM; i0 += G) {
            int t_row[G][L::REGS], slot[G][L::REGS];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int r = 0; r < L::REGS; ++r) {
                    const int row = min(row0 + L::row(i0 + g, r, lane), M - 1);
                    t_row[g][r] = rope_rows ? row : pos[row];
                    slot[g][r] = row_slot ? row_slot[row] : -1;
                }
            float2 cs[G][NJ][L::REGS];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj) {
                    const int j = (jj / L::PAIR) * 2 * L::PAIR + jj % L::PAIR;
                    const int p = col0 + j * L::BLOCK;
                    const int i_rot = ((p % 128) / 64) * 32 + p % 32 + lane % L::BLOCK;
#pragma unroll
                    for (int r = 0; r < L::REGS; ++r)
                        cs[g][jj][r] = p < d_rot ? tab[(int64_t)t_row[g][r] * 64 + i_rot] : make_float2(1.f, 0.f);
                }
            // stores of the batch; repeated with clamping by a lane that met a value beyond the half range
            auto store_batch = [&](auto clamp_c) {
                constexpr bool CLAMP = decltype(clamp_c)::value;
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int jj = 0; jj < NJ; ++jj) {
                        const int j = (jj / L::PAIR) * 2 * L::PAIR + jj % L::PAIR;
                        const int p = col0 + j * L::BLOCK;              // packed column of this block
                        const bool rot = p < d_rot;
                        const int head = p / 128, i_rot = ((p % 128) / 64) * 32 + p % 32 + lane % L::BLOCK;
                        const int c0 = rot ? head * 128 + i_rot : p + lane % L::BLOCK;
                        const int c1 = rot ? c0 + 64 : c0 + 32;
#pragma unroll
                        for (int r = 0; r < L::REGS; ++r) {
                            const int row = row0 + L::row(i0 + g, r, lane);
                            if (row >= M) continue;
                            const float a = acc[i0 + g][j][r] * descale, b = acc[i0 + g][j + L::PAIR][r] * descale;
                            const float2 c = cs[g][jj][r];
                            f16_t* o = qkv + (int64_t)row * ldq;
                            const f16_t v0 = Op16<BF>::template store<CLAMP>(a * c.x - b * c.y, peak), v1 = Op16<BF>::template store<CLAMP>(b * c.x + a * c.y, peak);
                            o[c0] = v0;
                            o[c1] = v1;
                            if (slot[g][r] >= 0 && c0 >= d_q) {           // a group of 64 lies inside q, k or v
                                f16_t* dst = (rot ? kc : vc) + (int64_t)slot[g][r] * d_kv - (rot ? d_q : d_rot);
                                dst[c0] = v0;
                                dst[c1] = v1;
                            }
                        }
                    }
            };
            const float before = peak;
            store_batch(std::false_type());
            if (!(peak <= F16_MAX)) {
                peak = before;                              // keep later batches on the plain pass unless they overflow too
                store_batch(std::true_type());
                raise_flag(flags, SSD_FLAG_ACT_OVERFLOW);
            }
        }
        }
    }
};

template <bool BF_>
struct EpiSwiglu {
    static constexpr bool WANTS_SPLIT = false, BF = BF_, TRANSPOSE = true, USES_LDS = false;
    f16_t* h; int d_ff; float descale; int32_t* flags;
    template <int TM, int TN, class L = Layout32>
    __device__ __forceinline__ void operator()(typename L::vec_t (&acc)[TM][TN], int row0, int col0, int M, int lane) const {
        static_assert((TN * L::BLOCK) % 64 == 0, "gate/up live 32 packed columns apart in groups of 64");
        float peak = 0.f;                                   // largest magnitude stored by this lane
        if constexpr (L::TRANSPOSED) {
            // a lane holds one row and four consecutive packed columns per block: four outputs, one 8-byte store
            auto store_allT = [&](auto clamp_c) {
                constexpr bool CLAMP = decltype(clamp_c)::value;
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    const int row = row0 + L::row(i, lane);
                    if (row >= M) continue;
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        if ((j / L::PAIR) % 2 != 0) continue;
                        const int p = col0 + j * L::BLOCK;
                        const int f = (p / 64) * 32 + p % 32 + 4 * (lane / 16);
                        uint16_t v[4];
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float g = acc[i][j][r] * descale, u = acc[i][j + L::PAIR][r] * descale;
                            v[r] = Op16<BF>::template store<CLAMP>(g * u * __builtin_amdgcn_rcpf(1.0f + __expf(-g)), peak);
                        }
                        *reinterpret_cast<uint2*>(h + (int64_t)row * d_ff + f) =
                            make_uint2((uint32_t)v[0] | ((uint32_t)v[1] << 16), (uint32_t)v[2] | ((uint32_t)v[3] << 16));
                    }
                }
            };
            store_allT(std::false_type());
            if (!(peak <= F16_MAX)) {
                store_allT(std::true_type());
                raise_flag(flags, SSD_FLAG_ACT_OVERFLOW);
            }
        } else {
        auto store_all = [&](auto clamp_c) {
            constexpr bool CLAMP = decltype(clamp_c)::value;
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                if ((j / L::PAIR) % 2 != 0) continue;
                const int p = col0 + j * L::BLOCK;
                const int f = (p / 64) * 32 + p % 32 + lane % L::BLOCK;
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int r = 0; r < L::REGS; ++r) {
                        const int row = row0 + L::row(i, r, lane);
                        if (row >= M) continue;
                        const float g = acc[i][j][r] * descale, u = acc[i][j + L::PAIR][r] * descale;
                        // silu(g) * u with the hardware reciprocal (1 ulp) instead of an IEEE division: the epilogue is
                        // 48 outputs per lane and the division was half of its instructions
                        h[(int64_t)row * d_ff + f] = Op16<BF>::template store<CLAMP>(g * u * __builtin_amdgcn_rcpf(1.0f + __expf(-g)), peak);
                    }
            }
        };
        store_all(std::false_type());
        if (!(peak <= F16_MAX)) {                           // rare: repeat this lane's stores saturated
            store_all(std::true_type());
            raise_flag(flags, SSD_FLAG_ACT_OVERFLOW);
        }
        }
    }
};

// Stores the scaled accumulator as an fp32 partial sum of one K split: part[split][row][col].
// Whoever consumes it (the RMSNorm that follows) adds the splits in a fixed order.
template <bool BF_>
struct EpiPartial {
    static constexpr bool WANTS_SPLIT = true, BF = BF_, TRANSPOSE = false, USES_LDS = false;
    float* part; int ld; int64_t split_stride; float descale;
    template <int TM, int TN, class L = Layout32>
    __device__ __forceinline__ void operator()(typename L::vec_t (&acc)[TM][TN], int row0, int col0, int M, int lane, int split) const {
        float* base = part + split * split_stride;
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < L::REGS; ++r) {
                const int row = row0 + L::row(i, r, lane);
                if (row >= M) continue;
#pragma unroll
                for (int j = 0; j < TN; ++j) base[(int64_t)row * ld + col0 + L::col(j, lane)] = acc[i][j][r] * descale;
            }
    }
};

// Epilogues for products outside the decoder layer (the projector's windowed cross-attention).
// EpiScoresValues: the product [frames, 64 score columns | d_h value columns | padding] is split on the way out.
// The score columns stay fp32 (they go through an exponential), rows of 64; the value columns are rounded to IEEE
// half (2^-12 relative, an eighth of the bf16 rounding their weighted sums get afterwards; beyond 65504 they
// saturate and SSD_FLAG_ACT_OVERFLOW is raised), rows of d_h: 2.3 KB per frame instead of 5 KB of fp32.
template <bool BF_>
struct EpiScoresValues {
    static constexpr bool WANTS_SPLIT = false, BF = BF_, TRANSPOSE = true, USES_LDS = false;
    float* scores; uint16_t* vals; int d_h; int32_t* flags;
    template <int TM, int TN, class L = Layout32>
    __device__ __forceinline__ void operator()(typename L::vec_t (&acc)[TM][TN], int row0, int col0, int M, int lane) const {
        bool bad = false;
        if constexpr (L::TRANSPOSED) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = row0 + L::row(i, lane);
                if (row >= M) continue;
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const int col = col0 + L::col4(j, lane);           // blocks of 16 columns never straddle column 64
                    if (col < QF_SCORE_COLS)
                        *reinterpret_cast<float4*>(scores + (int64_t)row * QF_SCORE_COLS + col) =
                            make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
                    else if (col - QF_SCORE_COLS < d_h)
                        *reinterpret_cast<uint2*>(vals + (int64_t)row * d_h + (col - QF_SCORE_COLS)) =
                            make_uint2(pack_f16x2_sat(acc[i][j][0], acc[i][j][1], bad), pack_f16x2_sat(acc[i][j][2], acc[i][j][3], bad));
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int r = 0; r < L::REGS; ++r) {
                    const int row = row0 + L::row(i, r, lane);
                    if (row >= M) continue;
#pragma unroll
                    for (int j = 0; j < TN; ++j) {
                        const int col = col0 + L::col(j, lane);
                        if (col < QF_SCORE_COLS) scores[(int64_t)row * QF_SCORE_COLS + col] = acc[i][j][r];
                        else if (col - QF_SCORE_COLS < d_h) vals[(int64_t)row * d_h + (col - QF_SCORE_COLS)] = f32_to_f16_sat(acc[i][j][r], bad);
                    }
                }
        }
        if (bad) raise_flag(flags, SSD_FLAG_ACT_OVERFLOW);
    }
};
template <bool BF_>
struct EpiStore16 {
    static constexpr bool WANTS_SPLIT = false, BF = BF_, TRANSPOSE = true, USES_LDS = false;
    uint16_t* c; int ldc;
    template <int TM, int TN, class L = Layout32>
    __device__ __forceinline__ void operator()(typename L::vec_t (&acc)[TM][TN], int row0, int col0, int M, int lane) const {
        if constexpr (L::TRANSPOSED) {
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                const int row = row0 + L::row(i, lane);
                if (row >= M) continue;
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    *reinterpret_cast<uint2*>(c + (int64_t)row * ldc + col0 + L::col4(j, lane)) =
                        make_uint2(op_pack2<BF>(acc[i][j][0], acc[i][j][1]), op_pack2<BF>(acc[i][j][2], acc[i][j][3]));
            }
            return;
        } else {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int r = 0; r < L::REGS; ++r) {
                const int row = row0 + L::row(i, r, lane);
                if (row >= M) continue;
#pragma unroll
                for (int j = 0; j < TN; ++j) c[(int64_t)row * ldc + col0 + L::col(j, lane)] = Op16<BF>::cvt(acc[i][j][r]);
            }
        }
    }
};

// The same from the 256-wide tiles through the workgroup's LDS (free after the K loop): a wavefront's 64 columns of a row are one
// 128-byte line, written by eight lanes with 16 bytes each instead of sixteen with 8 that lie 16 lane ids apart.  Projector
// output, 39700 rows of 3072 from K = 1024 (244 MB stored): 267 -> 254 us; 3000 rows 25.2 -> 23.7.  (The SwiGLU epilogue in the same way, 64
// bytes a row: gate/up of 2048 0.9 % faster, of 3072 the same: not taken.)
constexpr int ST_LDS_STRIDE = 72;                            // 16-bit values per staged row: 64 + 8
template <bool BF_>
struct EpiStore16Lds {
    static constexpr bool WANTS_SPLIT = false, BF = BF_, TRANSPOSE = true, USES_LDS = true;
    uint16_t* c; int ldc;
    template <int TM> static constexpr int wave_lds_bytes() { return TM * 16 * ST_LDS_STRIDE * 2; }
    template <int TM, int TN>
    __device__ __forceinline__ void run_lds(f32x4_t (&acc)[TM][TN], int row0, int col0, int M, int lane, float* stage_f) const {
        static_assert(TN == 4, "a wavefront tile of 64 columns");
        uint16_t* stage = reinterpret_cast<uint16_t*>(stage_f);
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
                *reinterpret_cast<uint2*>(stage + Layout16T::row(i, lane) * ST_LDS_STRIDE + Layout16T::col4(j, lane)) =
                    make_uint2(op_pack2<BF>(acc[i][j][0], acc[i][j][1]), op_pack2<BF>(acc[i][j][2], acc[i][j][3]));
        __builtin_amdgcn_s_waitcnt(0xC07F);                  // lgkmcnt(0): the stores have landed
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < TM * 2; ++it) {
            const int r = 8 * it + lane / 8, row = row0 + r;
            const uint4 v = *reinterpret_cast<const uint4*>(stage + r * ST_LDS_STRIDE + 8 * (lane % 8));
            if (row < M) *reinterpret_cast<uint4*>(c + (int64_t)row * ldc + col0 + 8 * (lane % 8)) = v;
        }
    }
};

// grid = tiles * splits; split s of a tile accumulates K slices [s*KT/splits, (s+1)*KT/splits)
template <int BM, int BN, int WAVES_M, int WAVES_N, int NSTAGE, class Epi>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N)
gemm_mfma_kernel(const f16_t* __restrict__ A, const f16_t* __restrict__ W, int M, int N, int K, int splits, Epi epi) {
    using Tile = GemmTile<BM, BN, WAVES_M, WAVES_N, NSTAGE, Epi::BF>;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int tiles_m = (M + BM - 1) / BM, tiles_n = N / BN;
    const int split = blockIdx.x % splits;
    int tm, tn;
    tile_of_workgroup(blockIdx.x / splits, tiles_m * tiles_n, tiles_m, tiles_n, tm, tn);
    const int KT = K / GEMM_BK;
    const int kt0 = (int)((int64_t)KT * split / splits), kt1 = (int)((int64_t)KT * (split + 1) / splits);
    f32x16_t acc[Tile::TM][Tile::TN];
#pragma unroll
    for (int i = 0; i < Tile::TM; ++i)
#pragma unroll
        for (int j = 0; j < Tile::TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    Tile::run(A, W, M, K, tm * BM, tn * BN, kt0, kt1, smem_raw, acc);
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    if constexpr (Epi::WANTS_SPLIT)
        epi.template operator()<Tile::TM, Tile::TN>(acc, tm * BM + wm * Tile::WTM, tn * BN + wn * Tile::WTN, M, lane, split);
    else
        epi.template operator()<Tile::TM, Tile::TN>(acc, tm * BM + wm * Tile::WTM, tn * BN + wn * Tile::WTN, M, lane);
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int NSTAGE, class Epi>
static void launch_gemm(const f16_t* A, const f16_t* W, int M, int N, int K, int splits, const Epi& epi, hipStream_t st) {
    if (M <= 0) return;
    auto kern = gemm_mfma_kernel<BM, BN, WAVES_M, WAVES_N, NSTAGE, Epi>;
    constexpr size_t lds = gemm_lds_bytes<BM, BN, NSTAGE>();
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        attr_set = true;
    }
    const int tiles = ((M + BM - 1) / BM) * (N / BN);
    hipLaunchKernelGGL(kern, dim3(tiles * splits), dim3(64 * WAVES_M * WAVES_N), lds, st, A, W, M, N, K, splits, epi);
}

// One-wavefront tile with the K range split over KG wavefronts of the workgroup, each with its own LDS ring; the
// partial accumulators are added through LDS in group order (deterministic), a quarter of the tile per group, with the epilogue.  For
// projections with few rows, few column tiles and an epilogue that needs whole sums (QKV + RoPE at 33-128 rows): a
// CU then keeps KG rings of weight and activation slices in flight instead of one.
template <int BM, int BN, int NSTAGE, int KG, class Epi>
__global__ void __launch_bounds__(64 * KG)
gemm_mfma_kgroups_kernel(const f16_t* __restrict__ A, const f16_t* __restrict__ W, int M, int N, int K, Epi epi) {
    using Tile = GemmTile<BM, BN, 1, 1, NSTAGE, Epi::BF>;
    constexpr int RING = (int)gemm_lds_bytes<BM, BN, NSTAGE>();
    constexpr int ACC_FLOATS = Tile::TM * Tile::TN * 16;               // per lane
    static_assert(ACC_FLOATS * 64 * 4 <= RING, "a group's partial tile must fit its ring");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int tiles_m = (M + BM - 1) / BM, tiles_n = N / BN;
    int tm, tn;
    tile_of_workgroup(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, tm, tn);
    const int g = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const int per = K / GEMM_BK / KG;                                   // the launcher checks divisibility
    f32x16_t acc[Tile::TM][Tile::TN];
#pragma unroll
    for (int i = 0; i < Tile::TM; ++i)
#pragma unroll
        for (int j = 0; j < Tile::TN; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    Tile::run(A, W, M, K, tm * BM, tn * BN, g * per, (g + 1) * per, smem_raw + g * RING, acc);
    // a group's ring is read by that group only and all its reads have completed: it may hold the partial tile
    static_assert(Tile::TM == 1 && Tile::TN == 2, "finish_quarter takes 32 x 64 blocks");
    store_partial(reinterpret_cast<float4*>(smem_raw + g * RING), acc[0], lane);
    __syncthreads();
    for (int q = g; q < 4; q += KG) finish_quarter<KG>(reinterpret_cast<const float4*>(smem_raw), RING / 16, q, tm * BM, tn * BN, M, lane, 0, epi);
}

template <int BM, int BN, int NSTAGE, int KG, class Epi>
static void launch_gemm_kgroups(const f16_t* A, const f16_t* W, int M, int N, int K, const Epi& epi, hipStream_t st) {
    if (M <= 0) return;
    auto kern = gemm_mfma_kgroups_kernel<BM, BN, NSTAGE, KG, Epi>;
    constexpr size_t lds = KG * gemm_lds_bytes<BM, BN, NSTAGE>();
    static_assert(lds <= 160 * 1024, "LDS of a compute unit");
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        attr_set = true;
    }
    const int tiles = ((M + BM - 1) / BM) * (N / BN);
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(64 * KG), lds, st, A, W, M, N, K, epi);
}

// Big tiles on v_mfma_f32_16x16x32_f16 (gemm_core16.h): same tile shapes, workgroup order, K splits and epilogues.
template <int BM, int BN, int WAVES_M, int WAVES_N, class Epi>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N)
gemm_mfma16_kernel(const f16_t* __restrict__ A, const f16_t* __restrict__ W, int M, int N, int K, int splits, Epi epi) {
    using Tile = GemmTile16<BM, BN, WAVES_M, WAVES_N, Epi::BF, Epi::TRANSPOSE>;   // transposed accumulator blocks where the epilogue gains from them
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int tiles_m = (M + BM - 1) / BM, tiles_n = N / BN;
    int tm, tn;
    const int split = blockIdx.x % splits;
    tile_of_workgroup(blockIdx.x / splits, tiles_m * tiles_n, tiles_m, tiles_n, tm, tn);
    const int KT = K / GEMM_BK;
    f32x4_t acc[Tile::TM][Tile::TN];
#pragma unroll
    for (int i = 0; i < Tile::TM; ++i)
#pragma unroll
        for (int j = 0; j < Tile::TN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
    Tile::run(A, W, M, K, tm * BM, tn * BN, KT * split / splits, KT * (split + 1) / splits, smem_raw, acc);
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int wm = wave / WAVES_N, wn = wave % WAVES_N;
    if constexpr (Epi::USES_LDS)
        epi.template run_lds<Tile::TM, Tile::TN>(acc, tm * BM + wm * Tile::WTM, tn * BN + wn * Tile::WTN, M, lane,
                                                 reinterpret_cast<float*>(smem_raw + wave * Epi::template wave_lds_bytes<Tile::TM>()));
    else if constexpr (Epi::WANTS_SPLIT)
        epi.template operator()<Tile::TM, Tile::TN, Layout16>(acc, tm * BM + wm * Tile::WTM, tn * BN + wn * Tile::WTN, M, lane, split);
    else if constexpr (Epi::TRANSPOSE)
        epi.template operator()<Tile::TM, Tile::TN, Layout16T>(acc, tm * BM + wm * Tile::WTM, tn * BN + wn * Tile::WTN, M, lane);
    else
        epi.template operator()<Tile::TM, Tile::TN, Layout16>(acc, tm * BM + wm * Tile::WTM, tn * BN + wn * Tile::WTN, M, lane);
}

// the epilogue of the 256-wide tiles' kernels that stands for one
template <class Epi> const Epi& big_tile_epilogue(const Epi& e) { return e; }
template <bool BF> EpiStore16Lds<BF> big_tile_epilogue(const EpiStore16<BF>& e) { return {e.c, e.ldc}; }

template <int BM, int BN, int WAVES_M, int WAVES_N, class Epi>
static void launch_gemm16(const f16_t* A, const f16_t* W, int M, int N, int K, int splits, const Epi& epi, hipStream_t st) {
    if (M <= 0) return;
    auto kern = gemm_mfma16_kernel<BM, BN, WAVES_M, WAVES_N, Epi>;
    constexpr size_t ring = GemmTile16<BM, BN, WAVES_M, WAVES_N, Epi::BF, Epi::TRANSPOSE>::LDS_BYTES;
    constexpr size_t lds = [] {
        if constexpr (Epi::USES_LDS) {
            constexpr size_t stage = (size_t)WAVES_M * WAVES_N * Epi::template wave_lds_bytes<BM / WAVES_M / 16>();
            return stage > ring ? stage : ring;
        } else {
            return ring;
        }
    }();
    static_assert(lds <= 160 * 1024, "LDS of a compute unit");
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        attr_set = true;
    }
    const int tiles = ((M + BM - 1) / BM) * (N / BN);
    hipLaunchKernelGGL(kern, dim3(tiles * splits), dim3(64 * WAVES_M * WAVES_N), lds, st, A, W, M, N, K, splits, epi);
}

// Register-streaming kernel for at most 32 rows (gemm_stream.h); it reads the stream-layout copy of the
// weights.  A workgroup takes K/64/splits steps of 64; they must divide evenly over 8 or 4 wavefronts.
constexpr int STREAM_MAX_ROWS = 32;
template <int NW, int DEPTH, int AQ, class Epi>
static void launch_stream_pieces(const f16_t* A, const void* Ws, int M, int N, int K, int splits, const Epi& epi, hipStream_t st) {
    auto kern = gemm_stream_kernel<NW, DEPTH, AQ, Epi::BF, Epi>;
    constexpr size_t lds = gemm_stream_lds_bytes<NW, DEPTH>();
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3((N / 64) * splits), dim3(64 * NW), lds, st, A, static_cast<const u32x4_t*>(Ws), M, N, K, splits, epi);
}
// Loads of rows that do not exist take the address path of ones that do, and their outputs the time of the epilogue.  Eight greedy steps, 32
// rows' worth / as many eights as there are: 2048 wide, 1 row 8.76 / 8.33 ms, 8 rows 9.29 / 8.82, 16 rows 9.62 / 9.34, 24 rows 10.03 / 9.83; 3072 wide, 2 rows 15.66 /
// 14.75, 8 rows 16.17 / 15.39, 16 rows 16.45 / 16.09.
template <int NW, int DEPTH, class Epi>
static void launch_stream_cfg(const f16_t* A, const void* Ws, int M, int N, int K, int splits, const Epi& epi, hipStream_t st) {
    if (M <= 8) launch_stream_pieces<NW, DEPTH, 1>(A, Ws, M, N, K, splits, epi, st);
    else if (M <= 16) launch_stream_pieces<NW, DEPTH, 2>(A, Ws, M, N, K, splits, epi, st);
    else if (M <= 24) launch_stream_pieces<NW, DEPTH, 3>(A, Ws, M, N, K, splits, epi, st);
    else launch_stream_pieces<NW, DEPTH, 4>(A, Ws, M, N, K, splits, epi, st);
}
template <int R, int NW, int D, class Epi>
static void launch_stream_rows(const f16_t* A, const void* Ws, int M, int N, int K, int splits, const Epi& epi, hipStream_t st) {
    auto kern = gemm_stream_rows_kernel<R, NW, D, Epi::BF, Epi>;
    constexpr size_t lds = gemm_stream_rows_lds_bytes<R, NW, D>();
    static_assert(lds <= 160 * 1024, "LDS of a compute unit");
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        attr_set = true;
    }
    const int row_tiles = (M + 32 * R - 1) / (32 * R);
    hipLaunchKernelGGL(kern, dim3((N / 64) * splits * row_tiles), dim3(64 * NW), lds, st, A, static_cast<const u32x4_t*>(Ws), M, N, K, splits, row_tiles, epi);
}
bool stream_layout_supported(int N, int K) { return N > 0 && K > 0 && N % 64 == 0 && K % 256 == 0; }
static bool stream_shape_ok(int M, int N, int K, int splits) {
    if (M <= 0 || M > STREAM_MAX_ROWS || !stream_layout_supported(N, K) || splits < 1) return false;
    if ((int64_t)M * K * 2 >= (int64_t)1 << 32) return false;
    const int KT = K / 64;
    return KT % splits == 0 && (KT / splits) % 4 == 0;
}
template <class Epi>
static bool try_launch_stream(const f16_t* A, const void* Ws, int M, int N, int K, int splits, const Epi& epi, hipStream_t st) {
    if (!Ws || !stream_shape_ok(M, N, K, splits)) return false;
    const int per = K / 64 / splits;
    const int nw = per % 8 == 0 ? 8 : 4;
    const int steps = per / nw;
    const int depth = steps % 4 == 0 ? 4 : steps % 3 == 0 ? 3 : steps % 2 == 0 ? 2 : 1;
#define SSD_STREAM_CASE(NW_, D_) if (nw == NW_ && depth == D_) { launch_stream_cfg<NW_, D_>(A, Ws, M, N, K, splits, epi, st); return true; }
    SSD_STREAM_CASE(8, 4) SSD_STREAM_CASE(8, 3) SSD_STREAM_CASE(8, 2) SSD_STREAM_CASE(8, 1)
    SSD_STREAM_CASE(4, 4) SSD_STREAM_CASE(4, 3) SSD_STREAM_CASE(4, 2) SSD_STREAM_CASE(4, 1)
#undef SSD_STREAM_CASE
    return false;
}
// 33..128 rows from the stream layout (gemm_stream_rows_kernel), where it is faster than the LDS-ring tiles.  Times in us
// of one launch with cold weights, stream / ring, at d_model 2048 and 3072:
//   gate/up, 48 rows 15.5 / 19.9 and 20.9 / 28.1, 70 rows 17.7 / 20.5 and 23.4 / 28.6, 116 rows 19.9 / 21.3 and 28.6 / 29.2
//   K splits, at most 64 rows: down 9.8 / 12.6 and 12.9 / 16.7, O 5.4 / 5.9 and 7.3 / 8.9, QKV 6.7 / 8.5 and 9.6 / 12.4
//   K splits, 65..96 rows: down 11.6 / 13.2 and 15.4 / 18.1 (16 and 25 K steps per workgroup), QKV 3072 11.7 / 13.0 (16),
//     but O 7.2 / 6.3 and 9.2 / 9.4 (4 and 9), QKV 2048 8.9 / 8.7 (8): short K ranges don't pay for adding three row blocks
//     (these with two wavefronts of three stages; four of two, from 8 K steps on, and two stages instead of three for whole sums:
//     eight greedy steps, 3072 wide, 70 rows 22.35 -> 22.15 ms, 90 rows 23.52 -> 23.06, 2048 wide 13.20 -> 13.09 and 14.23 -> 13.88)
//   K splits, 97..128 rows: O 8.1 / 6.8, down 13.5 / 14.0 and 17.7 / 17.7, with two wavefronts of three stages; four of two, which are faster at
//     65..96 rows, were not measured here
//   whole QKV sums: the in-workgroup K split is faster (10.4 and 14.8 at 70 rows) while its row tiles of 32 give at most one
//     workgroup per CU; with 320 of them (116 rows, 5120 columns) 27.5 against 17.5 here with two row tiles of 64
// (The limits of 8 K steps and 96 column tiles lie between these two widths' figures; no other width was measured.)
// Two wavefronts per workgroup rather than four: half of the partial products to be added at the end (O at 48 rows 6.8 -> 5.4); at 65..96
// rows what a step has in flight counts more.
template <class Epi>
static bool try_launch_stream_rows(const f16_t* A, const void* Ws, int M, int N, int K, int splits, const Epi& epi, hipStream_t st) {
    if (M <= STREAM_MAX_ROWS || M > SKINNY_MAX_ROWS || !stream_layout_supported(N, K) || (int64_t)N * K * 2 >= (int64_t)1 << 31) return false;
    const int KT = K / 64;
    if constexpr (Epi::WANTS_SPLIT) {
        if (KT < 2 * splits) return false;                   // every wavefront needs a step
        if (M <= 64) launch_stream_rows<2, 2, 2>(A, Ws, M, N, K, splits, epi, st);
        else if (M <= 96 && KT >= 8 * splits) launch_stream_rows<3, 4, 2>(A, Ws, M, N, K, splits, epi, st);
        else return false;
    } else {
        if (splits != 1 || KT < 4) return false;
        if (N / 64 <= 96) {                                  // few column tiles
            if ((N / 64) * ((M + 31) / 32) <= 256) return false;
            launch_stream_rows<2, 4, 4>(A, Ws, M, N, K, 1, epi, st);
        }
        else if (M <= 64) launch_stream_rows<2, 2, 4>(A, Ws, M, N, K, 1, epi, st);
        else if (M <= 96) launch_stream_rows<3, 2, 2>(A, Ws, M, N, K, 1, epi, st);
        else launch_stream_rows<4, 2, 2>(A, Ws, M, N, K, 1, epi, st);
    }
    return true;
}
void launch_stream_layout(const uint16_t* w, void* out, int N, int K, hipStream_t st) {
    const int64_t units = (int64_t)N * K / 8;
    hipLaunchKernelGGL(stream_layout_kernel, dim3((unsigned)((units + 255) / 256)), dim3(256), 0, st,
                       reinterpret_cast<const u32x4_t*>(w), static_cast<u32x4_t*>(out), N, K);
}

// Tile choice.  All candidates use eight wavefronts as 2 x 4 and a 256-wide tile (N is a multiple
// of 256 for every GEMM here) on the 16x16x32 matrix instruction; the tile height is picked per launch
// so that the number of tiles wastes as little of the last round over the 256 CUs as possible:
// cost = rounds * (height * K / efficiency + what a round costs beside its K loop: first loads, epilogue, the burst of stores).
// The last term is TILE_OVERHEAD row-slices, about eleven slices of the highest tile: 40 K x 3072 outputs of K = 1024 take 290 us
// in ten rounds of 192 rows and 268 us in eight of 256.  Five heights because a coarser step leaves up to a quarter of a round
// empty (256, 192 and 128 only, against these, us: QKV of 3400 rows 68.9 -> 62.4 and 136.6 -> 125.2 at 2048 and 3072 wide, gate/up of
// 2600 rows 162.5 -> 149.4, down of 4200 rows 166 -> 157, of 6400 rows 196 -> 184 and 327 -> 310).  Over 30 row counts from 2100 to 15214
// and four projections at two widths the rule is 0.04 % from the best of the five heights on average and 2 % at most.  (Tiles of 160 rows,
// which three ring stages fit since their pieces have no padding: QKV of 4620 rows of 2048, two rounds, 97 -> 86.7 us, 192 rows 94.)
// With at most 128 rows the job is weight streaming and what counts is the number of weight bytes in
// flight: at most 32 rows go to the register-streaming kernel when the shape divides evenly, more to its variant
// with row blocks where that is faster (try_launch_stream_rows); otherwise a skinny 128 x 64 tile (four wavefronts, each 32 rows x 64 columns) with a six-stage LDS ring
// (144 KB, five slices in flight), and for at most 32 rows a 32 x 64 tile of one wavefront, six stages
// of 12 KB, two workgroups per CU.
// four K groups, at least four slices each
static bool kgroups_shape_ok(int K) { return (K / GEMM_BK) % 4 == 0 && K / GEMM_BK >= 16; }
template <class Epi>
static void launch_skinny(const f16_t* A, const f16_t* W, const void* Ws, int M, int N, int K, int splits, const Epi& epi, hipStream_t st) {
    if (try_launch_stream(A, Ws, M, N, K, splits, epi, st)) return;
    if (Ws && try_launch_stream_rows(A, Ws, M, N, K, splits, epi, st)) return;
    // 33..128 rows through the LDS ring: the launch should put a workgroup on every CU.  A projection with few column
    // tiles and no K split (QKV: 64-80 tiles) is cut into row tiles of 32 or 64 as well; the row tiles of a column slab
    // then read the same weights, which the L2 serves.
    const int col_tiles = (N / 64) * splits;
    if constexpr (!Epi::WANTS_SPLIT) {
        // whole sums wanted (no K split across workgroups) and few column tiles: split K inside the workgroup
        if (col_tiles <= 96 && M > 32 && kgroups_shape_ok(K)) {
            launch_gemm_kgroups<32, 64, 3, 4>(A, W, M, N, K, epi, st);
            return;
        }
    }
    if (M <= 32 || (col_tiles <= 96 && M > 32)) launch_gemm<32, 64, 1, 1, 6>(A, W, M, N, K, splits, epi, st);
    else if (col_tiles <= 160 && M > 64) launch_gemm<64, 64, 2, 1, 6>(A, W, M, N, K, splits, epi, st);
    else launch_gemm<128, 64, 4, 1, 6>(A, W, M, N, K, splits, epi, st);
}

template <class Epi>
static void launch_big(const f16_t* A, const f16_t* W, int M, int N, int K, const Epi& small_epi, hipStream_t st) {
    const auto& epi = big_tile_epilogue(small_epi);
    const int heights[5] = {256, 224, 192, 160, 128};
    const double eff[5] = {1.0, 0.98, 0.96, 0.94, 0.86};
    constexpr double TILE_OVERHEAD = 2800;
    int best = 0;
    double best_cost = 1e30;
    for (int c = 0; c < 5; ++c) {
        const long tiles = (long)((M + heights[c] - 1) / heights[c]) * (N / 256);
        const long rounds = (tiles + 255) / 256;
        const double cost = (double)rounds * (heights[c] / eff[c] * (K / GEMM_BK) + TILE_OVERHEAD);
        if (cost < best_cost - 1e-9) { best_cost = cost; best = c; }
    }
    if (best == 0) launch_gemm16<256, 256, 2, 4>(A, W, M, N, K, 1, epi, st);
    else if (best == 1) launch_gemm16<224, 256, 2, 4>(A, W, M, N, K, 1, epi, st);
    else if (best == 2) launch_gemm16<192, 256, 2, 4>(A, W, M, N, K, 1, epi, st);
    else if (best == 3) launch_gemm16<160, 256, 2, 4>(A, W, M, N, K, 1, epi, st);
    else launch_gemm16<128, 256, 2, 4>(A, W, M, N, K, 1, epi, st);
}
// Whole sums (QKV, gate/up, the projector).  Beyond 128 rows the 256-wide tiles leave most of the chip idle until there
// are about 256 of them, and a workgroup then has its whole K range in front of it whatever the row count.  Narrower tiles are
// faster while they run in one round, the narrowest that do: 32 x 64 with K split over four wavefronts, 64 x 64 (LDS ring), 64 x 128,
// 128 x 128 of eight wavefronts.  (The projector's fused product, 1088 columns of K = 1024, 250 frames: 6.0 us as 32 x 64, 10.8 as 64 x 64; 1250
// frames: 12.0 us in the one round of 64 x 128 that it is without columns of padding.  N is rounded up to the tile's width.)
// Cold weights, us, 2048 / 3072 wide: QKV of 136 rows 16.0 / 21.8 as 64 x 64 (18.2 / 25.2 as 64 x 128), 256 rows of 3072 26.6 as 64 x 128
// (34.6 as 128 x 128), 512 rows of 2048 19.5 as 64 x 128 (23.6), 640 rows 23.9 / 34.7 as 128 x 128 (27.9 / 41.5 as two rounds of
// 64 x 128), 980 rows of 2048 27.6 as 128 x 128 (34.4 as 128 x 256); gate/up of 256 rows 26.3 / 38.8 as 128 x 128 (32.1 / 47.0 as 64 x 128).
template <class Epi>
static void launch_by_shape(const f16_t* A, const f16_t* W, const void* Ws, int M, int N, int K, const Epi& epi, hipStream_t st) {
    auto cols = [&](int bn) { return (N + bn - 1) / bn * bn; };
    auto tiles = [&](int bm, int bn) { return (int64_t)((M + bm - 1) / bm) * (cols(bn) / bn); };
    if (M <= SKINNY_MAX_ROWS) launch_skinny(A, W, Ws, M, cols(64), K, 1, epi, st);
    else if (tiles(32, 64) <= 256 && kgroups_shape_ok(K)) launch_gemm_kgroups<32, 64, 3, 4>(A, W, M, cols(64), K, epi, st);
    else if (tiles(64, 64) <= 256) launch_gemm<64, 64, 2, 1, 6>(A, W, M, cols(64), K, 1, epi, st);
    else if (tiles(64, 128) <= 256) launch_gemm16<64, 128, 2, 2>(A, W, M, cols(128), K, 1, big_tile_epilogue(epi), st);
    else if (tiles(128, 128) <= 256) launch_gemm16<128, 128, 4, 2>(A, W, M, cols(128), K, 1, big_tile_epilogue(epi), st);
    else launch_big(A, W, M, cols(256), K, epi, st);
}

void launch_gemm_qkv_rope(const uint16_t* A, const uint16_t* Wqkv_packed, const void* W_stream, uint16_t* qkv, const int32_t* pos,
                          const float* rope_tab, int M, int d_model, int d_q, int d_kv, float descale,
                          const int32_t* row_slot, uint16_t* kc, uint16_t* vc, const float* rope_rows, int32_t* flags,
                          bool bf16_ops, hipStream_t st) {
    const int N = d_q + 2 * d_kv;
    if (bf16_ops) {
        EpiQkvRope<true> epi{qkv, N, d_q + d_kv, descale, pos, reinterpret_cast<const float2*>(rope_tab), row_slot, kc, vc, d_q,
                             reinterpret_cast<const float2*>(rope_rows), flags};
        launch_by_shape(A, Wqkv_packed, W_stream, M, N, d_model, epi, st);
    } else {
        EpiQkvRope<false> epi{qkv, N, d_q + d_kv, descale, pos, reinterpret_cast<const float2*>(rope_tab), row_slot, kc, vc, d_q,
                              reinterpret_cast<const float2*>(rope_rows), flags};
        launch_by_shape(A, Wqkv_packed, W_stream, M, N, d_model, epi, st);
    }
}

int launch_gemm_qkv_partial(const uint16_t* A, const uint16_t* W, const void* W_stream, float* part, int M, int d_model, int N, float descale,
                            bool bf16_ops, hipStream_t st) {
    if (!W_stream || M > SKINNY_MAX_ROWS) return 0;
    int splits = 0;
    if (M <= STREAM_MAX_ROWS) {
        for (int s = SKINNY_MAX_SPLITS; s >= 2 && !splits; --s)             // about one workgroup per CU
            if (stream_shape_ok(M, N, d_model, s) && (N / 64) * s <= 320) splits = s;
    } else {
        splits = min(min(SKINNY_MAX_SPLITS, 256 / (N / 64)), d_model / GEMM_BK / 4);
    }
    if (splits < 2) return 0;
    if (bf16_ops) launch_skinny(A, W, W_stream, M, N, d_model, splits, EpiPartial<true>{part, N, (int64_t)M * N, descale}, st);
    else launch_skinny(A, W, W_stream, M, N, d_model, splits, EpiPartial<false>{part, N, (int64_t)M * N, descale}, st);
    return splits;
}

// Residual projections of more than 128 rows.  Unsplit in 256-wide tiles, a workgroup walks the whole K range (down, K = 8192, of
// 136 to 1568 rows: 132-136 us), so K is split, or the tile is narrower, until one round fills the CUs.  Three tiles, up to eight
// splits: the cheapest by
//   us = fixed + K steps of a workgroup * (step + busy * workgroups / 256) + MB of split sums * (write + read by the RMSNorm)
// fitted to 700 launches (O and down of 136 to 1960 rows at 2048 and 3072 columns, cold weights; 7-9 % off on average), which picks
// within 2 % of the best of ten tiles on average and 11 % at worst.  At 392 rows of 2048 columns: O 9.6 us (two splits of 128 x 64), down
// 21.6 (four of 128 x 128); 128 x 256 tiles with eight splits 10.2 and 23.8, and a norm that reads twice the sums.  Without a split the
// projection adds to x in place: from the row count at which 128 x 128 tiles alone fill the round.
struct ResidualSplit { int splits, tile; };                  // tile: 0 128 x 64, 1 128 x 128, 2 128 x 256 or, unsplit, launch_big's choice
static ResidualSplit mid_residual_split(int M, int N, int K) {
    static const struct { int bn, least; double fixed, step, busy, write; } T[3] = {
        {64, 2, 2.6, 0.293, 0.066, 0.335}, {128, 1, 2.1, 0.408, 0.119, 0.302}, {256, 1, 3.7, 0.661, 0.149, 0.206}};
    ResidualSplit best{1, 2};
    double best_us = 1e30;
    for (int t = 0; t < 3; ++t) {
        const int64_t tiles = (int64_t)((M + 127) / 128) * (N / T[t].bn);
        for (int s = T[t].least; s <= SKINNY_MAX_SPLITS; ++s) {
            if (tiles * s > 256 || K / GEMM_BK < 4 * s) break;
            const double mb = (double)M * N * 4e-6 * s;
            const double us = T[t].fixed + K / GEMM_BK / (double)s * (T[t].step + T[t].busy * tiles * s / 256) + mb * (T[t].write + 0.2);
            if (us < best_us) { best_us = us; best = {s, t}; }
        }
    }
    return best;
}

int gemm_residual_splits(int M, int N, int K, bool have_stream) {
    if (M > SKINNY_MAX_ROWS) return mid_residual_split(M, N, K).splits;
    if (have_stream && M <= STREAM_MAX_ROWS) {
        // register-streaming kernel: the most splits (workgroups) whose K range still divides over 4 wavefronts
        for (int s = SKINNY_MAX_SPLITS; s >= 2; --s)
            if (stream_shape_ok(M, N, K, s) && (N / 64) * s <= 512) return s;
    }
    // as many as still give every CU at most one workgroup: 3072 columns are 48 tiles, whose 8 splits ran in one and a
    // half rounds (70 rows: O 13.4 us and down 21.8 us, with 5 splits 9.4 and 18.1)
    return max(1, min(min(SKINNY_MAX_SPLITS, 256 / (N / 64)), K / GEMM_BK / 4));
}

// x += A W^T.  Where a launch would leave CUs idle the K range is split over several workgroups per tile to get enough
// of them for weight streaming; the splits land in `partials` ([splits][M][N] fp32) and the caller
// hands them to the next RMSNorm, which adds them to x in a fixed order.  Returns the split count
// (1: x has been updated in place).
template <bool BF>
static int gemm_residual_impl(const uint16_t* A, const uint16_t* W, const void* W_stream, float* x, float* partials, int M, int N, int K,
                              float descale, hipStream_t st) {
    const int splits = gemm_residual_splits(M, N, K, W_stream != nullptr);
    const int tile = M > SKINNY_MAX_ROWS ? mid_residual_split(M, N, K).tile : -1;
    if (splits > 1) {
        EpiPartial<BF> epi{partials, N, (int64_t)M * N, descale};
        if (M <= SKINNY_MAX_ROWS) launch_skinny(A, W, W_stream, M, N, K, splits, epi, st);
        else if (tile == 0) launch_gemm<128, 64, 4, 1, 6>(A, W, M, N, K, splits, epi, st);
        else if (tile == 1) launch_gemm16<128, 128, 4, 2>(A, W, M, N, K, splits, epi, st);
        else launch_gemm16<128, 256, 2, 4>(A, W, M, N, K, splits, epi, st);
        return splits;
    }
    if (tile == 1) launch_gemm16<128, 128, 4, 2>(A, W, M, N, K, 1, EpiResidualLds<BF>{x, N, descale}, st);
    else if (M > SKINNY_MAX_ROWS) launch_big(A, W, M, N, K, EpiResidualLds<BF>{x, N, descale}, st);
    else launch_skinny(A, W, W_stream, M, N, K, 1, EpiResidual<BF>{x, N, descale}, st);
    return 1;
}
int launch_gemm_residual(const uint16_t* A, const uint16_t* W, const void* W_stream, float* x, float* partials, int M, int N, int K,
                         float descale, bool bf16_ops, hipStream_t st) {
    return bf16_ops ? gemm_residual_impl<true>(A, W, W_stream, x, partials, M, N, K, descale, st)
                    : gemm_residual_impl<false>(A, W, W_stream, x, partials, M, N, K, descale, st);
}

void launch_gemm_scores_values(const uint16_t* A, const uint16_t* W, float* scores, uint16_t* vals, int M, int N, int K, int d_h,
                               int32_t* flags, bool bf16_ops, hipStream_t st) {
    if (bf16_ops) launch_by_shape(A, W, nullptr, M, N, K, EpiScoresValues<true>{scores, vals, d_h, flags}, st);
    else launch_by_shape(A, W, nullptr, M, N, K, EpiScoresValues<false>{scores, vals, d_h, flags}, st);
}
void launch_gemm_scores(const uint16_t* A, const uint16_t* W, float* scores, int M, int K, hipStream_t st) {
    launch_gemm<128, 64, 4, 1, 3>(A, W, M, QF_SCORE_COLS, K, 1, EpiScoresValues<true>{scores, nullptr, 0, nullptr}, st);
}
void launch_gemm_store_16(const uint16_t* A, const uint16_t* W, uint16_t* C, int M, int N, int K, bool bf16_ops, hipStream_t st) {
    if (bf16_ops) launch_by_shape(A, W, nullptr, M, N, K, EpiStore16<true>{C, N}, st);
    else launch_by_shape(A, W, nullptr, M, N, K, EpiStore16<false>{C, N}, st);
}

void launch_gemm_swiglu(const uint16_t* A, const uint16_t* Wgu_packed, const void* W_stream, uint16_t* h, int M, int d_ff, int K,
                        float descale, int32_t* flags, bool bf16_ops, hipStream_t st) {
    if (bf16_ops) {
        EpiSwiglu<true> epi{h, d_ff, descale, flags};
        launch_by_shape(A, Wgu_packed, W_stream, M, 2 * d_ff, K, epi, st);
    } else {
        EpiSwiglu<false> epi{h, d_ff, descale, flags};
        launch_by_shape(A, Wgu_packed, W_stream, M, 2 * d_ff, K, epi, st);
    }
}

}  // namespace ssd
