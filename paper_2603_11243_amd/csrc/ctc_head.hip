// CTC output layer fused with the frame statistics of the gate.
//
// The encoder's output layer (Sec. 3.1: 1024-wide states, 348 CTC symbols) produces the scores that
// Eq. 2 (greedy symbol per frame) and Eq. 3 (frame entropy) consume.  Here the scores
//     z[t, v] = enc_h[t] . W[v] + b[v]
// only ever exist in MFMA accumulators.  The accumulator blocks are transposed, so that a lane owns one frame and
// four consecutive symbols of a 16x16 block: the per-frame reductions over symbols run inside the lane, with two
// exchanges between the 16-lane groups at the end.  Every wavefront reduces its [frames x 64 symbols] slab to
//     m = max_v z,  arg = lowest v with z = m,  S = sum_v e^(z-m),  W = sum_v e^(z-m) (z-m)
// per frame (16 bytes; slabs of 96 symbols in the widest tiles), and a second small kernel merges the symbol groups of a frame (and mostly goes on to the gate's decisions) into
//     H_t = log S - W / S   ( = -sum_v p log p for p = softmax(z) ),   argmax_t.
// Written per frame: 16 bytes per group of 64 or 96 symbols instead of 2 x 2 bytes per symbol (a store of
// bf16 scores and the gate's load of them).  Operands are the stored bf16 values (bf16 MFMA, exact
// products, fp32 accumulation); the accumulators start at the bias, and symbols added as padding
// have zero weights and bias -inf, i.e. probability zero.
#include <algorithm>

#include "gate_utterance.h"
#include "gemm_core16.h"
#include "ssd_internal.h"

namespace ssd {

constexpr int CH_BN = 128, CH_WIDE = 384;    // symbols per tile
constexpr int CH_GROUP = 64;        // fewest symbols per partial: the width of a wavefront's tile, 96 in the wide tiles
constexpr int CH_PAD = 128;         // symbol count is padded to a multiple of this

// BM frames x BN symbols on v_mfma_f32_16x16x32_bf16 with transposed blocks: a lane has one frame (lane % 16 of a block) and four
// consecutive symbols, the four 16-lane groups of a wavefront share a frame.
template <int BM, int BN, int WM, int WN>
__global__ void __launch_bounds__(64 * WM * WN)
ctc_head_partials_kernel(const uint16_t* __restrict__ enc_h, const uint16_t* __restrict__ w_pad,
                         const float* __restrict__ bias_pad, int n_rows, int d_enc, int V, int V_pad,
                         float4* __restrict__ part) {
    using Tile = GemmTile16<BM, BN, WM, WN, true, true>;
    using L = Layout16T;
    static_assert(Tile::WTN >= CH_GROUP, "one partial per wave tile");
    extern __shared__ __align__(16) unsigned char smem_raw[];
    // symbol tiles vary fastest, and the tiles of one slab of frames run on one XCD (one fetch of the slab)
    const int tiles_v = V_pad / BN;
    const int v = xcd_contiguous_index(blockIdx.x, gridDim.x);
    const int tv = v % tiles_v, tf = v / tiles_v;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int wm = wave / WN, wn = wave % WN;
    const int sym0 = tv * BN + wn * Tile::WTN;            // first symbol of this wavefront
    const int frame0 = tf * BM + wm * Tile::WTM;

    f32x4_t acc[Tile::TM][Tile::TN];
#pragma unroll
    for (int j = 0; j < Tile::TN; ++j) {
        const f32x4_t b4 = *reinterpret_cast<const f32x4_t*>(bias_pad + sym0 + L::col4(j, lane));
#pragma unroll
        for (int i = 0; i < Tile::TM; ++i) acc[i][j] = b4;
    }
    Tile::run(reinterpret_cast<const f16_t*>(enc_h), reinterpret_cast<const f16_t*>(w_pad), n_rows, d_enc, tf * BM, tv * BN, 0,
              d_enc / GEMM_BK, smem_raw, acc);

    if (sym0 >= V) return;                                   // slab made of padding symbols only
    const int group = sym0 / Tile::WTN;
    constexpr float LOG2E = 1.4426950408889634f;
#pragma unroll
    for (int i = 0; i < Tile::TM; ++i) {
        const int frame = frame0 + L::row(i, lane);
        float m = -INFINITY;
#pragma unroll
        for (int j = 0; j < Tile::TN; ++j)
#pragma unroll
            for (int r = 0; r < 4; r += 2) m = fmaxf(m, fmaxf(acc[i][j][r], acc[i][j][r + 1]));
        m = fmaxf(m, __shfl_xor(m, 16));
        m = fmaxf(m, __shfl_xor(m, 32));                     // finite: symbol sym0 is real
        const float mL = m * LOG2E;
        float s = 0.f, w = 0.f;
        int rel = 0x7fffffff;                                // symbol index relative to sym0 + 4 * (lane / 16)
        // descending symbol order: the last match is the lowest index
#pragma unroll
        for (int j = Tile::TN - 1; j >= 0; --j)
#pragma unroll
            for (int r = 3; r >= 0; --r) {
                const float z = acc[i][j][r];
                const float t2 = fmaf(z, LOG2E, -mL);        // (z - m) log2 e  <= 0; -inf for padding
                const float e = __builtin_amdgcn_exp2f(t2);
                s += e;
                w = fmaf(e, fmaxf(t2, -200.f), w);           // e is 0 there; keeps 0 * inf out
                if (z == m) rel = 16 * j + r;
            }
        int arg = rel == 0x7fffffff ? rel : sym0 + 4 * (lane / 16) + rel;
#pragma unroll
        for (int o = 16; o < 64; o *= 2) {
            s += __shfl_xor(s, o);
            w += __shfl_xor(w, o);
            arg = min(arg, __shfl_xor(arg, o));
        }
        if (frame < n_rows && lane < 16)
            part[(int64_t)group * n_rows + frame] = make_float4(m, s, w * (1.0f / LOG2E), __int_as_float(arg));
    }
}

// One thread per frame merges its column groups (coalesced: group-major partials).
__global__ void __launch_bounds__(256) ctc_head_finalize_kernel(const float4* __restrict__ part, int n_groups,
                                                                int n_rows, float* __restrict__ H,
                                                                int32_t* __restrict__ arg) {
    const int row = blockIdx.x * 256 + threadIdx.x;
    if (row >= n_rows) return;
    float M = -INFINITY;
    for (int g = 0; g < n_groups; ++g) M = fmaxf(M, part[(int64_t)g * n_rows + row].x);
    float S = 0.f, W = 0.f;
    int best = 0x7fffffff;
    for (int g = 0; g < n_groups; ++g) {
        const float4 p = part[(int64_t)g * n_rows + row];
        const float shift = p.x - M;                      // <= 0
        const float f = __expf(shift);
        S += f * p.y;
        W += f * (p.z + shift * p.y);
        if (p.x == M) best = min(best, __float_as_int(p.w));
    }
    H[row] = logf(S) - W / S;
    arg[row] = best;
}

// The merge and the second half of the gate in one launch, a workgroup per utterance; H and arg may be null.  Both are small: a launch of
// its own costs the merge more than its work does.  All partials of a frame are requested at once (a group beyond the last is
// a second copy of it and left out).
struct MergeOut { float* H; int32_t* arg; float* max_entropy; uint8_t* gate_pass; int32_t* draft; int32_t* draft_len; };
template <int NG, int WAVES, int AHEAD, class CU>
__global__ void __launch_bounds__(64 * WAVES) ctc_head_utterances_kernel(const float4* __restrict__ part, int n_groups, int n_rows, const CU cu, int blank,
                                                                  float tau, MergeOut out) {
    const int b = blockIdx.x, lo = cu(b), hi = cu(b + 1);
    auto merge = [&](int t, float& h, int& best) {
        float4 p[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) p[g] = part[(int64_t)min(g, n_groups - 1) * n_rows + t];
        float M = p[0].x;
#pragma unroll
        for (int g = 1; g < NG; ++g) M = fmaxf(M, p[g].x);
        float S = 0.f, W = 0.f;
        best = 0x7fffffff;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            if (g >= n_groups) continue;
            const float shift = p[g].x - M, f = __expf(shift);
            S += f * p[g].y;
            W += f * (p[g].z + shift * p[g].y);
            if (p[g].x == M) best = min(best, __float_as_int(p[g].w));
        }
        h = logf(S) - W / S;
    };
    gate_utterance<WAVES, AHEAD>(b, lo, hi, blank, tau, out.max_entropy, out.gate_pass, out.draft, out.draft_len,
                      [&](int t, float& h, int& a) {
                          merge(t, h, a);
                          if (out.H) out.H[t] = h;
                          if (out.arg) out.arg[t] = a;
                      },
                      [&](int t, int a) {                    // the lane before has it; the first lane merges that frame as well
                          float h;
                          int edge;
                          merge(max(__builtin_amdgcn_readfirstlane(t) - 1, lo), h, edge);
                          const int before = __shfl_up(a, 1);
                          return threadIdx.x % 64 == 0 ? edge : before;
                      });
}
// Every trip of a workgroup over its utterance is a chain of memory and barriers, so one trip is made of all frames: four wavefronts with two
// frames a lane up to 512, sixteen with one beyond.  us of the merge and the decisions, their own launches / four / sixteen wavefronts: one
// utterance of 250 frames 5.0 / 3.6 / 3.5, of 1000 6.2 / 6.6 / 4.4, of 2000 6.3 / 11.2 / 6.8 (and a gap between launches less), of 4000 9.5 / 20.6 / 12.0;
// 300 of 212 9.8 / 5.4 / 7.6, 64 of 1000 9.6 / 7.2 / 5.0, 256 of 2000 20.3 / 16.8 / 13.9.
constexpr int MERGE_FEW_FRAMES = 512, MERGE_MAX_FRAMES = 2048, MERGE_MAX_GROUPS = 8;
template <class CU>
static void launch_merge(const float4* part, int n_groups, int n_rows, const CU& cu, int B, int longest, int blank, float tau, const MergeOut& out, hipStream_t st) {
#define SSD_MERGE(NG) do { \
        if (longest <= MERGE_FEW_FRAMES) hipLaunchKernelGGL((ctc_head_utterances_kernel<NG, 4, 2, CU>), dim3(B), dim3(256), 0, st, part, n_groups, n_rows, cu, blank, tau, out); \
        else hipLaunchKernelGGL((ctc_head_utterances_kernel<NG, 16, 1, CU>), dim3(B), dim3(1024), 0, st, part, n_groups, n_rows, cu, blank, tau, out); } while (0)
    if (n_groups <= 2) SSD_MERGE(2); else if (n_groups <= 4) SSD_MERGE(4); else if (n_groups <= 6) SSD_MERGE(6); else SSD_MERGE(MERGE_MAX_GROUPS);
#undef SSD_MERGE
}

template <int BM, int BN, int WM, int WN>
static int launch_partials(const uint16_t* enc_h, const uint16_t* w_pad, const float* bias_pad, int n_rows, int d_enc,
                           int V, int V_pad, float4* part, hipStream_t st) {
    using Tile = GemmTile16<BM, BN, WM, WN, true, true>;
    auto kern = ctc_head_partials_kernel<BM, BN, WM, WN>;
    static bool attr_set = false;
    if (!attr_set) {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)Tile::LDS_BYTES);
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3((n_rows + BM - 1) / BM * (V_pad / BN)), dim3(64 * WM * WN), Tile::LDS_BYTES, st, enc_h, w_pad, bias_pad,
                       n_rows, d_enc, V, V_pad, part);
    return (V + Tile::WTN - 1) / Tile::WTN;
}

int ctc_head_groups(int V) { return (V + CH_GROUP - 1) / CH_GROUP; }
int ctc_head_padded(int V) { return (V + CH_PAD - 1) / CH_PAD * CH_PAD; }

// enc_h [n_rows, d_enc] bf16; w_pad [V_pad, d_enc] bf16 with zero rows beyond V; bias_pad [V_pad] fp32, -inf
// beyond V; part: ctc_head_groups(V) * n_rows float4.  n_rows * d_enc * 2 must stay below 4 GiB.
int launch_ctc_head_partials(const uint16_t* enc_h, const uint16_t* w_pad, const float* bias_pad, int n_rows, int d_enc, int V,
                             int V_pad, float4* part, hipStream_t st) {
    if (n_rows <= 0) return 0;
    auto tiles = [&](int bm, int bn) { return (int64_t)((n_rows + bm - 1) / bm) * (V_pad / bn); };
#define SSD_HEAD(BM, BN, WM, WN) return launch_partials<BM, BN, WM, WN>(enc_h, w_pad, bias_pad, n_rows, d_enc, V, V_pad, part, st)
    // The smallest tile of frames that runs in one round: in 256-frame tiles a few thousand frames leave most CUs idle.  Front end of 275 /
    // 4100 frames 42.7 -> 37.5 / 60.2 -> 50.3 us (mostly this kernel).
    if (tiles(64, CH_BN) <= 256) SSD_HEAD(64, CH_BN, 2, 2);
    if (tiles(128, CH_BN) <= 256) SSD_HEAD(128, CH_BN, 4, 2);
    // More: 256 x 128 tiles fetch the states three times for the paper's 348 symbols and read two LDS bytes for every three that tiles of
    // all 384 columns do.  Those are up to 192 frames high (242 registers) and come in three heights, whose rounds over the CUs
    // take these us at K = 1024.  us of the launch, 256 x 128 / the height that wins: 22 K frames 32.6 / 24.0 (128), 40 K 35.1 / 31.8 (160),
    // 45 K 49.1 / 34.5 (192), 64 K 55.8 / 48.0 (128), 90 K 85.2 / 66.8 (192), 120 K 110 / 87.0 (160), 140 K 138 / 106 (192), 160 K 156 / 137
    // (160), 198 K 179 / 168 (160); up to 21760 frames, one round, 19.2 / 23.9.  The same costs serve every K, although a round's fixed part
    // does not grow with it: of calls with K = 64 to 4096, 100 to 4000 symbols and 250 to 90 K frames one (K = 64, 4000 symbols) was 5 % slower than in
    // 256 x 128 tiles alone, the others no more than 3 %.
    constexpr double NARROW = 18.5, H128 = 26.5, H160 = 32, H192 = 35;
    auto cost = [&](int bm, int bn, double round) { return (double)((tiles(bm, bn) + 255) / 256) * round; };
    if (V_pad % CH_WIDE == 0) {
        const double c128 = cost(128, CH_WIDE, H128), c160 = cost(160, CH_WIDE, H160), c192 = cost(192, CH_WIDE, H192);
        const double least = std::min({c128, c160, c192});
        if (least < cost(256, CH_BN, NARROW)) {
            if (least == c192) SSD_HEAD(192, CH_WIDE, 2, 4);
            if (least == c160) SSD_HEAD(160, CH_WIDE, 2, 4);
            SSD_HEAD(128, CH_WIDE, 2, 4);
        }
    }
    SSD_HEAD(256, CH_BN, 4, 2);
#undef SSD_HEAD
}
void launch_ctc_head_merge(const float4* part, int n_groups, int n_rows, float* H, int32_t* arg, hipStream_t st) {
    if (n_rows <= 0) return;
    hipLaunchKernelGGL(ctc_head_finalize_kernel, dim3((n_rows + 255) / 256), dim3(256), 0, st, part, n_groups, n_rows, H, arg);
}
bool launch_ctc_head_merge_gate(const float4* part, int n_groups, int n_rows, const int32_t* cu_frames, int B, int blank, float tau, float* H, int32_t* arg,
                                float* max_entropy, uint8_t* gate_pass, int32_t* draft, int32_t* draft_len, hipStream_t st) {
    int longest = 0;
    for (int b = 0; b < B; ++b) longest = std::max(longest, cu_frames[b + 1] - cu_frames[b]);
    if (n_groups > MERGE_MAX_GROUPS || longest > MERGE_MAX_FRAMES) return false;
    const MergeOut out{H, arg, max_entropy, gate_pass, draft, draft_len};
    if (B <= GATE_MAX_ARG_UTTS) {
        CuArgs cu;
        for (int b = 0; b <= B; ++b) cu.cu[b] = cu_frames[b];
        launch_merge(part, n_groups, n_rows, cu, B, longest, blank, tau, out, st);
        return true;
    }
    CuPairs cu;
    if (!make_cu_pairs(cu_frames, B, cu)) return false;
    launch_merge(part, n_groups, n_rows, cu, B, longest, blank, tau, out, st);
    return true;
}

// padded copy of the output layer: rows [V, V_pad) are zero and their bias is -inf
__global__ void ctc_head_pack_kernel(const uint16_t* __restrict__ w, const float* __restrict__ bias, int V, int V_pad,
                                     int d_enc, uint16_t* __restrict__ w_pad, float* __restrict__ bias_pad) {
    const int64_t n = (int64_t)V_pad * d_enc;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        w_pad[i] = (i / d_enc < V) ? w[i] : (uint16_t)0;
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < V_pad) bias_pad[c] = c < V ? (bias ? bias[c] : 0.f) : -INFINITY;
}

void launch_ctc_head_pack(const uint16_t* w, const float* bias, int V, int V_pad, int d_enc, uint16_t* w_pad,
                          float* bias_pad, hipStream_t st) {
    const int64_t n = (int64_t)V_pad * d_enc;
    const unsigned grid = (unsigned)std::max<int64_t>((V_pad + 255) / 256, std::min<int64_t>((n + 255) / 256, 4096));
    hipLaunchKernelGGL(ctc_head_pack_kernel, dim3(grid), dim3(256), 0, st, w, bias, V, V_pad, d_enc, w_pad, bias_pad);
}

}  // namespace ssd
