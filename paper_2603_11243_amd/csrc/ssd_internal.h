// Internal declarations shared by the kernel files and the C-ABI layer.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "../../include/ssd.h"

namespace ssd {

// ---- gate.hip
// first half of the gate: frame entropies and greedy labels
void launch_gate_frames(const void* logits, int dtype, int64_t n_rows, int V, float* H, int32_t* arg, hipStream_t st);

// second half of the gate on its own: per-utterance max entropy, threshold test and collapse
// (frame ranges are clamped into [0, n_rows] on the device)
void launch_gate_utterances(const float* H, const int32_t* arg, const int32_t* cu_frames_dev, int64_t n_rows, int B, int blank,
                            float tau, float* max_entropy, uint8_t* gate_pass, int32_t* draft, int32_t* draft_len,
                            hipStream_t st);

// The same with the prefix sums in host memory: they travel as kernel arguments, which spares the call its upload (one ten-second
// utterance 15.2 -> 10.7 us, 400 utterances of 3 to 9 s 23.2 -> 17.4 us, 1024 of 1 to 30 s 76.5 -> 70.5 us).  Up to GATE_MAX_ARG_UTTS
// utterances 1 KB of them as they are;
constexpr int GATE_MAX_ARG_UTTS = 256;
struct CuArray {                             // prefix sums in device memory
    const int32_t* cu;
    __device__ __forceinline__ int operator()(int b) const { return cu[b]; }
};
struct CuArgs {                              // among the kernel's arguments
    int32_t cu[GATE_MAX_ARG_UTTS + 1];
    __device__ __forceinline__ int operator()(int b) const { return cu[b]; }
};
// up to GATE_MAX_PAIR_UTTS of at most 65535 frames: every second prefix sum, and the lengths between in 16 bits (a thousand 32-bit
// sums are more than the 4 KB of arguments a launch has).
constexpr int GATE_MAX_PAIR_UTTS = 1280;
struct CuPairs {
    int32_t even[GATE_MAX_PAIR_UTTS / 2 + 1];
    uint32_t odd[GATE_MAX_PAIR_UTTS / 4];        // two lengths a word
    __device__ __forceinline__ int operator()(int b) const {
        const int p = b / 2;
        return even[p] + (b % 2 ? (int)(odd[p / 2] >> (16 * (p % 2)) & 0xffffu) : 0);
    }
};
bool make_cu_pairs(const int32_t* cu, int B, CuPairs& out);      // false: more utterances or longer ones
bool gate_prefix_fits_arguments(const int32_t* cu, int B);       // as one or the other
// false: they do not fit, nothing was launched
bool launch_gate_utterances_host(const float* H, const int32_t* arg, const int32_t* cu_frames, int64_t n_rows, int B, int blank,
                                 float tau, float* max_entropy, uint8_t* gate_pass, int32_t* draft, int32_t* draft_len,
                                 hipStream_t st);

// Frames and utterances in one launch for batches of few enough frames; false: not served, nothing was launched.  arrived:
// GATE_ARRIVED_BYTES of zeros, which the call leaves as zeros.
constexpr int GATE_ARRIVED_BYTES = GATE_MAX_ARG_UTTS * 64;
bool launch_gate_fused(const void* logits, int dtype, const int32_t* cu_frames, int64_t n_rows, int B, int V, int blank, float tau, float* H, int32_t* arg,
                       float* max_entropy, uint8_t* gate_pass, int32_t* draft, int32_t* draft_len, unsigned* arrived, hipStream_t st);

// ---- ctc_head.hip: output layer of the CTC encoder fused with the frame statistics of the gate
int ctc_head_groups(int V);      // groups of 64 symbols that hold at least one real symbol
int ctc_head_padded(int V);      // symbol count after padding
void launch_ctc_head_pack(const uint16_t* w, const float* bias, int V, int V_pad, int d_enc, uint16_t* w_pad,
                          float* bias_pad, hipStream_t st);
// part: ctc_head_groups(V) * n_rows float4 of scratch; n_rows * d_enc * 2 bytes must stay below 4 GiB
// returns the number of symbol groups it left partials of, at most ctc_head_groups(V)
int launch_ctc_head_partials(const uint16_t* enc_h, const uint16_t* w_pad, const float* bias_pad, int n_rows, int d_enc, int V,
                             int V_pad, float4* part, hipStream_t st);
void launch_ctc_head_merge(const float4* part, int n_groups, int n_rows, float* H, int32_t* arg, hipStream_t st);
// the merge with the second half of the gate, H and arg if they are wanted; false: the symbols, the longest utterance or the batch are too many
bool launch_ctc_head_merge_gate(const float4* part, int n_groups, int n_rows, const int32_t* cu_frames, int B, int blank, float tau, float* H, int32_t* arg,
                                float* max_entropy, uint8_t* gate_pass, int32_t* draft, int32_t* draft_len, hipStream_t st);

// ---- qformer.hip: windowed cross-attention of the projector (Sec. 3.1)
constexpr int QF_SCORE_COLS = 64;    // columns of the fused weight that hold the folded (query, head) score rows
constexpr int QF_MAX_WINDOW = 32;
constexpr int QF_MAX_QUERIES = 4;
struct QWindow { int32_t frame0, n_frames; };
int qformer_cat_rows(int d_h);       // rows of the fused [scores | values] weight, padded to a multiple of 256
// w_cat [qformer_cat_rows(d_h), d_enc] bf16: rows j * n_heads + h hold w_k[head h]^T q_proj[j, head h] / sqrt(d_head),
// rows 64 .. 64 + d_h - 1 hold w_v, the rest is zero
void launch_qformer_fold(const uint16_t* q_proj, const uint16_t* w_k, const uint16_t* w_v, int n_q, int n_heads, int d_h,
                         int d_enc, uint16_t* w_cat, hipStream_t st);
// scores [frames, 64] fp32 and vals [frames, d_h] IEEE half = enc_h w_cat^T; for every window: softmax of its score
// columns over its frames, then the weighted sum of its value columns: o [n_windows * n_q, d_h] bf16
void launch_qformer_pool(const float* scores, const uint16_t* vals, const QWindow* wins, int n_windows, int n_q, int n_heads,
                         int d_h, uint16_t* o, hipStream_t st);
// At most QF_ARG_WINDOWS windows in host memory, as kernel arguments; more of them listed on the device from the prefix sums of the
// frames.  Either spares the upload: the front end of 2 utterances (19 windows) 54.5 -> 42.8 us, of 30 (280) 68.6 -> 59.5, of 300 (3000; the host
// does not build the list either) 204 -> 173.
constexpr int QF_ARG_WINDOWS = 448;
struct QWindowArgs { QWindow w[QF_ARG_WINDOWS]; };
void launch_qformer_pool_host(const float* scores, const uint16_t* vals, const QWindowArgs& wins, int n_windows, int n_q, int n_heads,
                              int d_h, uint16_t* o, hipStream_t st);
void launch_qformer_windows(const CuPairs& cu, int B, int window, QWindow* wins, hipStream_t st);

// ---- qformer_values.hip: the same with the values projected after the pooling; for 16 heads of 64 dims, at most 3 queries and
// windows of at most 16 frames.  w_frag: fragment-ordered copy of w_v [d_h, d_enc].
bool qformer_values_supported(int n_q, int n_heads, int d_h, int d_enc, int window);
void launch_qformer_value_fragments(const uint16_t* w_v, int d_enc, uint16_t* w_frag, hipStream_t st);
void launch_qformer_values(const uint16_t* enc_h, const float* scores, const uint16_t* w_frag, const QWindow* wins, int n_windows, int n_q,
                           int d_enc, uint16_t* o, int32_t* flags, hipStream_t st);

// ---- row metadata built on the host for one verify_forward call
// src code of a decoder row: speech rows hold the speech_emb row index; token rows hold
// SRC_PROMPT | index into prompt_ids or SRC_DRAFT | index into draft_ids.
constexpr int32_t SRC_PROMPT = 0x40000000;
constexpr int32_t SRC_DRAFT = (int32_t)0x80000000u;
constexpr int32_t SRC_MASK = 0x3fffffff;

// One attention work item: a tile of query rows of one utterance.
struct AttnTile {
    int32_t seq_start;   // first decoder row of the utterance
    int32_t seq_len;     // rows in the utterance
    int32_t q_start;     // first query position of this tile (multiple of the tile height)
    int32_t pad;
};

// ---- elementwise.hip
// flags (may be NULL): SSD_FLAG_TOKEN_CLAMPED is raised if a token id had to be clamped into [0, vocab)
void launch_embed_rows(int dtype, const void* speech_emb, const void* embed, const int32_t* prompt_ids,
                       const int32_t* draft_ids, const int32_t* row_src, int M, int d, int vocab, float* x,
                       int32_t* flags, hipStream_t st);
// Metadata of one call small enough for kernel arguments (4 KB with the rest): PARTS arrays of 32-bit words one behind the other, the
// first of them the row sources; part s goes to word at[s] of the workspace and ends before word end[s].
struct EmbedMeta {
    static constexpr int PARTS = 5, WORDS = 960;
    int32_t at[PARTS], end[PARTS];
    uint32_t word[WORDS];
};
void launch_embed_rows_meta(int dtype, const void* speech_emb, const void* embed, const int32_t* prompt_ids, const int32_t* draft_ids,
                            const EmbedMeta& meta, int M, int d, int vocab, float* x, void* ws, int32_t* flags, hipStream_t st);
void launch_gather_rows(const void* src, const int32_t* row_idx, int n_rows, int64_t row_bytes, void* dst, hipStream_t st);
// out[i] = src[idx[i]], passed through table (clamped into [0, n_table)) when table is not NULL
void launch_gather_ids(const int32_t* src, const int32_t* idx, int n, const int32_t* table, int n_table, int32_t* out, hipStream_t st);
// a = rmsnorm(x) * gain;  rows optionally gathered through row_idx (NULL = identity).
// If n_splits > 1, x[row] is first increased by partials[s][row] for s = 0..n_splits-1 (fixed order;
// partials is [n_splits][M][d] fp32) and, when row_idx is NULL, written back.
// flags (may be NULL): SSD_FLAG_ACT_OVERFLOW is raised when a half-precision output had to be saturated
void launch_rmsnorm(int dtype, float* x, const void* gain, const int32_t* row_idx, int n_rows, int d,
                    float eps, void* out, const float* partials, int n_splits, int64_t split_stride, int32_t* flags,
                    bool bf16_ops, hipStream_t st);

// ---- f32_path.hip (all-fp32 decoder)
// qkv = rope(rmsnorm(x) Wqkv^T); rows with row_slot[row] >= 0 (row_slot may be NULL) also go to the K/V cache of the layer
void launch_gemm_f32_qkv(const float* x, const float* gain, float eps, const float* Wqkv, float* qkv, const int32_t* pos,
                         const float* rope_tab, int M, int d_model, int d_q, int d_kv, int head_dim, const int32_t* row_slot,
                         float* kc, float* vc, hipStream_t st);
// h = silu(gate) * up with [gate | up] = rmsnorm(x) Wgu^T.  Row lists (distinct rows) may be NULL: all rows in order
void launch_gemm_f32_swiglu(const float* x, const float* gain, float eps, const float* Wgu, float* h, int M, int d_ff, int d_model,
                            const int32_t* x_rows, hipStream_t st);
// x[x_rows] += A[a_rows] W^T
void launch_gemm_f32_residual(const float* A, const float* W, float* x, int M, int N, int K, const int32_t* a_rows, const int32_t* x_rows,
                              hipStream_t st);
constexpr int F32_ATTN_ROWS = 16;        // query rows of one attention work item
void launch_attn_f32(const float* qkv, float* out, const AttnTile* tiles, int n_tiles, int n_q_heads,
                     int n_kv_heads, int head_dim, hipStream_t st);
void launch_decode_attn_f32(const float* qkv, const float* kc, const float* vc, const int32_t* kv_start, const int32_t* n_ctx, int Br,
                            int n_q_heads, int n_kv_heads, int head_dim, float* out, hipStream_t st);
// partials per group of 64 vocabulary entries, merged by launch_lmhead_finalize
int lmhead_f32_groups(int vocab);
void launch_lmhead_f32(const float* hv, const float* w_lm, const int32_t* targets, int Mv, int d, int vocab, float2* part_ms,
                       float* tgt_logit, int2* part_arg, hipStream_t st);

// ---- gemm_mfma.hip (16-bit MFMA GEMMs with fused epilogues), attn_mfma.hip, lmhead_mfma.hip.
// Activations and converted weights are 16-bit operand patterns: IEEE half, or bfloat16 when bf16_ops is set (the
// context's operand type); `descale` undoes the weight scale (1 for bfloat16 operands).
// row_slot / kc / vc (all or none): rows with row_slot[row] >= 0 also store their rotated k part and their v
// part into the K/V cache of this layer at that slot
// W_stream (may be NULL): the same weights in the stream layout of launch_stream_layout, read when at
// most 128 rows are projected (the rule is in gemm_mfma.hip)
// rope_rows (may be NULL): rope_tab[pos[row]] gathered per row, [M][64] (cos, sin); read instead of pos and rope_tab
void launch_gemm_qkv_rope(const uint16_t* A, const uint16_t* Wqkv_packed, const void* W_stream, uint16_t* qkv, const int32_t* pos,
                          const float* rope_tab, int M, int d_model, int d_q, int d_kv, float descale,
                          const int32_t* row_slot, uint16_t* kc, uint16_t* vc, const float* rope_rows, int32_t* flags,
                          bool bf16_ops, hipStream_t st);
constexpr int SKINNY_MAX_ROWS = 128;     // at most this many decoder rows: weight-streaming GEMM variants
constexpr int SKINNY_MAX_SPLITS = 8;
int gemm_residual_splits(int M, int N, int K, bool have_stream);
// fp32 values the partial sums of a residual projection of at most `rows` rows and d columns need: SKINNY_MAX_SPLITS sums
// per value, but no more than one round of 128 x 256 tiles over 256 CUs (which covers 128 rows of up to 8192 columns)
inline int64_t residual_partial_floats(int64_t rows, int64_t d) {
    const int64_t all = SKINNY_MAX_SPLITS * rows * d, round = (int64_t)128 * 256 * 256;
    return all < round ? all : round;
}
// returns the number of K splits written to `partials` ([splits][M][N] fp32), or 1 if x was updated in place
int launch_gemm_residual(const uint16_t* A, const uint16_t* W, const void* W_stream, float* x, float* partials, int M, int N, int K,
                         float descale, bool bf16_ops, hipStream_t st);
void launch_gemm_swiglu(const uint16_t* A, const uint16_t* Wgu_packed, const void* W_stream, uint16_t* h, int M, int d_ff, int K,
                        float descale, int32_t* flags, bool bf16_ops, hipStream_t st);
// plain products C[M,N] = A[M,K] W[N,K]^T with fp32 accumulation, stored as fp32 or rounded to the operand type
// (N % 256 == 0, K % 64 == 0, row-major 16-bit operands of the type bf16_ops selects)
// C = A W^T with W = [64 score rows | d_h value rows | zero rows up to a multiple of 256], N = 64 + d_h: scores [M, 64] fp32, vals [M, d_h]
// IEEE half (saturating)
void launch_gemm_scores_values(const uint16_t* A, const uint16_t* W, float* scores, uint16_t* vals, int M, int N, int K, int d_h,
                               int32_t* flags, bool bf16_ops, hipStream_t st);
// the score rows of the same W alone: scores [M, 64] fp32 (bfloat16 operands)
void launch_gemm_scores(const uint16_t* A, const uint16_t* W, float* scores, int M, int K, hipStream_t st);
void launch_gemm_store_16(const uint16_t* A, const uint16_t* W, uint16_t* C, int M, int N, int K, bool bf16_ops, hipStream_t st);
// second copy of an f16 weight matrix W[N,K] for the few-row kernel (N % 64 == 0, K % 256 == 0)
bool stream_layout_supported(int N, int K);
void launch_stream_layout(const uint16_t* w, void* out, int N, int K, hipStream_t st);
void launch_attn_mfma(const uint16_t* qkv, uint16_t* out, const AttnTile* tiles, int n_tiles, int n_q_heads,
                      int n_kv_heads, bool bf16_ops, hipStream_t st);
// partial log-sum-exp of the LM head over column groups; see lmhead_mfma.hip
int lmhead_col_groups(int vocab);
void launch_lmhead_mfma(const uint16_t* hv, const uint16_t* w_lm, const int32_t* targets, int Mv, int d,
                        int vocab, float2* part_ms, float* tgt_logit, int2* part_arg, bool want_greedy,
                        float descale, bool bf16_ops, hipStream_t st);
// flags (may be NULL): SSD_FLAG_ACT_OVERFLOW is raised when a log-likelihood is not finite
void launch_lmhead_finalize(const float2* part_ms, const float* tgt_logit, const int2* part_arg, int n_groups,
                            int Mv, float* logp, int32_t* greedy, int32_t* flags, hipStream_t st);

// weight re-layout at context creation
// (bf16 weights are converted to f16 times the power of two `scale`, or kept as they are when scale is 0;
// fp32 weights are copied)
void launch_absmax(int dtype, const void* w, int64_t n, unsigned int* out_bits, hipStream_t st);
// inexact (device counter, may be NULL) is increased by the number of values whose half representation is not exact
void launch_convert_weight(int dtype, const void* w, void* out, int rows, int cols, float scale, unsigned long long* inexact,
                           hipStream_t st);
void launch_pack_qkv(int dtype, const void* wq, const void* wk, const void* wv, void* out, int d_q, int d_kv,
                     int d_model, int head_dim, float scale, unsigned long long* inexact, hipStream_t st);
void launch_pack_gate_up(int dtype, const void* wg, const void* wu, void* out, int d_ff, int d_model, float scale,
                         unsigned long long* inexact, hipStream_t st);

// ---- ar_decode.hip (auto-regressive fallback of the 16-bit models): K/V cache of one layer is K [slots, d_kv],
// V [slots, d_kv] in the operand type
void launch_decode_attn(const void* qkv, const void* kc, const void* vc, const int32_t* kv_start,
                        const int32_t* n_ctx, int Br, int n_q_heads, int n_kv_heads, void* out, bool bf16_ops, hipStream_t st);

// head_dim 128, half precision: decode attention that finishes the QKV projection itself.  qkv_part is
// [n_splits][Br][d_q + 2 d_kv] fp32 partial sums in the packed column order of the fused QKV weight; the
// kernel adds the splits, rotates q and k at position n_ctx[b] - 1 (the number of rows the utterance already
// has in the cache), stores the new k / v row at cache slot kv_start[b] + n_ctx[b] - 1 and attends to the
// cached rows plus the new one.
void launch_decode_attn_fused(const float* qkv_part, int n_splits, const float* rope_tab, void* kc, void* vc,
                              const int32_t* kv_start, const int32_t* n_ctx, int Br, int n_q_heads, int n_kv_heads,
                              void* out, int32_t* flags, bool bf16_ops, hipStream_t st);
// QKV projection left as K-split partial sums for launch_decode_attn_fused; returns the split count, or 0 if
// the shape is not served (then nothing was launched)
int launch_gemm_qkv_partial(const uint16_t* A, const uint16_t* W, const void* W_stream, float* part, int M, int d_model, int N, float descale,
                            bool bf16_ops, hipStream_t st);

// threshold grids: outputs are [n_tau][B] / [n_tau][Bv]
void launch_gate_grid(const float* max_entropy, int B, const float* taus_dev, int n_tau, uint8_t* gate_pass, hipStream_t st);
void launch_accept_grid(const float* logp, const int32_t* cu_draft_dev, int Bv, const float* ln_taus_dev, int n_tau,
                        int32_t* accept_len, uint8_t* all_accepted, hipStream_t st);

// measurement aid: MFMA-only loop (sink: n_workgroups*512 floats, clocks: 2 x int64)
// measurement aid: plain streaming read of `bytes` (multiple of 16) from buf
void launch_hbm_read(const void* buf, size_t bytes, uint32_t* sink, hipStream_t st);
void launch_mfma_ceiling(float* sink, long long* clocks, int n_workgroups, int iters, hipStream_t st);

// ---- accept (shared by both dtypes): first failing token per utterance
void launch_accept_scan(const float* logp, const int32_t* cu_draft_dev, int Bv, float ln_tau, int32_t* accept_len,
                        uint8_t* all_accepted, hipStream_t st);
// the prefix sums in host memory, Bv <= GATE_MAX_ARG_UTTS, as kernel arguments: an upload is a copy kernel of 2.4 us and a gap
// (four short utterances of the small fp32 decoder, verification and acceptance: 107.4 -> 101.9 us)
void launch_accept_scan_host(const float* logp, const int32_t* cu_draft, int Bv, float ln_tau, int32_t* accept_len,
                             uint8_t* all_accepted, hipStream_t st);

}  // namespace ssd
