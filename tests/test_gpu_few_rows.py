"""The 16-bit decoder on up to 128 rows, at the edges of its kernels: row blocks of 32, K ranges that do not divide over
splits and wavefronts, the rule for few column tiles, and both variants of the decode attention for every head-group ratio
with contexts around its blocks of 32 keys and 128-key passes.  Against the oracle."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import ssd_oracle as O
from paper_2603_11243_amd.binding import Context
from tests.test_gpu_verify import _compare, _run_gpu
from workloads import WORKLOADS, make_model_weights
from workloads.configs import ModelCfg
from workloads.synth import VerifyInputs

pytestmark = pytest.mark.gpu


def _inputs(m, lengths, seed):
    S, P, U = map(list, zip(*lengths))
    cu = lambda a: np.concatenate([[0], np.cumsum(a)]).astype(np.int32)
    r, g = np.random.default_rng(seed), torch.Generator().manual_seed(seed)
    return VerifyInputs((torch.randn(sum(S), m.d_model, generator=g) * 0.02).bfloat16(), cu(S), r.integers(0, m.vocab, sum(P)).astype(np.int32),
                        cu(P), r.integers(0, m.vocab, sum(U)).astype(np.int32), cu(U))


# 768 / 3200: 12 and 50 K steps (neither divides over 8 splits of two wavefronts), 100 gate/up tiles, 12 O / down tiles;
# 256 with 36 heads: 72 QKV tiles, which with more than 96 rows exceed one workgroup per CU as row tiles of 32
@pytest.mark.parametrize("shape", [(2, 768, 6, 2, 128, 3200, 512), (1, 256, 24, 6, 128, 256, 512)])
@pytest.mark.parametrize("M", [33, 64, 65, 96, 97, 128])
def test_verify_row_blocks(shape, M):
    m = ModelCfg(*shape, dtype="bf16")
    wl = replace(WORKLOADS["cfg3_1b_ragged64"], model=m)
    w = make_model_weights(m, 50 + M)
    vi = _inputs(m, [(M - 20, 3, 5), (4, 4, 4)], M)
    tau = 1.0 / m.vocab
    _compare(wl, w, vi, _run_gpu(wl, w, vi, tau), tau)


def _layer_kv(x, L, m):
    """Cache rows of one layer in 64 bits: rotated keys and values of every position of x."""
    a = O.rmsnorm(x, L["norm_attn"], m.rms_eps)
    k = (a @ L["wk"].T).reshape(len(x), m.n_kv_heads, m.head_dim)
    return O.rope(k, np.arange(len(x)), m.rope_theta).reshape(len(x), m.d_kv), a @ L["wv"].T


def _weights(m, seed):
    """Every cached row matters: attention is spread over the context (scores of unit spread) and its output is larger than
    the embedding beside it, so that a lost, repeated or misplaced row of n changes the next layer by about 1/sqrt(n);
    logits are spread widely, so that greedy tokens are seldom near ties."""
    w = make_model_weights(m, seed)
    scale = (512 / m.d_model) ** 0.5
    for L in w["layers"]:
        for k in ("wq", "wk", "wv", "wo"):
            L[k] = (L[k].float() * 2.5 * scale).to(torch.bfloat16)
    w["lm_head"] = (w["lm_head"].float() * 8).to(torch.bfloat16)
    return w


def _continue_and_check(m, w, vi, n_steps, operand, row_tol, tol, sample=None):
    """Verification with the K/V cache, acceptance, fallback.  Then, with the tokens it chose, the rows it wrote to the cache
    (those of the second layer are behind the first one's decode attention) and the tokens themselves against 64 bits."""
    ctx = Context(m, w, operand=operand)
    Bv = len(vi.cu_draft) - 1
    S, P, U = np.diff(vi.cu_speech), np.diff(vi.cu_prompt), np.diff(vi.cu_draft)
    cap = S + P + U + n_steps + 3
    kv_start = np.concatenate([[0], np.cumsum(cap)[:-1]]).astype(np.int32)
    slots = int(cap.sum())
    ctx.set_kv_cache(slots)
    ctx.reserve(max_tokens=int((S + P + U).sum()), max_verify_rows=int(U.sum()), max_utts=Bv, ar_utts=Bv, ar_steps=n_steps)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    d_ids = dev(vi.draft_ids)
    hv = ctx.verify_forward(vi.speech_emb.cuda(), vi.cu_speech, dev(vi.prompt_ids), vi.cu_prompt, d_ids, vi.cu_draft, kv_start=kv_start)
    acc = ctx.accept_prefix(hv, d_ids, vi.cu_draft, 0.9, want_greedy=True)
    acc_len, greedy = acc["accept_len"].cpu().numpy(), acc["greedy_tok"].cpu().numpy()
    assert (acc_len < U).all()                               # no random token is that likely
    first = greedy[vi.cu_draft[:-1] + acc_len].astype(np.int32)
    ctx_len = (S + P + acc_len).astype(np.int32)
    toks = ctx.ar_fallback(kv_start, ctx_len, dev(first), n_steps).cpu().numpy()
    cache = ctx._kv.view(ctx.act_dtype).float().cpu().numpy().reshape(m.n_layers, 2, slots, m.d_kv)
    assert ctx.device_flags() == 0
    ctx.close()
    w_f, w_lm = O._f64(w["norm_final"]), O._f64(w["lm_head"])
    layers = [{k: O._f64(v) for k, v in L.items()} for L in w["layers"]]
    worst, n_exact, n_tok = 0.0, 0, 0
    for b in range(Bv) if sample is None else sample:
        got = np.concatenate([[first[b]], toks[:, b]])
        ids = np.concatenate([vi.prompt_ids[vi.cu_prompt[b]:vi.cu_prompt[b + 1]],
                              vi.draft_ids[vi.cu_draft[b]:vi.cu_draft[b] + acc_len[b]], got[:-1]]).astype(np.int64)
        x = np.concatenate([O._f64(vi.speech_emb[vi.cu_speech[b]:vi.cu_speech[b + 1]]), O._f64(w["embed"][ids])])
        rows = slice(int(ctx_len[b]), int(ctx_len[b]) + n_steps)
        at = slice(int(kv_start[b]) + rows.start, int(kv_start[b]) + rows.stop)
        for l, L in enumerate(layers):
            for part, want in enumerate(_layer_kv(x, L, m)):
                err = np.linalg.norm(cache[l, part, at] - want[rows], axis=1) / np.linalg.norm(want[rows], axis=1)
                worst = max(worst, float(err.max()))
                assert err.max() <= row_tol, f"utterance {b} (context {ctx_len[b]}), layer {l}, {'kv'[part]}: rows off by {err}"
            x = O.decoder_layer(x, L, m)
        for t in range(n_steps + 1):
            logits = w_lm @ O.rmsnorm(x[int(ctx_len[b]) - 1 + t], w_f, m.rms_eps)
            n_tok += 1
            n_exact += int(np.argmax(logits)) == got[t]
            assert logits.max() - logits[got[t]] <= tol, f"utterance {b} step {t}: token {got[t]}"
    print(f"worst relative error of a cached row {worst:.2e}, {n_exact} of {n_tok} tokens identical")
    assert n_exact >= 0.9 * n_tok


# Half operands: each of the about eight roundings to 11 bits between an input row and a second-layer cache row (norm, q, k, v,
# probabilities, attention, norm, hidden units) is 2^-11 / sqrt(3) = 2.8e-4 in the root mean square, together 8e-4; five times
# that is allowed.  bfloat16 operands keep 8 bits: eight times as much.  A row of a context of 300 left out of the first layer's
# attention is 2e-2 in 64 bits (median over the rows and shapes): half operands find a wrong index, bfloat16 ones a wrong
# conversion.
# Logits have a spread of 0.16 sqrt(d) = 3.6 and inherit the relative error of the hidden row.
ROW_TOL = {"f16": 4e-3, "bf16": 3.2e-2}
LOGIT_TOL = {"f16": 5e-2, "bf16": 0.4}


# 512 columns are eight K steps: the QKV projection is K-split and finished in the attention, at most 32 rows (17) from the
# register-streaming kernel, more (34) from row blocks; 256 columns are too few steps and take the plain variant
@pytest.mark.parametrize("d_model,copies", [(512, 1), (512, 2), (256, 1)])
@pytest.mark.parametrize("heads", [(2, 2), (2, 1), (6, 2), (4, 1)])
@pytest.mark.parametrize("operand", ["f16", "bf16"])
def test_decode_attention_contexts(d_model, copies, heads, operand):
    m = ModelCfg(2, d_model, *heads, 128, 256, 512, dtype="bf16")
    # a rejected draft leaves a context of S + P rows or a little more
    vi = _inputs(m, [(c, 0, 3) for c in (1, 2, 30, 31, 32, 33, 63, 64, 65, 126, 127, 128, 129, 255, 256, 257, 300)] * copies, 7)
    _continue_and_check(m, _weights(m, 60 + heads[0]), vi, 4, operand, ROW_TOL[operand], LOGIT_TOL[operand])


@pytest.mark.parametrize("Br", [33, 64, 65, 96, 97, 128, 129])
def test_fallback_row_blocks(Br):
    m = ModelCfg(2, 768, 6, 2, 128, 3200, 512, dtype="bf16")
    vi = _inputs(m, [(1 + 5 * (b % 9), 1, 1) for b in range(Br)], Br)
    _continue_and_check(m, _weights(m, 70 + Br), vi, 2, "f16", ROW_TOL["f16"], LOGIT_TOL["f16"], sample=range(0, Br, 8))


# pieces of eight rows in the register-streaming kernel
@pytest.mark.parametrize("Br", [1, 7, 8, 9, 16, 17, 24, 25, 32])
def test_fallback_pieces_of_eight_rows(Br):
    test_fallback_row_blocks(Br)


# 768 columns are 12, 6 or 3 tiles per 128 rows: K splits of 128 x 64, 128 x 128 or 128 x 256 tiles over 12 and 50 K steps; QKV and
# gate/up pass from 64 x 64 over 64 x 128 and 128 x 128 to the 256-wide tiles
@pytest.mark.parametrize("M", [129, 256, 257, 500, 641, 1100, 1700])
def test_verify_mid_rows(M):
    m = ModelCfg(2, 768, 6, 2, 128, 3200, 512, dtype="bf16")
    wl = replace(WORKLOADS["cfg3_1b_ragged64"], model=m)
    w = make_model_weights(m, 80 + M)
    vi = _inputs(m, [(M // 2 - 40, 3, 37), (M - M // 2 - 9, 4, 5)], M)
    tau = 1.0 / m.vocab
    _compare(wl, w, vi, _run_gpu(wl, w, vi, tau), tau)


# 32 x 64 tiles with K split over the wavefronts beyond 128 rows: 24 tiles of QKV columns, one round up to 320 rows, 8 of gate/up, 1024
@pytest.mark.parametrize("M", [129, 320, 321, 1024])
def test_verify_k_groups(M):
    m = ModelCfg(2, 1024, 8, 2, 128, 256, 512, dtype="bf16")
    wl = replace(WORKLOADS["cfg3_1b_ragged64"], model=m)
    w = make_model_weights(m, 90 + M)
    vi = _inputs(m, [(M // 2 - 40, 3, 37), (M - M // 2 - 9, 4, 5)], M)
    tau = 1.0 / m.vocab
    _compare(wl, w, vi, _run_gpu(wl, w, vi, tau), tau)


# 128 x 128 tiles of 2048 columns that add to x in place, up to a full round (2048 rows) and one row beyond it: O over 32 K steps; down
# over four, as many as the ring has stages; QKV and gate/up in two rounds of them would be more, so they are 256 wide there
@pytest.mark.parametrize("M", [1281, 1409, 2048, 2049])
def test_verify_square_tiles_in_place(M):
    m = ModelCfg(2, 2048, 16, 8, 128, 256, 512, dtype="bf16")
    wl = replace(WORKLOADS["cfg3_1b_ragged64"], model=m)
    w = make_model_weights(m, 85 + M)
    n = M // 150
    vi = _inputs(m, [(130 + (M - 150 * n if b == 0 else 0), 8, 12) for b in range(n)], M)
    tau = 1.0 / m.vocab
    _compare(wl, w, vi, _run_gpu(wl, w, vi, tau), tau)


# the heights of the 256-wide tiles with an odd number of 16-row blocks per wavefront, 160 and 224: gate/up (25 tiles per row of
# tiles) of 1281..1440 and 1921..2240 rows; then 16 QKV and 8 O / down tiles: QKV of 2200 and 3300 rows, O and down of 4500 and 6500
@pytest.mark.parametrize("shape,M", [((2, 768, 6, 2, 128, 3200, 512), M) for M in (1282, 1440, 1921, 2240)]
                         + [((2, 2048, 16, 8, 128, 256, 512), M) for M in (2200, 3300, 4500, 6500)])
def test_verify_tile_heights(shape, M):
    m = ModelCfg(*shape, dtype="bf16")
    wl = replace(WORKLOADS["cfg3_1b_ragged64"], model=m)
    w = make_model_weights(m, 90 + M)
    n = M // 150
    vi = _inputs(m, [(130 + (M - 150 * n if b == 0 else 0), 8, 12) for b in range(n)], M)
    tau = 1.0 / m.vocab
    _compare(wl, w, vi, _run_gpu(wl, w, vi, tau), tau)


# the QKV epilogue at the same heights with everything it stores: rotated keys and values of every row in the K/V cache, slots in
# another order than rows, either operand type.  Two roundings to it lie before a cached row (norm, store); ROW_TOL allows for eight.
@pytest.mark.parametrize("M", [2200, 3300])
@pytest.mark.parametrize("operand", ["f16", "bf16"])
def test_cached_rows_at_tile_heights(M, operand):
    m = ModelCfg(1, 2048, 16, 8, 128, 256, 512, dtype="bf16")
    w = make_model_weights(m, 95)
    n = M // 150
    vi = _inputs(m, [(130 + (M - 150 * n if b == 0 else 0), 8, 12) for b in range(n)], M)
    rows = np.diff(vi.cu_speech) + np.diff(vi.cu_prompt) + np.diff(vi.cu_draft)
    kv_start = (int(rows.sum()) + 3 - np.cumsum(rows)).astype(np.int32)      # the last utterance first
    ctx = Context(m, w, operand=operand)
    ctx.set_kv_cache(int(rows.sum()) + 3)
    ctx._kv.zero_()
    ctx.reserve(max_tokens=M, max_verify_rows=int(vi.cu_draft[-1]), max_utts=n)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    ctx.verify_forward(vi.speech_emb.cuda(), vi.cu_speech, dev(vi.prompt_ids), vi.cu_prompt, dev(vi.draft_ids), vi.cu_draft, kv_start=kv_start)
    cache = ctx._kv.view(ctx.act_dtype).float().cpu().numpy().reshape(2, -1, m.d_kv)
    assert ctx.device_flags() == 0
    ctx.close()
    L = {k: O._f64(v) for k, v in w["layers"][0].items()}
    for b in range(n):
        ids = np.concatenate([vi.prompt_ids[vi.cu_prompt[b]:vi.cu_prompt[b + 1]], vi.draft_ids[vi.cu_draft[b]:vi.cu_draft[b + 1]]]).astype(np.int64)
        x = np.concatenate([O._f64(vi.speech_emb[vi.cu_speech[b]:vi.cu_speech[b + 1]]), O._f64(w["embed"][ids])])
        for part, want in enumerate(_layer_kv(x, L, m)):
            got = cache[part, kv_start[b]:kv_start[b] + rows[b]]
            assert (np.linalg.norm(got - want, axis=1) <= ROW_TOL[operand] * np.linalg.norm(want, axis=1)).all(), (b, "kv"[part])
    assert not cache[:, :3].any()                            # nothing beside them


# K splits of at least eight K steps on 65 to 96 rows, row blocks of the stream layout by four wavefronts: down of 512 columns in eight
# splits of eight steps each (4096), or of eight and nine (4352), which the wavefronts share unevenly
@pytest.mark.parametrize("d_ff", [4096, 4352])
@pytest.mark.parametrize("rows", [65, 70, 96])
@pytest.mark.parametrize("operand", ["f16", "bf16"])
def test_row_blocks_of_k_splits(d_ff, rows, operand):
    m = ModelCfg(2, 512, 4, 2, 128, d_ff, 512, dtype="bf16")
    vi = _inputs(m, [(1 + 5 * (b % 9), 1, 1) for b in range(rows)], rows)
    _continue_and_check(m, _weights(m, 75 + rows), vi, 2, operand, ROW_TOL[operand], LOGIT_TOL[operand], sample=range(0, rows, 8))
    if operand == "f16":
        wl = replace(WORKLOADS["cfg3_1b_ragged64"], model=m)
        w = make_model_weights(m, 76 + rows)
        vi = _inputs(m, [(rows - 20, 3, 5), (4, 4, 4)], rows)
        _compare(wl, w, vi, _run_gpu(wl, w, vi, 1.0 / m.vocab), 1.0 / m.vocab)


# the QKV projection of 2048 columns: four splits of eight K steps, finished in the decode attention
@pytest.mark.parametrize("rows", [65, 96])
@pytest.mark.parametrize("operand", ["f16", "bf16"])
def test_row_blocks_of_k_split_qkv(rows, operand):
    m = ModelCfg(2, 2048, 16, 8, 128, 256, 512, dtype="bf16")
    vi = _inputs(m, [(1 + 5 * (b % 9), 1, 1) for b in range(rows)], rows)
    _continue_and_check(m, _weights(m, 78 + rows), vi, 2, operand, ROW_TOL[operand], LOGIT_TOL[operand], sample=range(0, rows, 16))
