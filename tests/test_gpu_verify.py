"""GPU parity of verify_forward + accept_prefix (through the C ABI) against the oracle."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import ssd_oracle as O
from tests.parity import TOL_LOGP, check_accept_len
from workloads import (WORKLOADS, make_ctc_batch, make_ctc_to_llm_map, make_model_weights, make_verify_inputs)
from workloads.configs import scaled_down

pytestmark = pytest.mark.gpu


def _dev(ids):
    return torch.from_numpy(np.ascontiguousarray(ids, dtype=np.int32)).cuda()


def _gate_drafts(wl, cb):
    """Drafts and the utterances that fail the gate, decided by the oracle."""
    g = O.ctc_gate(cb.logits.float().numpy(), cb.cu_frames, wl.blank_id, wl.tau_ctc)
    table = make_ctc_to_llm_map(wl)
    fail = np.flatnonzero(~g["gate_pass"])
    return fail, [table[g["drafts"][b]] for b in fail]


def _tau_for(wl, q=1.9):
    """Synthetic threshold: ln tau = -ln V - sigma^2/2 - q sigma with sigma = 0.02 sqrt(d)."""
    s = 0.02 * np.sqrt(wl.model.d_model)
    return float(np.exp(-np.log(wl.model.vocab) - s * s / 2 - q * s))


def _run_gpu(wl, weights, vi, tau, want_greedy=True, reserve_tokens=None, operand="f16"):
    from paper_2603_11243_amd.binding import Context
    ctx = Context(wl.model, weights, operand=operand)
    M = int(vi.cu_speech[-1] + vi.cu_prompt[-1] + vi.cu_draft[-1])
    ctx.reserve(max_tokens=reserve_tokens or M, max_verify_rows=int(vi.cu_draft[-1]), max_utts=len(vi.cu_draft) - 1)
    p_ids, d_ids = _dev(vi.prompt_ids), _dev(vi.draft_ids)
    hv = ctx.verify_forward(vi.speech_emb.cuda(), vi.cu_speech, p_ids, vi.cu_prompt, d_ids, vi.cu_draft)
    out = ctx.accept_prefix(hv, d_ids, vi.cu_draft, tau, want_greedy=want_greedy)
    torch.cuda.synchronize()
    res = {k: v.cpu().numpy() for k, v in out.items()}
    res["h_verify"] = hv.float().cpu().numpy()
    ctx.close()
    return res


def _subset(vi, idx):
    """Inputs of the utterances idx only (utterances are independent)."""
    from workloads.synth import VerifyInputs
    cat = lambda parts, dt: np.concatenate(parts).astype(dt) if parts else np.zeros(0, dt)
    cu = lambda lens: np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    sp = torch.cat([vi.speech_emb[vi.cu_speech[b]:vi.cu_speech[b + 1]] for b in idx])
    return VerifyInputs(sp, cu([vi.cu_speech[b + 1] - vi.cu_speech[b] for b in idx]),
                        cat([vi.prompt_ids[vi.cu_prompt[b]:vi.cu_prompt[b + 1]] for b in idx], np.int32),
                        cu([vi.cu_prompt[b + 1] - vi.cu_prompt[b] for b in idx]),
                        cat([vi.draft_ids[vi.cu_draft[b]:vi.cu_draft[b + 1]] for b in idx], np.int32),
                        cu([vi.cu_draft[b + 1] - vi.cu_draft[b] for b in idx]))


def _compare(wl, weights, vi, res, tau, sample=None, tol=None, stats=None):
    """stats (dict, optional) receives the largest relative L2 error of a final-normed hidden row."""
    tol = TOL_LOGP[wl.model.dtype] if tol is None else tol
    idx = list(range(len(vi.cu_draft) - 1)) if sample is None else list(sample)
    sub = _subset(vi, idx)
    lp, hid, greedy = O.draft_logp(weights, wl.model, sub.speech_emb, sub.cu_speech, sub.prompt_ids, sub.cu_prompt,
                                   sub.draft_ids, sub.cu_draft, return_hidden=True, return_greedy=True)
    worst = 0.0
    w_lm = None
    for k, b in enumerate(idx):
        lo, hi = vi.cu_draft[b], vi.cu_draft[b + 1]
        got = res["draft_logp"][lo:hi]
        assert np.isfinite(got).all()
        err = np.abs(got - lp[k]).max() if hi > lo else 0.0
        worst = max(worst, err)
        assert err <= tol, f"utt {b}: |logp - oracle| = {err:.3e} > {tol}"
        check_accept_len(res["accept_len"][b], res["all_accepted"][b], lp[k], tau, tol)
        if stats is not None and hi > lo:
            dh = np.linalg.norm(res["h_verify"][lo:hi] - hid[k], axis=1) / np.linalg.norm(hid[k], axis=1)
            stats["hidden_rel_err"] = max(stats.get("hidden_rel_err", 0.0), float(dh.max()))
        if "greedy_tok" in res and hi > lo:
            mism = np.flatnonzero(res["greedy_tok"][lo:hi] != greedy[k])
            if len(mism):                      # only legal when the oracle's top two logits are within tolerance
                if w_lm is None:
                    w_lm = weights["lm_head"].double().cpu().numpy()
                for i in mism:
                    logits = w_lm @ hid[k][i]
                    assert logits.max() - logits[res["greedy_tok"][lo + i]] <= tol
    return worst


# ------------------------------------------------------------------ tiny fp32 configuration (full)

def test_cfg1_tiny_f32_full_chain():
    wl = WORKLOADS["cfg1_tiny_f32"]
    cb = make_ctc_batch(wl)
    fail, drafts = _gate_drafts(wl, cb)
    assert len(fail) == wl.B
    vi = make_verify_inputs(wl, cb.seconds[fail], drafts)
    w = make_model_weights(wl.model, wl.seed)
    tau = _tau_for(wl)
    res = _run_gpu(wl, w, vi, tau)
    worst = _compare(wl, w, vi, res, tau)
    print(f"cfg1 worst |dlogp| = {worst:.3e}")
    # the threshold sits inside the spread of this model's likelihoods: prefixes of different length occur
    assert 0 < res["accept_len"].sum() < vi.cu_draft[-1]


def test_tiny_f32_sharper_model_and_edge_shapes():
    """Larger weights (peaked attention and output distributions), empty drafts, a single speech row."""
    wl = replace(WORKLOADS["cfg1_tiny_f32"], model=replace(WORKLOADS["cfg1_tiny_f32"].model, n_layers=3))
    w = make_model_weights(wl.model, 77)
    g = torch.Generator().manual_seed(5)
    for L in w["layers"]:
        for k in ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down"):
            L[k] = torch.randn(L[k].shape, generator=g) * 0.08
    w["lm_head"] = torch.randn(w["lm_head"].shape, generator=g) * 0.15
    rng = np.random.default_rng(3)
    S, P, U = [1, 30, 7, 64], [0, 10, 3, 5], [5, 0, 40, 70]
    from workloads.synth import VerifyInputs
    cu = lambda a: np.concatenate([[0], np.cumsum(a)]).astype(np.int32)
    vi = VerifyInputs(torch.randn(sum(S), 256, generator=g) * 0.5, cu(S),
                      rng.integers(0, 4096, sum(P)).astype(np.int32), cu(P),
                      rng.integers(0, 4096, sum(U)).astype(np.int32), cu(U))
    tau = 2e-4
    res = _run_gpu(wl, w, vi, tau)
    _compare(wl, w, vi, res, tau)
    assert res["accept_len"][1] == 0 and res["all_accepted"][1] == 1          # empty draft: vacuous accept


def test_out_of_range_token_ids_are_clamped_and_flagged():
    """Ids outside [0, vocab) cannot be seen by the host: the device clamps them and raises a sticky flag."""
    from paper_2603_11243_amd.binding import Context
    from workloads.synth import VerifyInputs
    wl = WORKLOADS["cfg1_tiny_f32"]
    w = make_model_weights(wl.model, 5)
    V = wl.model.vocab
    cu = lambda a: np.concatenate([[0], np.cumsum(a)]).astype(np.int32)
    g = torch.Generator().manual_seed(2)
    sp = torch.randn(12, wl.model.d_model, generator=g) * 0.02
    bad_p, bad_d = np.array([3, -7, V + 5], np.int32), np.array([10, V, 20, -1], np.int32)
    ok_p, ok_d = np.clip(bad_p, 0, V - 1), np.clip(bad_d, 0, V - 1)
    ctx = Context(wl.model, w)
    try:
        ctx.reserve(max_tokens=32, max_verify_rows=8, max_utts=1)
        run = lambda p, d: ctx.accept_prefix(ctx.verify_forward(sp.cuda(), cu([12]), _dev(p), cu([3]), _dev(d), cu([4])),
                                             _dev(d), cu([4]), 1e-5)["draft_logp"].cpu().numpy()
        good = run(ok_p, ok_d)
        assert ctx.device_flags() == 0
        clamped = run(bad_p, bad_d)
        assert ctx.device_flags() == 1 and ctx.device_flags() == 0          # reported once, then cleared
        assert np.array_equal(good, clamped)
    finally:
        ctx.close()


def test_tiny_f32_causality_and_batch_isolation():
    wl = WORKLOADS["cfg1_tiny_f32"]
    cb = make_ctc_batch(wl)
    fail, drafts = _gate_drafts(wl, cb)
    vi = make_verify_inputs(wl, cb.seconds[fail], drafts)
    w = make_model_weights(wl.model, wl.seed)
    base = _run_gpu(wl, w, vi, 0.1, want_greedy=False)
    # utterance 2 alone gives bit-identical scores (no cross-utterance leakage)
    alone = _run_gpu(wl, w, _subset(vi, [2]), 0.1, want_greedy=False)
    lo, hi = vi.cu_draft[2], vi.cu_draft[3]
    assert np.array_equal(alone["draft_logp"], base["draft_logp"][lo:hi])
    # changing a later draft token leaves earlier scores bit-identical (causal mask)
    vi2 = _subset(vi, [0, 1, 2, 3])
    k = 7
    vi2.draft_ids[lo + k] = (vi2.draft_ids[lo + k] + 1) % wl.model.vocab
    mod = _run_gpu(wl, w, vi2, 0.1, want_greedy=False)
    assert np.array_equal(mod["draft_logp"][lo:lo + k], base["draft_logp"][lo:lo + k])
    assert mod["draft_logp"][lo + k] != base["draft_logp"][lo + k]
    assert np.array_equal(mod["draft_logp"][:lo], base["draft_logp"][:lo])


# draft lengths and poisoned draft positions: the poisoned row is the first, second, ninth and last of a 16-row attention
# tile, in the first tile and in later ones
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
@pytest.mark.parametrize("head_dim", [64, 128])
def test_tiny_f32_non_finite_rows_do_not_reach_earlier_positions(value, head_dim):
    from workloads.synth import VerifyInputs
    wl = WORKLOADS["cfg1_tiny_f32"]
    wl = replace(wl, model=replace(wl.model, head_dim=head_dim))
    S, P, U, at = [1, 9, 20, 30, 40, 5], [4] * 6, [20, 30, 40, 24, 30, 8], [0, 3, 9, 13, 27, None]
    rows = [(s + p + a) % 16 for s, p, a in zip(S, P, at) if a is not None]
    assert rows == [5, 0, 1, 15, 7]
    cu = lambda a: np.concatenate([[0], np.cumsum(a)]).astype(np.int32)
    r, poison = np.random.default_rng(3), 5
    ids = lambda n: r.integers(poison + 1, wl.model.vocab, n).astype(np.int32)
    vi = VerifyInputs(torch.randn(sum(S), wl.model.d_model, generator=torch.Generator().manual_seed(3)) * 0.02, cu(S), ids(sum(P)),
                      cu(P), ids(sum(U)), cu(U))
    w = make_model_weights(wl.model, wl.seed)
    w["embed"][poison] = value
    base = _run_gpu(wl, w, vi, 1e-30)
    assert np.isfinite(base["draft_logp"]).all()
    for b, a in enumerate(at):
        if a is not None:
            vi.draft_ids[vi.cu_draft[b] + a] = poison
    mod = _run_gpu(wl, w, vi, 1e-30)
    for b, a in enumerate(at):
        lo, hi = vi.cu_draft[b], vi.cu_draft[b + 1]
        end = hi if a is None else lo + a
        assert np.array_equal(mod["draft_logp"][lo:end], base["draft_logp"][lo:end]), f"utterance {b}"
        assert np.array_equal(mod["greedy_tok"][lo:end], base["greedy_tok"][lo:end])
        if a is None:
            assert mod["accept_len"][b] == U[b]
            continue
        assert np.isfinite(mod["draft_logp"][end])               # the poisoned token is scored by the row before it
        assert not np.isfinite(mod["draft_logp"][end + 1:hi]).any()
        assert mod["accept_len"][b] == a + 1


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_tiny_f32_head_and_hidden_rows_at_any_float(shift):
    """accept_prefix reads the caller's hidden rows and head in place: neither has to start at a multiple of 16 bytes."""
    from paper_2603_11243_amd.binding import Context
    wl = WORKLOADS["cfg1_tiny_f32"]
    d, n = wl.model.d_model, 37
    w = make_model_weights(wl.model, wl.seed)
    h = torch.randn(n, d, generator=torch.Generator().manual_seed(1))
    ids = _dev(np.arange(n))

    def shifted(t, by):
        buf = torch.empty(t.numel() + by, device="cuda")
        return buf[by:].view(t.shape).copy_(t)

    def accept(by):
        ctx = Context(wl.model, dict(w, lm_head=shifted(w["lm_head"], by)))
        assert ctx._keep[1].data_ptr() % 16 == 4 * by
        ctx.reserve(max_tokens=n, max_verify_rows=n, max_utts=1)
        res = ctx.accept_prefix(shifted(h, by), ids, [0, n], 0.1)
        res = {k: v.cpu() for k, v in res.items()}
        ctx.close()
        return res

    want, got = accept(0), accept(shift)
    assert torch.isfinite(want["draft_logp"]).all()
    for k in want:
        assert torch.equal(want[k], got[k])


def test_tiny_f32_does_not_raise_the_operand_overflow_flag():
    """fp32 models have no matrix-core operand type to leave: a likelihood that is not finite is returned as it is."""
    from paper_2603_11243_amd.binding import Context
    wl = WORKLOADS["cfg1_tiny_f32"]
    w = make_model_weights(wl.model, wl.seed)
    ctx = Context(wl.model, w)
    try:
        ctx.reserve(max_tokens=8, max_verify_rows=4, max_utts=1, ar_utts=1, ar_steps=1)
        ctx.set_kv_cache(16)
        speech = torch.zeros(3, wl.model.d_model)
        speech[1] = float("nan")
        d_ids = _dev([5, 6])
        hv = ctx.verify_forward(speech.cuda(), [0, 3], _dev([1]), [0, 1], d_ids, [0, 2], kv_start=[0])
        acc = ctx.accept_prefix(hv, d_ids, [0, 2], 0.1)
        ctx.ar_fallback([0], [4], _dev([7]), 1)
        assert not torch.isfinite(acc["draft_logp"]).any()
        assert ctx.device_flags() == 0
    finally:
        ctx.close()


# ------------------------------------------------------------------ bf16, reduced depth, whole batch

@pytest.mark.parametrize("name,layers,B", [("cfg3_1b_ragged64", 2, 12), ("cfg5_3b_ragged128", 1, 10),
                                           ("cfg4_1b_long_ml", 1, 2),
                                           ("cfg2_1b_b1", 3, 1),          # <= 128 rows: skinny tiles, split-K partials
                                           ("cfg3_1b_ragged64", 1, 2)])   # 33..128 verification rows
def test_bf16_reduced_depth_whole_batch(name, layers, B):
    wl = scaled_down(WORKLOADS[name], n_layers=layers, B=B)
    wl = replace(wl, gate_rate=0.0)
    cb = make_ctc_batch(wl)
    fail, drafts = _gate_drafts(wl, cb)
    vi = make_verify_inputs(wl, cb.seconds[fail], drafts, device="cuda")
    w = make_model_weights(wl.model, wl.seed, device="cuda")
    tau = _tau_for(wl)
    res = _run_gpu(wl, w, vi, tau)
    worst = _compare(wl, w, vi, res, tau)
    print(f"{wl.name}: worst |dlogp| = {worst:.3e} over {vi.cu_draft[-1]} tokens")


@pytest.mark.parametrize("M", [9, 31, 32, 33, 128, 129, 191, 257, 513, 770])
def test_bf16_row_counts_around_tile_and_split_thresholds(M):
    """One 1B-width layer; utterance lengths chosen so that the total row count M sits on and next to
    the boundaries the GEMM dispatch uses (register-streaming kernel up to 32 rows, skinny path up to 128
    rows, tile heights 128/192/256)."""
    from workloads.synth import VerifyInputs
    wl = scaled_down(WORKLOADS["cfg3_1b_ragged64"], n_layers=1, B=3)
    w = make_model_weights(wl.model, 4242, device="cuda")
    rng = np.random.default_rng(M)
    n = [M // 3, M // 3, M - 2 * (M // 3)]
    U = [max(1, k // 3) for k in n]
    P = [min(4, k - u - 1) for k, u in zip(n, U)]
    S = [k - u - p for k, u, p in zip(n, U, P)]
    cu = lambda a: np.concatenate([[0], np.cumsum(a)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(M)
    sp = (torch.randn(sum(S), wl.model.d_model, generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    vi = VerifyInputs(sp, cu(S), rng.integers(0, wl.model.vocab, sum(P)).astype(np.int32), cu(P),
                      rng.integers(0, wl.model.vocab, sum(U)).astype(np.int32), cu(U))
    tau = _tau_for(wl)
    # a workspace reserved for a somewhat larger batch must also serve the few-row path (split-K scratch)
    res = _run_gpu(wl, w, vi, tau, reserve_tokens=M + 40 if M in (33, 128) else None)
    worst = _compare(wl, w, vi, res, tau)
    assert worst < 5e-3           # one layer: far inside the 2e-2 budget, a dropped tile would be O(1)


@pytest.mark.parametrize("Mv", [129, 192, 193, 256, 257, 385])
def test_accept_prefix_alone_row_counts_around_lm_head_tiles(Mv):
    """accept_prefix on given hidden rows (no decoder forward): verification-row counts on and next to the
    boundaries of the LM head's 256-row tile and of the 64-row halves in which a wavefront reduces its slab;
    likelihoods, greedy tokens (lowest index on ties) and prefix lengths against the oracle's Eq. 5."""
    from paper_2603_11243_amd.binding import Context
    wl = scaled_down(WORKLOADS["cfg3_1b_ragged64"], n_layers=1, B=3)
    w = make_model_weights(wl.model, 777, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(Mv)
    # unit-RMS rows, as after the final norm; the library hands hidden rows over as IEEE half
    h = torch.randn(Mv, wl.model.d_model, generator=g, device="cuda").to(torch.float16)
    rng = np.random.default_rng(Mv)
    U = [Mv // 3, 0, Mv - Mv // 3]                      # an utterance without a draft in the middle
    cu_d = np.concatenate([[0], np.cumsum(U)]).astype(np.int32)
    y = rng.integers(0, wl.model.vocab, Mv).astype(np.int32)
    y[0], y[-1] = 0, wl.model.vocab - 1                 # first and last column of the vocabulary
    tau = _tau_for(wl)
    ctx = Context(wl.model, w)
    ctx.reserve(max_tokens=Mv + 8, max_verify_rows=Mv, max_utts=3)
    out = ctx.accept_prefix(h, _dev(y), cu_d, tau, want_greedy=True)
    torch.cuda.synchronize()
    res = {k: v.cpu().numpy() for k, v in out.items()}
    ctx.close()
    tol = TOL_LOGP[wl.model.dtype]
    w_lm = w["lm_head"].double().cpu().numpy()
    h64 = h.double().cpu().numpy()
    lp = np.zeros(Mv)
    for i in range(Mv):
        lp[i], gt = O.lm_head_logp(h64[i], w_lm, int(y[i]))
        assert abs(res["draft_logp"][i] - lp[i]) <= tol, f"row {i}: {res['draft_logp'][i]} vs {lp[i]}"
        if res["greedy_tok"][i] != gt:                  # only legal when the two logits are within tolerance
            logits = w_lm @ h64[i]
            assert logits.max() - logits[res["greedy_tok"][i]] <= tol
    assert np.abs(res["draft_logp"] - lp).max() < 5e-3   # one matrix product: far inside the budget
    for b in range(3):
        check_accept_len(res["accept_len"][b], res["all_accepted"][b], lp[cu_d[b]:cu_d[b + 1]], tau, tol)


@pytest.mark.parametrize("name", ["cfg3_1b_ragged64", "cfg5_3b_ragged128"])
def test_bf16_utterance_lengths_around_key_blocks(name):
    """One layer of the 1B-width (2 query heads per KV head) and of the 3B-width decoder (3 per KV head); utterance
    lengths on and next to the attention kernel's 64-key blocks and 32-row wavefronts, nearly every position a
    verification row: a block that ends exactly at the utterance's end is loaded whole, any other last block row by
    row with clamping, and the last utterance of the batch ends where the buffer ends."""
    from workloads.synth import VerifyInputs
    wl = scaled_down(WORKLOADS[name], n_layers=1, B=9)
    w = make_model_weights(wl.model, 77, device="cuda")
    rng = np.random.default_rng(5)
    n = [64, 1 + 2, 63, 65, 128, 127, 129, 33, 192]
    S, P = [1] * 9, [1] * 9
    U = [k - 2 for k in n]
    cu = lambda a: np.concatenate([[0], np.cumsum(a)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(5)
    sp = (torch.randn(sum(S), wl.model.d_model, generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    vi = VerifyInputs(sp, cu(S), rng.integers(0, wl.model.vocab, sum(P)).astype(np.int32), cu(P),
                      rng.integers(0, wl.model.vocab, sum(U)).astype(np.int32), cu(U))
    tau = _tau_for(wl)
    res = _run_gpu(wl, w, vi, tau)
    worst = _compare(wl, w, vi, res, tau)
    assert worst < 5e-3           # one layer: far inside the 2e-2 budget, a wrong key block would be O(1)


@pytest.mark.parametrize("seed", [11, 12, 13, 14, 15, 16])
def test_bf16_random_ragged_batches(seed):
    """Seeded random ragged batches through one decoder layer (1B width for even seeds, 3B width for odd ones): 1 to 12
    utterances with 1 to 300 speech rows, 0 to 20 prompt tokens and 0 to 120 draft tokens each, so that total row
    counts, utterance lengths, key-block counts and verification-row counts fall on no particular boundary."""
    from workloads.synth import VerifyInputs
    rng = np.random.default_rng(seed)
    B = int(rng.integers(1, 13))
    wl = scaled_down(WORKLOADS["cfg5_3b_ragged128" if seed % 2 else "cfg3_1b_ragged64"], n_layers=1, B=B)
    w = make_model_weights(wl.model, 1000 + seed, device="cuda")
    S = rng.integers(1, 301, B).tolist()
    P = rng.integers(0, 21, B).tolist()
    U = rng.integers(0, 121, B).tolist()
    if sum(U) == 0:
        U[0] = 5
    cu = lambda a: np.concatenate([[0], np.cumsum(a)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(seed)
    sp = (torch.randn(sum(S), wl.model.d_model, generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    vi = VerifyInputs(sp, cu(S), rng.integers(0, wl.model.vocab, sum(P)).astype(np.int32), cu(P),
                      rng.integers(0, wl.model.vocab, sum(U)).astype(np.int32), cu(U))
    tau = _tau_for(wl)
    res = _run_gpu(wl, w, vi, tau)
    worst = _compare(wl, w, vi, res, tau)
    assert worst < 5e-3           # one layer: far inside the 2e-2 budget


def test_bf16_empty_drafts_and_single_row_utterances():
    """bf16 path, two 1B-width layers: utterances without a draft inside a batch (vacuous acceptance), an
    utterance made of one speech row, and a batch in which nobody has a draft (nothing to score)."""
    from workloads.synth import VerifyInputs
    from paper_2603_11243_amd.binding import Context
    wl = scaled_down(WORKLOADS["cfg3_1b_ragged64"], n_layers=2, B=5)
    w = make_model_weights(wl.model, 99, device="cuda")
    rng = np.random.default_rng(8)
    cu = lambda a: np.concatenate([[0], np.cumsum(a)]).astype(np.int32)
    g = torch.Generator(device="cuda").manual_seed(8)
    S, P, U = [1, 40, 70, 3, 90], [0, 6, 0, 2, 12], [3, 0, 65, 0, 130]
    sp = (torch.randn(sum(S), wl.model.d_model, generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    vi = VerifyInputs(sp, cu(S), rng.integers(0, wl.model.vocab, sum(P)).astype(np.int32), cu(P),
                      rng.integers(0, wl.model.vocab, sum(U)).astype(np.int32), cu(U))
    tau = _tau_for(wl)
    res = _run_gpu(wl, w, vi, tau)
    _compare(wl, w, vi, res, tau)
    for b in (1, 3):
        assert res["accept_len"][b] == 0 and res["all_accepted"][b] == 1
    # nobody has a draft: the forward runs (K/V would be complete), nothing is scored
    ctx = Context(wl.model, w)
    try:
        ctx.reserve(max_tokens=sum(S) + sum(P), max_verify_rows=0, max_utts=5)
        p_ids = _dev(vi.prompt_ids)
        d_ids = torch.zeros(0, dtype=torch.int32, device="cuda")
        zero = np.zeros(6, np.int32)
        hv = ctx.verify_forward(sp, vi.cu_speech, p_ids, vi.cu_prompt, d_ids, zero)
        out = ctx.accept_prefix(hv, d_ids, zero, tau)
        torch.cuda.synchronize()
        assert hv.shape[0] == 0
        assert out["accept_len"].cpu().tolist() == [0] * 5 and out["all_accepted"].cpu().tolist() == [1] * 5
    finally:
        ctx.close()


# ------------------------------------------------------------------ bf16, full depth, sampled utterances

@pytest.mark.parametrize("name,n_random", [("cfg2_1b_b1", None), ("cfg3_1b_ragged64", None), ("cfg4_1b_long_ml", None),
                                           ("cfg5_3b_ragged128", 4)])
def test_bf16_full_size_against_oracle(name, n_random):
    """The whole batch runs on the GPU in the benchmark's launch configuration.  The oracle scores every verified
    utterance of the three 1B-class configurations; of the 3B-class one (90 utterances, 32 layers) it scores the
    longest, the shortest, n_random seeded random ones and the two whose GPU likelihoods come closest to the
    threshold (utterances are independent, so their results do not depend on the rest of the batch)."""
    wl = WORKLOADS[name]
    cb = make_ctc_batch(wl)
    fail, drafts = _gate_drafts(wl, cb)
    vi = make_verify_inputs(wl, cb.seconds[fail], drafts, device="cuda")
    w = make_model_weights(wl.model, wl.seed, device="cuda")
    tau = _tau_for(wl)
    res = _run_gpu(wl, w, vi, tau)
    assert np.isfinite(res["draft_logp"]).all()
    lens = np.diff(vi.cu_speech) + np.diff(vi.cu_prompt) + np.diff(vi.cu_draft)
    Bv = len(lens)
    if n_random is None:
        sample = list(range(Bv))
    else:
        rng = np.random.default_rng(wl.seed)
        order = np.argsort(lens, kind="stable")
        margin = np.array([np.abs(res["draft_logp"][vi.cu_draft[b]:vi.cu_draft[b + 1]] - np.log(tau)).min()
                           if vi.cu_draft[b + 1] > vi.cu_draft[b] else np.inf for b in range(Bv)])
        sample = sorted(set([int(order[-1]), int(order[0])] + [int(x) for x in np.argsort(margin)[:2]]
                            + [int(x) for x in rng.choice(Bv, size=n_random, replace=False)]))
        assert int(order[-1]) in sample and lens[order[-1]] == lens.max()
    worst = _compare(wl, w, vi, res, tau, sample=sample)
    print(f"{name}: worst |dlogp| = {worst:.3e} on {len(sample)} of {Bv} utterances "
          f"({int(sum(lens[b] for b in sample))} of {int(lens.sum())} rows, longest {int(lens.max())})")
    # properties that hold at any size: accepted prefix is consistent with the GPU's own scores
    ln_tau = np.float32(np.log(np.float64(np.float32(tau))))
    for b in range(len(vi.cu_draft) - 1):
        lp = res["draft_logp"][vi.cu_draft[b]:vi.cu_draft[b + 1]]
        bad = np.flatnonzero(~(lp > ln_tau))
        want = int(bad[0]) if len(bad) else len(lp)
        assert res["accept_len"][b] == want and res["all_accepted"][b] == (want == len(lp))
        assert (lp <= 0).all()


# ------------------------------------------------------------------ bf16, hard inputs for the half-precision operands

def _sharp_weights(m, seed):
    """Projection matrices 4x, LM head 8x the usual scale: attention scores with a spread of about 13
    (peaked attention), logits with a spread of about 7 (peaked output distribution), residual rows in the tens to
    hundreds after a few layers."""
    w = make_model_weights(m, seed, device="cuda")
    for L in w["layers"]:
        for k in ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down"):
            L[k] = (L[k].float() * 4).to(torch.bfloat16)
    w["lm_head"] = (w["lm_head"].float() * 8).to(torch.bfloat16)
    return w


@pytest.mark.parametrize("layers", [1, 3])
def test_bf16_sharper_model(layers):
    from workloads.synth import VerifyInputs
    wl = replace(scaled_down(WORKLOADS["cfg3_1b_ragged64"], n_layers=layers, B=6), gate_rate=0.0)
    w = _sharp_weights(wl.model, 31 + layers)
    cb = make_ctc_batch(wl)
    fail, drafts = _gate_drafts(wl, cb)
    vi = make_verify_inputs(wl, cb.seconds[fail], drafts, device="cuda")
    vi = VerifyInputs((vi.speech_emb.float() * 25).to(torch.bfloat16), vi.cu_speech, vi.prompt_ids, vi.cu_prompt,
                      vi.draft_ids, vi.cu_draft)
    tau = float(np.exp(-np.log(wl.model.vocab) - 30.0))        # inside the (wide) spread of these likelihoods
    from paper_2603_11243_amd.binding import Context
    ctx = Context(wl.model, w)
    assert ctx.inexact_weights() == 0
    ctx.close()
    res = _run_gpu(wl, w, vi, tau)
    # What the 16-bit operands cost here: attention scores of magnitude up to ~40 formed from q and k rounded to 11
    # significant bits carry an absolute error of about 5e-3, i.e. 0.5 % on a softmax weight, and a hidden row ends
    # up 4e-3 (one layer) to 1e-2 (three layers) off in relative terms.  That error reaches log p multiplied by the
    # spread of the logits, which the 8x LM head makes 8 times that of the five configurations (0.16 sqrt(d) = 7.2
    # against 0.9).  So the likelihood tolerance is 10 x the 2e-2 of those configurations, and the hidden rows
    # themselves are held to a relative error of 2e-2; a dropped tile or a wrong scale would be O(1) in both.
    stats = {}
    worst = _compare(wl, w, vi, res, tau, tol=10 * TOL_LOGP["bf16"], stats=stats)
    spread = float(np.std(res["draft_logp"]))
    print(f"sharp model, {layers} layer(s): worst |dlogp| = {worst:.3e}, spread of log p = {spread:.2f}, "
          f"worst relative error of a hidden row = {stats['hidden_rel_err']:.2e}")
    assert spread > 3.0                      # the output distribution really is peaked
    assert stats["hidden_rel_err"] < 2e-2


def test_bf16_activation_overflow_is_saturated_and_flagged():
    """Gate and up projections scaled until SiLU(gate) * up leaves the half range: the store saturates, the
    sticky flag is raised once, every output stays finite; the unscaled model raises nothing."""
    from paper_2603_11243_amd.binding import Context
    wl = replace(scaled_down(WORKLOADS["cfg3_1b_ragged64"], n_layers=1, B=3), gate_rate=0.0)
    cb = make_ctc_batch(wl)
    fail, drafts = _gate_drafts(wl, cb)
    vi = make_verify_inputs(wl, cb.seconds[fail], drafts, device="cuda")
    p_ids, d_ids = _dev(vi.prompt_ids), _dev(vi.draft_ids)
    M = int(vi.cu_speech[-1] + vi.cu_prompt[-1] + vi.cu_draft[-1])
    for scale, want in ((1.0, 0), (512.0, 2)):
        w = make_model_weights(wl.model, 17, device="cuda")
        for k in ("w_gate", "w_up"):
            w["layers"][0][k] = (w["layers"][0][k].float() * scale).to(torch.bfloat16)
        ctx = Context(wl.model, w)
        try:
            ctx.reserve(max_tokens=M, max_verify_rows=int(vi.cu_draft[-1]), max_utts=len(vi.cu_draft) - 1)
            hv = ctx.verify_forward(vi.speech_emb, vi.cu_speech, p_ids, vi.cu_prompt, d_ids, vi.cu_draft)
            out = ctx.accept_prefix(hv, d_ids, vi.cu_draft, 1e-6)
            flags = ctx.device_flags()
            assert flags == want, f"scale {scale}: flags {flags}"
            assert ctx.device_flags() == 0                       # reported once, then cleared
            assert torch.isfinite(hv.float()).all() and torch.isfinite(out["draft_logp"]).all()
        finally:
            ctx.close()


def test_bf16_causality_and_batch_isolation():
    """bf16 path, two 1B-width layers.  Changing a later draft token leaves every earlier score bit-identical (same
    launch shapes, causal mask); an utterance scored alone agrees with its scores inside the batch (not bitwise: the
    last layer of a small batch takes the few-row kernels, which sum K in a different order)."""
    wl = replace(scaled_down(WORKLOADS["cfg3_1b_ragged64"], n_layers=2, B=6), gate_rate=0.0)
    cb = make_ctc_batch(wl)
    fail, drafts = _gate_drafts(wl, cb)
    vi = make_verify_inputs(wl, cb.seconds[fail], drafts, device="cuda")
    w = make_model_weights(wl.model, 23, device="cuda")
    tau = _tau_for(wl)
    base = _run_gpu(wl, w, vi, tau, want_greedy=False)
    b = int(np.argmax(np.diff(vi.cu_draft)))
    lo, hi = vi.cu_draft[b], vi.cu_draft[b + 1]
    k = (hi - lo) // 2
    vi2 = _subset(vi, list(range(len(vi.cu_draft) - 1)))
    vi2.draft_ids[lo + k] = (vi2.draft_ids[lo + k] + 1) % wl.model.vocab
    mod = _run_gpu(wl, w, vi2, tau, want_greedy=False)
    assert np.array_equal(mod["draft_logp"][:lo + k], base["draft_logp"][:lo + k])
    assert np.array_equal(mod["draft_logp"][hi:], base["draft_logp"][hi:])
    assert mod["draft_logp"][lo + k] != base["draft_logp"][lo + k]
    alone = _run_gpu(wl, w, _subset(vi, [b]), tau, want_greedy=False)
    assert np.abs(alone["draft_logp"] - base["draft_logp"][lo:hi]).max() < 2e-3


def test_sizes_beyond_32_bit_offsets_and_odd_head_dim_are_refused():
    """Host-side refusals that need a context with a model: an activation matrix of 4 GiB or more (the GEMM
    loaders use 32-bit byte offsets), and the AR fallback with a head_dim that is not a multiple of 8."""
    from paper_2603_11243_amd.binding import Context, SsdError
    wl = WORKLOADS["cfg1_tiny_f32"]
    ctx = Context(wl.model, make_model_weights(wl.model, 5))
    try:
        ctx.reserve(max_tokens=64, max_verify_rows=8, max_utts=2)
        n = 1100                                  # 1100 utterances x 1000 rows x d_ff 1024 x 4 bytes >= 4 GiB
        cu_s = (np.arange(n + 1) * 1000).astype(np.int32)
        zero = np.zeros(n + 1, np.int32)
        fake = torch.zeros(16, device="cuda")
        with pytest.raises(SsdError, match="4 GiB") as ei:
            ctx._check(ctx._lib.verify_forward(ctx._h, fake.data_ptr(), cu_s.ctypes.data, None, zero.ctypes.data, None,
                                               zero.ctypes.data, n, None))
        assert ei.value.code == -2
    finally:
        ctx.close()
    m = replace(wl.model, head_dim=12)            # 4 heads x 12: legal for verify_forward, not for the decode attention
    ctx = Context(m, make_model_weights(m, 6))
    try:
        ctx.set_kv_cache(64)
        ctx.reserve(max_tokens=64, max_verify_rows=8, max_utts=2, ar_utts=1, ar_steps=2)
        with pytest.raises(SsdError, match="multiple of 8"):
            ctx.ar_fallback([0], [5], _dev([1]), 2)
    finally:
        ctx.close()


# ------------------------------------------------------------------ the two matrix-core operand types

@pytest.mark.parametrize("name,layers,B", [("cfg2_1b_b1", 24, 1), ("cfg3_1b_ragged64", 4, 12)])
def test_operand_types_against_oracle(name, layers, B):
    """The same batch through both operand types of the 16-bit path: IEEE half (the default) and bfloat16 (what
    the paper's stack runs in).  Both are compared with the oracle; half has to meet the stated 2e-2, bfloat16
    (8 significant bits at every contraction input) is bounded by 10 times that and is expected to be worse."""
    wl = replace(scaled_down(WORKLOADS[name], n_layers=layers, B=B), gate_rate=0.0)
    cb = make_ctc_batch(wl)
    fail, drafts = _gate_drafts(wl, cb)
    vi = make_verify_inputs(wl, cb.seconds[fail], drafts, device="cuda")
    w = make_model_weights(wl.model, wl.seed, device="cuda")
    tau = _tau_for(wl)
    worst, hidden = {}, {}
    for operand, tol in (("f16", TOL_LOGP["bf16"]), ("bf16", 10 * TOL_LOGP["bf16"])):
        res = _run_gpu(wl, w, vi, tau, operand=operand)
        stats = {}
        worst[operand] = _compare(wl, w, vi, res, tau, tol=tol, stats=stats)
        hidden[operand] = stats["hidden_rel_err"]
    print(f"{wl.name}: worst |dlogp| half {worst['f16']:.3e}, bfloat16 {worst['bf16']:.3e}; worst relative error of a "
          f"hidden row half {hidden['f16']:.2e}, bfloat16 {hidden['bf16']:.2e}")
    assert hidden["bf16"] > 2 * hidden["f16"]          # three mantissa bits fewer at every contraction input


@pytest.mark.parametrize("Bv", [1, 255, 256, 257])
def test_accept_prefix_with_prefix_sums_as_arguments(Bv):
    """Up to 256 utterances the prefix sums are kernel arguments, beyond they are uploaded: the decision follows from the stored
    likelihoods exactly, with empty drafts and the lowest and highest utterance among them."""
    from paper_2603_11243_amd.binding import Context
    wl = WORKLOADS["cfg1_tiny_f32"]
    ctx = Context(wl.model, make_model_weights(wl.model, 5))
    U = np.arange(Bv) * 5 % 4 + (Bv == 1)
    cu = np.concatenate([[0], np.cumsum(U)]).astype(np.int32)
    n = int(cu[-1])
    g = torch.Generator(device="cuda").manual_seed(Bv)
    h = torch.randn(n, wl.model.d_model, generator=g, device="cuda")
    ids = torch.randint(0, wl.model.vocab, (n,), generator=g, device="cuda", dtype=torch.int32)
    ctx.reserve(max_tokens=n, max_verify_rows=n, max_utts=Bv)
    tau = float(torch.exp(ctx.accept_prefix(h, ids, cu, 0.5)["draft_logp"]).median())
    out = {k: v.cpu().numpy() for k, v in ctx.accept_prefix(h, ids, cu, tau).items()}
    ctx.close()
    ok = out["draft_logp"] > np.float32(np.log(np.float64(np.float32(tau))))
    for b in range(Bv):
        bad = np.flatnonzero(~ok[cu[b]:cu[b + 1]])
        want = bad[0] if len(bad) else U[b]
        assert out["accept_len"][b] == want and out["all_accepted"][b] == (want == U[b])
