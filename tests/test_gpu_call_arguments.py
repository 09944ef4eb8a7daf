"""Index lists of a call that travel as kernel arguments instead of an upload, around the most that fits: prefix sums of the gate,
windows of the projector, row metadata of a verification and of greedy steps.  Against the oracle."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import ssd_oracle as O
from tests.parity import TOL_LOGP
from tests.test_gpu_ar_fallback import _check_against_oracle, _run_chain
from tests.test_gpu_gate import _run_and_compare, ctx  # noqa: F401
from tests.test_gpu_qformer import _check
from tests.test_gpu_verify import _compare, _run_gpu
from workloads import WORKLOADS, make_model_weights
from workloads.configs import ModelCfg
from workloads.synth import VerifyInputs

pytestmark = pytest.mark.gpu


# 1280 utterances as pairs of a 32-bit sum and a 16-bit length; one more, or one of 65536 frames before an odd sum, is uploaded
@pytest.mark.parametrize("B,at,frames", [(257, 0, 1), (258, 3, 9), (639, 5, 2), (1279, 0, 3), (1280, 1279, 4), (1281, 1280, 4), (300, 100, 65535),
                                         (300, 100, 65536), (300, 101, 65536), (301, 300, 65536)])
def test_gate_prefix_sums_in_pairs(ctx, B, at, frames):  # noqa: F811
    T = 1 + np.arange(B) * 7 % 5
    T[at] = frames
    cu = np.concatenate([[0], np.cumsum(T)])
    logits = torch.randn(int(cu[-1]), 8, generator=torch.Generator().manual_seed(B + at)) * 3
    _run_and_compare(ctx, logits, cu, 0, 1.5)


# 448 windows as arguments, more listed on the device from the prefix sums of up to 1280 utterances, else uploaded
@pytest.mark.parametrize("B,extra", [(447, 0), (448, 0), (449, 0), (7, 441), (7, 442), (300, 900), (1280, 30), (1281, 30)])
def test_projector_windows(B, extra):
    from paper_2603_11243_amd.binding import Context
    window = 5
    r, g = np.random.default_rng(B + extra), torch.Generator().manual_seed(B)
    T = r.integers(1, window + 1, B)                         # one window each
    np.add.at(T, r.integers(0, B, extra), window)
    cu = np.concatenate([[0], np.cumsum(T)]).astype(np.int32)
    enc = torch.randn(int(cu[-1]), 64, generator=g).to(torch.bfloat16)
    q, wk, wv, wo = (torch.randn(s, generator=g).mul(s[1] ** -0.5).to(torch.bfloat16) for s in ((2, 256), (256, 64), (256, 64), (256, 256)))
    c = Context()
    c.set_qformer(q.cuda(), wk.cuda(), wv.cuda(), wo.cuda(), n_heads=4, window=window)
    c.reserve(max_frames=len(enc), max_utts=B)
    got, cu_s = c.qformer_pool(enc.cuda(), cu)
    got = got.float().cpu().numpy()
    c.close()
    want, cu_want = O.qformer_window_pool(enc, cu, q, wk, wv, wo, 4, window)
    assert np.array_equal(cu_s, cu_want) and cu_s[-1] == 2 * (B + extra)
    _check(got, want)


def _inputs(m, lengths, seed):
    S, P, U = map(list, zip(*lengths))
    cu = lambda a: np.concatenate([[0], np.cumsum(a)]).astype(np.int32)
    r = np.random.default_rng(seed)
    emb = torch.randn(sum(S), m.d_model, generator=torch.Generator().manual_seed(seed))
    return VerifyInputs(emb if m.dtype == "f32" else emb.to(torch.bfloat16), cu(S), r.integers(0, m.vocab, sum(P)).astype(np.int32), cu(P),
                        r.integers(0, m.vocab, sum(U)).astype(np.int32), cu(U))


# 960 words: two a row, one a draft token, four an attention tile of 16 (fp32) or 64 rows
@pytest.mark.parametrize("dtype,rows,draft", [("f32", 360, 148), ("f32", 360, 149), ("bf16", 400, 132), ("bf16", 400, 133), ("f32", 20, 3)])
def test_verify_metadata(dtype, rows, draft):
    m = ModelCfg(1, 64, 2, 1, 32, 64, 130, dtype="f32") if dtype == "f32" else ModelCfg(1, 256, 2, 1, 128, 256, 512)
    wl = replace(WORKLOADS["cfg1_tiny_f32" if dtype == "f32" else "cfg3_1b_ragged64"], model=m)
    w = make_model_weights(m, 30 + rows)
    vi = _inputs(m, [(rows - draft - 5, 5, draft)], rows + draft)
    tau = 1.0 / m.vocab
    _compare(wl, w, vi, _run_gpu(wl, w, vi, tau), tau)


# twelve utterances: two words each and three a step and utterance; 26 steps are 960
@pytest.mark.parametrize("n_steps", [2, 26, 27])
def test_greedy_step_metadata(n_steps):
    m = ModelCfg(1, 64, 2, 1, 32, 64, 130, dtype="f32")
    wl = replace(WORKLOADS["cfg1_tiny_f32"], model=m)
    w = make_model_weights(m, 33)
    vi = _inputs(m, [(3 + b % 4, 2, 2) for b in range(12)], n_steps)
    res = _run_chain(wl, w, vi, 0.9, n_steps)                # no random token is that likely: all are rejected
    assert len(res[1]) == 12
    _check_against_oracle(wl, w, vi, 0.9, n_steps, *res, tol=TOL_LOGP["f32"])
