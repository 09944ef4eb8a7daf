"""The 16-bit decoder on up to 128 rows, at the edges of its kernels: row blocks of 32, K ranges that do not divide over
splits and wavefronts, the rule for few column tiles, and the decode attention for every head-group ratio with contexts
around its blocks of 32 keys and 128-key passes.  Against the oracle."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from tests.test_gpu_ar_fallback import _check_against_oracle, _run_chain
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


@pytest.mark.parametrize("heads", [(2, 2), (2, 1), (6, 2), (4, 1)])
@pytest.mark.parametrize("operand", ["f16", "bf16"])
def test_decode_attention_contexts(heads, operand):
    m = ModelCfg(1, 256, *heads, 128, 256, 512, dtype="bf16")
    wl = replace(WORKLOADS["cfg3_1b_ragged64"], model=m)
    w = make_model_weights(m, 60 + heads[0])
    # a rejected draft leaves a context of S + P rows or a little more
    vi = _inputs(m, [(c, 0, 3) for c in (1, 2, 30, 31, 32, 33, 63, 64, 65, 126, 127, 128, 129, 255, 256, 257, 300)], 7)
    res = _run_chain(wl, w, vi, 0.5, 4, operand)             # nothing is that likely: every utterance is rejected
    assert len(res[1]) == 17
    tol = 2e-2 if operand == "f16" else 0.1                  # the stated tolerance; bfloat16 operands: eight times the rounding, two layers' worth of it in one
    _check_against_oracle(wl, w, vi, 0.5, 4, *res, tol=tol)


@pytest.mark.parametrize("Br", [33, 64, 65, 96, 97, 128, 129])
def test_fallback_row_blocks(Br):
    m = ModelCfg(1, 768, 6, 2, 128, 3200, 512, dtype="bf16")
    wl = replace(WORKLOADS["cfg3_1b_ragged64"], model=m)
    w = make_model_weights(m, 70 + Br)
    vi = _inputs(m, [(1 + 5 * (b % 9), 1, 1) for b in range(Br)], Br)
    res = _run_chain(wl, w, vi, 0.5, 2)
    assert len(res[1]) == Br
    _check_against_oracle(wl, w, vi, 0.5, 2, *res, sample=range(0, Br, 8))


# 768 columns are 3 (12) tiles per 128 rows: K splits of 128 x 64 tiles while they use more CUs, then of 128 x 256 tiles,
# over 12 and 50 K steps; QKV and gate/up pass from 64 x 64 over 128 x 64 and 64 x 128 to the 256-wide tiles
@pytest.mark.parametrize("M", [129, 256, 257, 500, 641, 1100, 1700])
def test_verify_mid_rows(M):
    m = ModelCfg(2, 768, 6, 2, 128, 3200, 512, dtype="bf16")
    wl = replace(WORKLOADS["cfg3_1b_ragged64"], model=m)
    w = make_model_weights(m, 80 + M)
    vi = _inputs(m, [(M // 2 - 40, 3, 37), (M - M // 2 - 9, 4, 5)], M)
    tau = 1.0 / m.vocab
    _compare(wl, w, vi, _run_gpu(wl, w, vi, tau), tau)
