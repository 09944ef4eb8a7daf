"""The fp32 decoder at the sizes where its tiles end: rows around the 16- and 32-row tiles, column pairs and vocabularies
that are no multiple of a tile, head widths below, at and above one 64-dim block, K ranges that do not divide over the
four wavefronts.  Verification, acceptance and fallback against the oracle."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from tests.parity import TOL_LOGP
from tests.test_gpu_ar_fallback import _check_against_oracle, _run_chain
from tests.test_gpu_verify import _compare, _run_gpu
from workloads import WORKLOADS, make_model_weights
from workloads.configs import ModelCfg
from workloads.synth import VerifyInputs

pytestmark = pytest.mark.gpu

# layers, d_model, q heads, kv heads, head_dim, d_ff, vocab
SHAPES = [(1, 16, 2, 1, 8, 16, 33), (2, 48, 4, 2, 36, 80, 130), (1, 272, 2, 2, 72, 48, 63), (1, 1008, 4, 1, 128, 144, 4097),
          (2, 256, 4, 4, 64, 1024, 4096)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("lengths", [[(1, 0, 1)], [(9, 4, 3), (1, 0, 30), (10, 4, 3)], [(40, 16, 9), (120, 16, 150), (3, 0, 0)]])
def test_f32_edges_of_tiles(shape, lengths):
    m = ModelCfg(*shape, dtype="f32")
    wl = replace(WORKLOADS["cfg1_tiny_f32"], model=m)
    w = make_model_weights(m, 40 + shape[1])
    w["embed"] *= 25                              # rows of unit size: attention and hidden units are not all alike
    S, P, U = map(list, zip(*lengths))
    cu = lambda a: np.concatenate([[0], np.cumsum(a)]).astype(np.int32)
    r, g = np.random.default_rng(shape[1]), torch.Generator().manual_seed(shape[1])
    vi = VerifyInputs(torch.randn(sum(S), m.d_model, generator=g), cu(S), r.integers(0, m.vocab, sum(P)).astype(np.int32), cu(P),
                      r.integers(0, m.vocab, sum(U)).astype(np.int32), cu(U))
    tau = 1.0 / m.vocab
    _compare(wl, w, vi, _run_gpu(wl, w, vi, tau), tau)
    if m.head_dim % 8 == 0:                       # what ar_fallback takes
        res = _run_chain(wl, w, vi, tau, 3)
        if len(res[1]):
            _check_against_oracle(wl, w, vi, tau, 3, *res, tol=TOL_LOGP["f32"])


# Rows beyond one round of the smallest tiles.  tiny (K = 256 / 1024), 908 rows, 600 of them scored: QKV 32 x 16 pairs, gate/up 32 x 32 and on
# the scored rows 32 x 16, O and down 32 x 32 with K over four and eight wavefronts, on all rows and on the scored ones.  768 wide: gate/up of
# K > 512 in 32 x 32.  1008 wide: QKV and gate/up in 32 x 16 with K over eight wavefronts.
@pytest.mark.parametrize("shape", [(2, 256, 4, 4, 64, 1024, 512), (1, 768, 4, 2, 64, 3072, 512), (1, 1008, 4, 1, 128, 144, 512)])
@pytest.mark.parametrize("lengths", [[(150, 8, 300), (149, 1, 300)], [(270, 0, 360), (300, 2, 247), (200, 5, 301)]])
def test_f32_rows_beyond_one_round(shape, lengths):
    m = ModelCfg(*shape, dtype="f32")
    wl = replace(WORKLOADS["cfg1_tiny_f32"], model=m)
    w = make_model_weights(m, 50 + shape[1])
    w["embed"] *= 25
    S, P, U = map(list, zip(*lengths))
    cu = lambda a: np.concatenate([[0], np.cumsum(a)]).astype(np.int32)
    r, g = np.random.default_rng(shape[1]), torch.Generator().manual_seed(shape[1])
    vi = VerifyInputs(torch.randn(sum(S), m.d_model, generator=g), cu(S), r.integers(0, m.vocab, sum(P)).astype(np.int32), cu(P),
                      r.integers(0, m.vocab, sum(U)).astype(np.int32), cu(U))
    tau = 1.0 / m.vocab
    _compare(wl, w, vi, _run_gpu(wl, w, vi, tau), tau)
