"""GPU parity of the projector's windowed cross-attention (qformer_pool, through the C ABI) against the oracle."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from oracle import ssd_oracle as O
from workloads import WORKLOADS
from workloads.synth import make_ctc_head_batch, make_qformer_weights

pytestmark = pytest.mark.gpu


def _check(g_gpu, g_ref):
    """Rows are stored as bf16 (2^-9 relative rounding) from bf16 operands: elementwise within 2e-2 of the row's
    largest magnitude, and 1e-2 in relative L2 norm per row (a wrong window, head or query is O(1) in both)."""
    assert g_gpu.shape == g_ref.shape
    scale = np.abs(g_ref).max(axis=1, keepdims=True)
    assert (np.abs(g_gpu - g_ref) <= 2e-2 * scale).all(), float((np.abs(g_gpu - g_ref) / scale).max())
    rel = np.linalg.norm(g_gpu - g_ref, axis=1) / np.linalg.norm(g_ref, axis=1)
    assert rel.max() < 1e-2, float(rel.max())
    return float(rel.max())


@pytest.mark.parametrize("name,B,d_out", [("cfg3_1b_ragged64", 10, 2048), ("cfg5_3b_ragged128", 6, 3072), ("cfg1_tiny_f32", 2, 256)])
def test_qformer_pool_matches_oracle(name, B, d_out):
    """Paper shapes (1024-wide encoder states, 16 heads, windows of 15 frames, 3 queries) on ragged utterances
    whose lengths are mostly not multiples of 15; the third case has fewer than 128 frames in total (the few-row
    GEMM tiles)."""
    from paper_2603_11243_amd.binding import Context
    wl = replace(WORKLOADS[name], B=B, model=replace(WORKLOADS[name].model, dtype="bf16"))
    if name == "cfg1_tiny_f32":
        wl = replace(wl, seconds=(1.0, 2.5))
    hb = make_ctc_head_batch(wl, d_enc=1024, V_ctc=348)
    qw = make_qformer_weights(wl.seed, d_out=d_out)
    T = np.diff(hb.cu_frames)
    assert (T % 15 != 0).any()
    ctx = Context()
    try:
        ctx.set_qformer(*(qw[k].cuda() for k in ("q_proj", "w_k", "w_v", "w_o")), n_heads=16, window=15)
        ctx.reserve(max_frames=int(hb.cu_frames[-1]), max_utts=B)
        g, cu_s = ctx.qformer_pool(hb.enc_h.cuda(), hb.cu_frames)
        torch.cuda.synchronize()
        g2, _ = ctx.qformer_pool(hb.enc_h.cuda(), hb.cu_frames)            # same buffers, same answer
        torch.cuda.synchronize()
        assert torch.equal(g, g2)
    finally:
        ctx.close()
    ref, cu_ref = O.qformer_window_pool(hb.enc_h, hb.cu_frames, qw["q_proj"], qw["w_k"], qw["w_v"], qw["w_o"], 16, 15)
    assert np.array_equal(cu_s, cu_ref) and cu_s[-1] == 3 * sum(-(-int(t) // 15) for t in T)
    worst = _check(g.float().cpu().numpy(), ref)
    print(f"{wl.name}: {int(hb.cu_frames[-1])} frames -> {int(cu_s[-1])} rows, worst relative row error {worst:.2e}")


# 17 column tiles of 64 for scores and values, 48 for the output: both projections pass from the few-row kernels over 32 x 64 (K split in the
# workgroup), 64 x 64, 64 x 128 and 128 x 128 tiles to the 256-wide ones, at 128, 480, 960, 1792 and 3584 frames and at 128, 160, 320, 640 and 1280 rows
@pytest.mark.parametrize("frames", [128, 129, 768, 769, 1536, 1537, 3264, 3265, 6730])
def test_qformer_pool_frame_counts(frames):
    from paper_2603_11243_amd.binding import Context
    g = torch.Generator().manual_seed(frames)
    h = torch.randn(frames, 1024, generator=g).bfloat16()
    qw = make_qformer_weights(frames, d_out=3072)
    cu = np.array([0, 16, frames // 2, frames], dtype=np.int32)
    ctx = Context()
    try:
        ctx.set_qformer(*(qw[k].cuda() for k in ("q_proj", "w_k", "w_v", "w_o")), n_heads=16, window=15)
        ctx.reserve(max_frames=frames, max_utts=3)
        got, cu_s = ctx.qformer_pool(h.cuda(), cu)
        got = got.float().cpu().numpy()
    finally:
        ctx.close()
    ref, cu_ref = O.qformer_window_pool(h, cu, qw["q_proj"], qw["w_k"], qw["w_v"], qw["w_o"], 16, 15)
    assert np.array_equal(cu_s, cu_ref)
    _check(got, ref)


# The 1088 columns of scores and values are 17 tiles of 64 and 9 of 128: K-split 32 x 64 tiles up to 480 frames, 64 x 64 to 960,
# 64 x 128 to 1792, 128 x 128 to 3584.
@pytest.mark.parametrize("frames", [160, 161, 480, 481, 960, 961, 1792, 1793, 3584, 3585])
def test_qformer_pool_frames_around_tile_widths(frames):
    test_qformer_pool_frame_counts(frames)


# The pooling kernel: 16 frames of values in registers, a second pass for longer windows and for more than 1024 columns; widths that leave
# threads without a column; every number of queries.
@pytest.mark.parametrize("n_q,n_heads,d_h,window", [(1, 16, 64, 15), (2, 16, 1024, 16), (3, 16, 1088, 17), (4, 16, 2112, 32), (3, 4, 960, 31), (1, 1, 256, 3)])
def test_qformer_pool_windows_and_widths(n_q, n_heads, d_h, window):
    from paper_2603_11243_amd.binding import Context
    g = torch.Generator().manual_seed(d_h + window)
    r = lambda *s: (torch.randn(*s, generator=g) * s[-1] ** -0.5).bfloat16()
    lengths = [1, window, 3 * window + 1, 2 * window - 1, window + window // 2]
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    h = torch.randn(int(cu[-1]), 128, generator=g).bfloat16()
    q, w_k, w_v, w_o = torch.randn(n_q, d_h, generator=g).bfloat16(), r(d_h, 128), r(d_h, 128), r(256, d_h)
    ctx = Context()
    try:
        ctx.set_qformer(q.cuda(), w_k.cuda(), w_v.cuda(), w_o.cuda(), n_heads=n_heads, window=window)
        ctx.reserve(max_frames=int(cu[-1]), max_utts=len(lengths))
        got, cu_s = ctx.qformer_pool(h.cuda(), cu)
        got = got.float().cpu().numpy()
    finally:
        ctx.close()
    ref, cu_ref = O.qformer_window_pool(h, cu, q, w_k, w_v, w_o, n_heads, window)
    assert np.array_equal(cu_s, cu_ref)
    _check(got, ref)


def test_qformer_pool_argument_errors():
    from paper_2603_11243_amd.binding import Context, SsdError
    ctx = Context()
    try:
        h = torch.zeros((30, 1024), dtype=torch.bfloat16, device="cuda")
        ctx._qformer = (3, 1024, 2048, 15)
        with pytest.raises(SsdError, match="no projector set"):
            ctx.qformer_pool(h, [0, 30])
        qw = make_qformer_weights(1)
        with pytest.raises(SsdError, match="pairs"):
            ctx.set_qformer(*(qw[k].cuda() for k in ("q_proj", "w_k", "w_v", "w_o")), n_heads=32)     # 3 x 32 score rows
        ctx.set_qformer(*(qw[k].cuda() for k in ("q_proj", "w_k", "w_v", "w_o")), n_heads=16)
        with pytest.raises(SsdError, match="workspace"):
            ctx.qformer_pool(h, [0, 30])
        ctx.reserve(max_frames=30, max_utts=2)
        with pytest.raises(SsdError, match="increase strictly"):
            ctx.qformer_pool(h, [0, 30, 30])
    finally:
        ctx.close()


# From 28 K frames (20 K, 12 K for two queries, one) in windows of nine or more (six, three) the values are projected after the pooling,
# 16 windows to a workgroup: a last workgroup of 1 and of 15, windows of 4 and of 16 frames, every query count, encoder widths of one
# and several steps.  Fewer frames and shorter windows take the other order: the second line, and the last one just so.
@pytest.mark.parametrize("n_q,d_enc,window,windows", [(3, 1024, 15, 1937), (3, 64, 15, 2047), (2, 192, 16, 1552), (1, 128, 4, 4112), (1, 64, 16, 784), (3, 128, 10, 2881),
                                                      (3, 1024, 15, 1025), (3, 64, 15, 1039), (2, 192, 16, 1024), (1, 128, 1, 1040), (3, 128, 4, 1023),
                                                      (3, 64, 15, 1911), (3, 64, 8, 4096)])
def test_qformer_pool_values_after_pooling(n_q, d_enc, window, windows):
    from paper_2603_11243_amd.binding import Context
    g = torch.Generator().manual_seed(windows)
    r = lambda *s: (torch.randn(*s, generator=g) * s[-1] ** -0.5).bfloat16()
    last = max(1, window // 2)
    lengths = [window] * 5 + [1] + [window * (windows - 7) + last]      # whole windows, a one-frame window, a short last one
    cu = np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)
    h = torch.randn(int(cu[-1]), d_enc, generator=g).bfloat16()
    q, w_k, w_v, w_o = torch.randn(n_q, 1024, generator=g).bfloat16(), r(1024, d_enc), r(1024, d_enc), r(256, 1024)
    ctx = Context()
    try:
        ctx.set_qformer(q.cuda(), w_k.cuda(), w_v.cuda(), w_o.cuda(), n_heads=16, window=window)
        ctx.reserve(max_frames=int(cu[-1]), max_utts=len(lengths))
        got, cu_s = ctx.qformer_pool(h.cuda(), cu)
        got = got.float().cpu().numpy()
    finally:
        ctx.close()
    ref, cu_ref = O.qformer_window_pool(h, cu, q, w_k, w_v, w_o, 16, window)
    assert cu_s[-1] == n_q * windows and np.array_equal(cu_s, cu_ref)
    _check(got, ref)


def _unusual(kind, d_enc, windows, seed):
    """Weights and states of `windows` whole windows with `kind` in window 7; the oracle's rows, and which windows have none."""
    g = torch.Generator().manual_seed(seed)
    r = lambda *s: torch.randn(*s, generator=g)
    q, w_k, w_v = r(3, 1024), r(1024, d_enc) * d_enc ** -0.5, r(1024, d_enc) * d_enc ** -0.5
    h = r(15 * windows, d_enc)
    if kind == "large_states":                                 # far beyond the range of half; values and scores of unit spread
        h, w_k, w_v = h * 2.0 ** 20, w_k * 2.0 ** -20, w_v * 2.0 ** -20
    elif kind == "small_states":                               # far below it
        h, w_k, w_v = h * 2.0 ** -30, w_k * 2.0 ** 30, w_v * 2.0 ** 30
    elif kind == "uneven_weights":                             # 45 binades between the heads' rows of w_v
        w_v[3 * 64:4 * 64] *= 2.0 ** -45
    elif kind == "uneven_columns":                             # a tiny state column that its weights bring back
        h[:, 5] *= 2.0 ** -30
        w_v[:, 5] *= 2.0 ** 30
        w_k[:, 5] *= 2.0 ** 30
    elif kind == "large_values":
        w_v = w_v * 2.0 ** 17
    elif kind == "no_weight":                                  # every score falls with column 0
        q, w_k[:, 0] = q.abs(), 1.0
    q, w_k, w_v, h = (t.bfloat16() for t in (q, w_k, w_v, h))
    w_o = torch.eye(1024).bfloat16()
    ref, _ = O.qformer_window_pool(h, [0, len(h)], q, w_k, w_v, w_o, 16, 15)
    if kind in ("nan", "inf"):
        h[7 * 15 + 4, 11] = float(kind)
    if kind == "no_weight":                                    # a frame that no query gives any: as if it were not there
        rest = torch.cat([h[105:109], h[110:120]])
        ref[21:24] = O.qformer_window_pool(rest, [0, 14], q, w_k, w_v, w_o, 16, 15)[0]
        h[109, 0] = -float("inf")
    return q, w_k, w_v, w_o, h, ref


# The values pass through half in one order and are not rounded in the other: 40 windows take the one, 2048 the other
@pytest.mark.parametrize("windows", [40, 2048])
@pytest.mark.parametrize("kind", ["nan", "inf", "large_states", "small_states", "uneven_weights", "uneven_columns", "large_values", "no_weight"])
def test_qformer_pool_range(kind, windows):
    """States and weights of any scale give the oracle's rows (each head against its own largest magnitude), and states that are not
    finite give the flag and NaN in their window, unless no query gives their frame any weight.  Values beyond 65504 are clamped and flagged where they pass through half."""
    from paper_2603_11243_amd.binding import Context
    from workloads import make_model_weights
    q, w_k, w_v, w_o, h, ref = _unusual(kind, 128, windows, windows)
    model = WORKLOADS["cfg1_tiny_f32"].model                   # a context without a model has no flags
    ctx = Context(model, make_model_weights(model, 1))
    try:
        ctx.set_qformer(q.cuda(), w_k.cuda(), w_v.cuda(), w_o.cuda(), n_heads=16, window=15)
        ctx.reserve(max_frames=len(h), max_utts=1)
        ctx.device_flags()
        got, _ = ctx.qformer_pool(h.cuda(), [0, len(h)])
        got, flags = got.float().cpu().numpy(), ctx.device_flags()
    finally:
        ctx.close()
    keep = np.ones(len(ref), bool)
    if kind in ("nan", "inf"):
        keep[21:24] = False
        assert np.isnan(got[21:24]).all()
    clamped = kind == "large_values" and windows == 40
    assert flags == (2 if clamped or kind in ("nan", "inf", "no_weight") else 0)
    if clamped:
        assert np.isfinite(got).all() and np.abs(got).max() <= 65536      # 65504 as bfloat16
        return
    for head in range(16):
        if not (kind == "uneven_weights" and head == 3 and windows == 40):      # (values of 2^-45 are zeros in half)
            _check(got[keep, 64 * head:64 * head + 64], ref[keep, 64 * head:64 * head + 64])
