"""ctc_gate where its launches change: batches around the most whose prefix sums travel as kernel arguments, and fp32 rows
around the chunk counts of its layouts.  Against the oracle."""
import numpy as np
import pytest
import torch

from tests.test_gpu_gate import _run_and_compare, ctx  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 255, 256, 257])
def test_prefix_sums_as_arguments(ctx, B):  # noqa: F811
    T = 1 + np.arange(B) * 7 % 5
    cu = np.concatenate([[0], np.cumsum(T)])
    logits = torch.randn(int(cu[-1]), 40, generator=torch.Generator().manual_seed(B)) * 3
    _run_and_compare(ctx, logits, cu, 0, 2.0)


# up to 512 scores two chunks of 64 lanes for few frames, six or eight chunks of 16 lanes for more; then six or eight of 64
@pytest.mark.parametrize("V,n", [(V, 37) for V in (252, 256, 260, 320, 384, 388, 508, 512, 516, 1020, 1024, 1028, 1280, 1284, 1532, 1536, 1540)]
                         + [(V, n) for V in (260, 320, 324, 380, 384) for n in (2048, 2049)]
                         + [(V, n) for V in (388, 448, 508, 512) for n in (8192, 8193)])
def test_fp32_rows_around_chunk_counts(ctx, V, n):  # noqa: F811
    g = torch.Generator().manual_seed(V)
    logits = torch.randn(n, V, generator=g) * 3
    logits[5, ::2] = -float("inf")
    logits[6] = torch.round(logits[6])                      # ties
    logits[n - 1, V - 1] = logits[n - 2, V - 1] = 20        # the last score of the last rows
    _run_and_compare(ctx, logits, [0, 1, 17, n], 0, 3.0)
