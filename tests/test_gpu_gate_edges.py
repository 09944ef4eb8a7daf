"""ctc_gate where its launches change: batches around the most whose prefix sums travel as kernel arguments, and fp32 rows
around the six 16-lane chunks of the wide layout.  Against the oracle."""
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


@pytest.mark.parametrize("V", [316, 320, 324, 380, 384, 388])
def test_fp32_rows_of_six_chunks(ctx, V):  # noqa: F811
    g = torch.Generator().manual_seed(V)
    logits = torch.randn(37, V, generator=g) * 3
    logits[5, ::2] = -float("inf")
    logits[6] = torch.round(logits[6])                      # ties
    _run_and_compare(ctx, logits, [0, 1, 17, 37], 0, 3.0)
