"""The decode attention of 16-bit models launched by itself on cache rows of the caller's choice, against 64 bits: what tokens and
cache rows of a whole step cannot show, the ends of its number range and the precision of its probabilities."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2603_11243_amd.binding import lib

pytestmark = pytest.mark.gpu

HD = 128
DTYPE = {"f16": torch.float16, "bf16": torch.bfloat16}
LOG2_SCALE = np.log2(np.e) / np.sqrt(HD)


def _launch(operand, fused, q, k, v, n):
    """q [Br, query heads, 128] over the first n[b] rows of k, v [Br, slots, K/V heads, 128]; fused: the last of them is not in the
    cache but the new row, and the products of the projection come as partial sums of three K splits (all but one of them zero)."""
    Br, Hq, _ = q.shape
    slots, Hkv = k.shape[1:3]
    p = lambda t: C.c_void_p(t.data_ptr())
    out = torch.zeros(Br, Hq, HD, dtype=DTYPE[operand], device="cuda")
    start = torch.arange(Br, dtype=torch.int32, device="cuda") * slots
    rows = torch.tensor(n, dtype=torch.int32, device="cuda")
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    if fused:
        at = torch.arange(Br, device="cuda"), rows.long() - 1
        new_k, new_v = k[at].float(), v[at].float()
        k, v = k.clone(), v.clone()
        k[at], v[at] = float("nan"), float("nan")            # written by the launch, not read
        pairs = lambda t: t.view(Br, -1, 2, 2, 32).transpose(2, 3).reshape(Br, -1)     # dims i and i + 64 lie 32 columns apart
        packed = torch.cat([pairs(q.float()), pairs(new_k), new_v.reshape(Br, -1)], 1)
        part = torch.zeros(3, *packed.shape, device="cuda")
        part[1] = packed
        rope = torch.tensor([1.0, 0.0], device="cuda").repeat(max(n), 64, 1)          # no rotation
        flags = torch.zeros(64, dtype=torch.int32, device="cuda")
        f = lib()._ZN3ssd24launch_decode_attn_fusedEPKfiS1_PvS2_PKiS4_iiiS2_PibP12ihipStream_t
        f.restype = None
        f(p(part), 3, p(rope), p(k), p(v), p(start), p(rows), Br, Hq, Hkv, p(out), p(flags), C.c_bool(operand == "bf16"), st)
    else:
        qkv = torch.cat([q.reshape(Br, -1), torch.zeros(Br, 2 * Hkv * HD, dtype=q.dtype, device="cuda")], 1)
        f = lib()._ZN3ssd18launch_decode_attnEPKvS1_S1_PKiS3_iiiPvbP12ihipStream_t
        f.restype = None
        f(p(qkv), p(k), p(v), p(start), p(rows), Br, Hq, Hkv, p(out), C.c_bool(operand == "bf16"), st)
    torch.cuda.synchronize()
    return out.double().cpu().numpy()


def _exact(q, k, v, n):
    """(out, sum of p |v|) in 64 bits"""
    q, k, v = (t.double().cpu().numpy() for t in (q, k, v))
    out, mag = np.zeros_like(q), np.zeros_like(q)
    for b in range(len(q)):
        for h in range(q.shape[1]):
            kv = h * k.shape[2] // q.shape[1]
            s = k[b, :n[b], kv] @ q[b, h] * LOG2_SCALE
            p = np.exp2(s - s.max())
            p /= p.sum()
            out[b, h], mag[b, h] = p @ v[b, :n[b], kv], p @ abs(v[b, :n[b], kv])
    return out, mag


def _random(operand, heads, n, seed):
    g = torch.Generator().manual_seed(seed)
    r = lambda *s: torch.randn(*s, generator=g).to(DTYPE[operand]).cuda()
    return r(len(n), heads[0], HD), r(len(n), max(n), heads[1], HD), r(len(n), max(n), heads[1], HD)


# Output: one rounding to eight bits (2^-9 of it).  Sums over the keys: fp32, a few ulp of what is added; 2^-18 of that is allowed.
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("heads", [(2, 2), (4, 2), (3, 1)])
def test_bfloat16_values_up_to_the_end_of_the_range(fused, heads):
    n = [1, 2, 31, 33, 40, 129, 300]
    q, k, v = _random("bf16", heads, n, 3)
    v = (v.float().clamp(-3.5, 3.5) * 2.0 ** 118).bfloat16()     # a sum of 300 of them is within fp32's range
    got, (want, mag) = _launch("bf16", fused, q, k, v, n), _exact(q, k, v, n)
    assert np.isfinite(got).all()
    assert (abs(got - want) <= 2.0 ** -8 * abs(want) + 2.0 ** -18 * mag).all()


# An infinite value (the caller's cache is not checked; new rows of bfloat16 models are stored as they are) is the output of its column,
# whichever pieces its probability has, and nothing else's.
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("operand", ["f16", "bf16"])
def test_infinite_values(operand, fused):
    n = [31, 40, 200]
    q, k, v = _random(operand, (4, 2), n, 4)
    want, mag = _exact(q, k, v, n)
    for b, rows in enumerate(n):
        at = [0, rows // 2] + ([rows - 1] if fused and operand == "bf16" else [])        # the last one: the new row
        for i, row in enumerate(at):
            v[b, row, 1, 5 + 20 * i] = float("inf") if (b + i) % 2 else float("-inf")
            want[b, 2:, 5 + 20 * i] = float("inf") if (b + i) % 2 else float("-inf")
    got = _launch(operand, fused, q, k, v, n)
    inf = np.isinf(want)
    assert (got[inf] == want[inf]).all()
    tol = (2.0 ** -8 if operand == "bf16" else 2.0 ** -11) * abs(want) + 2.0 ** -18 * mag
    assert (abs(got[~inf] - want[~inf]) <= tol[~inf]).all()


# 64 K/V heads: 16 KB a row, 2^18 rows are 4 GiB.  All keys are alike; the rows behind that point hold the only values.
@pytest.mark.parametrize("fused", [False, True])
def test_cached_rows_beyond_four_gib(fused):
    rows, far = 2 ** 18, 64
    n = [rows + far]
    q = torch.ones(1, 64, HD, dtype=torch.float16, device="cuda")
    k = torch.zeros(1, n[0] + 1, 64, HD, dtype=torch.float16, device="cuda")
    v = torch.zeros_like(k)
    v[:, rows:] = 1024.0
    got = _launch("f16", fused, q, k, v, n)
    want = 1024.0 * far / n[0]                               # sums of whole numbers below 2^24: one rounding to 11 bits, one division
    assert (abs(got - want) <= 2.0 ** -10 * want).all()


# One key with the value 0, and 4095 whose probabilities are 2^-40.8 of its own, with values that make up for it.
@pytest.mark.parametrize("operand", ["f16", "bf16"])
def test_small_probabilities_count(operand):
    n = [4096]
    q = torch.zeros(1, 2, HD, dtype=DTYPE[operand], device="cuda")
    q[..., 0] = 16.0
    k, v = torch.zeros(1, 4096, 1, HD, dtype=q.dtype, device="cuda"), torch.full((1, 4096, 1, HD), 32768.0, dtype=q.dtype, device="cuda")
    k[:, 0, :, 0], v[:, 0] = 20.0, 0.0
    got, (want, _) = _launch(operand, False, q, k, v, n), _exact(q, k, v, n)
    assert want.min() > 2.0 ** -14                               # a normal number of either type
    # the exponent 40.8 in fp32 (2^-19 ln 2 of the probability), sums, output
    assert (abs(got - want) <= (2.0 ** -8 if operand == "bf16" else 2.0 ** -10) * want).all()


# Two probabilities, 1 and p2 (0.8 to 1) before the division: the second one's keys, three of them alike, hold -V / p2 in three pieces, so that
# the output is the error of p2.  It may be an ulp of the exponential function (2^-24), the rounding of the score (2^-25 at most, below 1) and of the
# factor to base 2 (2^-24 of 0.3), times ln 2, times 1.23 V; the sums of the products lose two ulp of V at most.  Together 3.9 ulp of V.
@pytest.mark.parametrize("operand", ["f16", "bf16"])
def test_probabilities_have_the_precision_of_fp32(operand):
    V, Br = 2.0 ** 14, 256
    g = torch.Generator().manual_seed(9)
    a = (1 + torch.rand(Br, generator=g)).to(DTYPE[operand]).cuda()
    b = (-0.1 - torch.rand(Br, generator=g)).to(a.dtype).cuda()
    q, k, v = (torch.zeros(Br, s, 1, HD, dtype=a.dtype, device="cuda") for s in (1, 4, 4))
    q[:, 0, 0, 0] = a
    k[:, 1:, 0, 0] = b[:, None]
    v[:, 0] = V
    p2 = torch.exp2(a.double() * b.double() * LOG2_SCALE)
    rest = -V / p2
    for i in range(3):
        v[:, 1 + i, 0] = rest[:, None].to(a.dtype)
        rest = rest - v[:, 1 + i, 0, 0].double()
    assert 0.7 < p2.min() and p2.max() < 1
    q, n = q[:, :, 0], [4] * Br
    got, (want, _) = _launch(operand, False, q, k, v, n), _exact(q, k, v, n)
    err = abs(got - want).max(axis=(1, 2)) * (1 + 3 * p2.cpu().numpy()) / (V * 2.0 ** -24)
    print(f"errors in ulp of V: largest {err.max():.2f}, root mean square {np.sqrt((err ** 2).mean()):.2f}")
    assert err.max() <= 3.9 * (1 + 2.0 ** -8)                # and the rounding of the output
