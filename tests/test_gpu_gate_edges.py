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


# one launch for both steps: utterances around a workgroup's 16 or 4 rows (one row fewer takes two launches), around the 192
# workgroups an utterance may have and the 2048 of a call, around 24 and 28 MiB, and through the 1024 frames a trip of the collapse.  Long
# and short ones in turn, so that every call finds the counts as the one before left them.
@pytest.mark.parametrize("dtype,V,rows", [("bfloat16", 512, 16), ("bfloat16", 40, 16), ("bfloat16", 1024, 4), ("float32", 256, 16), ("float32", 348, 4)])
def test_one_launch_around_its_limits(ctx, dtype, V, rows):  # noqa: F811
    long = rows * 192                                       # 1024 frames are more than that at four rows
    for T in ([rows], [rows - 1, rows], [rows, rows + 1, 2 * rows - 1, 2 * rows], [long, rows], [long + 1, rows], [1023, 1024, 1025],
              [rows] * 256, [rows + 3] * 257, [rows * 8] * 256, [rows * 8] * 255 + [rows * 8 + 1]):
        cu = np.concatenate([[0], np.cumsum(T)])
        g = torch.Generator().manual_seed(len(T) + T[0])
        z = torch.randn(int(cu[-1]), V, generator=g) * 3
        lab = torch.randint(0, V, (len(z) // 3 + 1,), generator=g).repeat_interleave(3)[: len(z)]
        lab[torch.rand(len(z), generator=g) < 0.4] = 7
        z[torch.arange(len(z)), lab] += 12
        z = z.to(getattr(torch, dtype))
        z[len(z) // 2] = -float("inf")
        z[len(z) // 2, V - 1] = 0
        _run_and_compare(ctx, z, cu, 7, 0.7)


@pytest.mark.parametrize("n", [24576 - 16, 24576, 24576 + 16, 28672 - 16, 28672, 28672 + 16])
def test_one_launch_around_its_bytes(ctx, n):  # noqa: F811
    z = torch.randn(n, 512, generator=torch.Generator().manual_seed(n)) * 3
    _run_and_compare(ctx, z.to(torch.bfloat16), np.linspace(0, n, 65).astype(np.int32), 0, 2.0)


def test_one_launch_in_a_graph(ctx):  # noqa: F811
    """A captured call, which takes two launches, replayed next to eager calls of other sizes, which take one."""
    T = [40, 300, 16, 700]
    cu = np.concatenate([[0], np.cumsum(T)]).astype(np.int32)
    g = torch.Generator().manual_seed(5)
    z = (torch.randn(int(cu[-1]), 348, generator=g) * 3).cuda()
    other = (torch.randn(640, 348, generator=g) * 3).cuda()
    ctx.reserve(max_frames=4096, max_utts=64)
    want = {k: v.clone() for k, v in ctx.ctc_gate(z, cu, 0, 2.0, want_frames=True).items()}
    out = {k: torch.zeros_like(v) for k, v in want.items()}
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    from paper_2603_11243_amd.binding import Context
    c = Context(stream=side)
    try:
        c.reserve(max_frames=4096, max_utts=64)
        with torch.cuda.graph(graph, stream=side):
            c.ctc_gate(z, cu, 0, 2.0, out=out)
        for i in range(4):
            for v in out.values():
                v.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for u in range(len(T)):
                n = int(want["draft_len"][u])
                assert torch.equal(out["draft_ctc"][cu[u]:cu[u] + n], want["draft_ctc"][cu[u]:cu[u] + n]), (i, u)
            for k in want:
                if k != "draft_ctc":
                    assert torch.equal(out[k], want[k]), (i, k)
            c.ctc_gate(other, np.arange(0, 641, 64 >> (i % 2)).astype(np.int32), 0, 2.0)
            torch.cuda.synchronize()
    finally:
        c.close()


def _kernel_nodes(graph):
    import ctypes
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(line.split()[-1] for line in f if "libamdhip64" in line))
    raw, n = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t()
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(n)) == 0
    return n.value


def test_captured_calls_are_independent(ctx):  # noqa: F811
    """Two captured calls of one context with their own outputs, replayed on two streams at once: nothing may be shared.  A call with
    frame outputs and prefix sums as arguments is the two kernels and nothing else; one launch would count in the context's memory."""
    from paper_2603_11243_amd.binding import Context
    side = torch.cuda.Stream()
    c = Context(stream=side)
    calls = []
    try:
        c.reserve(max_frames=4096, max_utts=64)
        for seed, T in ((1, [200, 16, 300, 90]), (2, [500, 40, 77])):
            cu = np.concatenate([[0], np.cumsum(T)]).astype(np.int32)
            z = (torch.randn(int(cu[-1]), 512, generator=torch.Generator().manual_seed(seed)) * 3).to(torch.bfloat16).cuda()
            ctx.reserve(max_frames=4096, max_utts=64)
            want = {k: v.clone() for k, v in ctx.ctc_gate(z, cu, 0, 2.0, want_frames=True).items()}
            out = {k: torch.zeros_like(v) for k, v in want.items()}
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph(keep_graph=True)
            with torch.cuda.graph(graph, stream=side):
                c.ctc_gate(z, cu, 0, 2.0, out=out)
            assert _kernel_nodes(graph) == 2
            graph.instantiate()
            calls.append((graph, torch.cuda.Stream(), cu, z, want, out))
        for i in range(10):
            for call in calls:
                for v in call[5].values():
                    v.zero_()
            torch.cuda.synchronize()
            for _ in range(20):
                for graph, stream, *_ in calls:
                    with torch.cuda.stream(stream):
                        graph.replay()
            torch.cuda.synchronize()
            for _, _, cu, _, want, out in calls:
                for u in range(len(cu) - 1):
                    n = int(want["draft_len"][u])
                    assert torch.equal(out["draft_ctc"][cu[u]:cu[u] + n], want["draft_ctc"][cu[u]:cu[u] + n]), (i, u)
                for k in want:
                    if k != "draft_ctc":
                        assert torch.equal(out[k], want[k]), (i, k)
    finally:
        torch.cuda.synchronize()
        c.close()


def test_device_memory_is_allocated_when_the_context_is_made():
    from torch.profiler import ProfilerActivity, profile
    from paper_2603_11243_amd.binding import Context

    def runtime_calls(f):
        with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
            result = f()
            torch.cuda.synchronize()
        return result, [e.key for e in prof.key_averages()]

    buf = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    c, made = runtime_calls(Context)
    try:
        _, then = runtime_calls(lambda: c.set_workspace(buf))
        assert "hipMalloc" in made                              # (what the profiler calls it)
        assert not any("Malloc" in key or "Memset" in key for key in then), then
    finally:
        c.close()


# (28 MiB; 2000 blocks of the longest utterance times MiB: 178 x 11.1 and 180 x 11.3)
@pytest.mark.parametrize("T,one", [([250], True), ([16] * 256, True), ([15, 250], False), ([16] * 257, False), ([448] * 64, True),
                                   ([448] * 63 + [464], False), ([2848] * 4, True), ([2880] * 4, False)])
def test_which_calls_take_one_launch(ctx, T, one):  # noqa: F811
    from torch.profiler import ProfilerActivity, profile
    cu = np.concatenate([[0], np.cumsum(T)]).astype(np.int32)
    z = torch.randn(int(cu[-1]), 512, generator=torch.Generator().manual_seed(1)).to(torch.bfloat16).cuda()
    ctx.reserve(max_frames=len(z), max_utts=512)
    out = ctx.ctc_gate(z, cu, 0, 2.0)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as prof:
        ctx.ctc_gate(z, cu, 0, 2.0, out=out)
        torch.cuda.synchronize()
    names = [e.key for e in prof.key_averages() if "gate_" in e.key]
    assert len(names) == (1 if one else 2) and ("gate_fused" in names[0]) == one, names
