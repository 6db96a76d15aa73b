"""Fused execs in place: their stage times cover the whole call, and they run
from a captured graph."""
import pytest

from paper_1302_6189_amd import fftrw

pytestmark = pytest.mark.gpu


def _spans(f, n=8):
    """least milliseconds between two events around f()"""
    import torch
    best = []
    for _ in range(n):
        e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        e0.record()
        f()
        e1.record()
        torch.cuda.synchronize()
        best.append(e0.elapsed_time(e1))
    return best


@pytest.mark.parametrize("dims", [(256, 256, 256), (160, 160, 160), (64, 64, 64, 64)])
@pytest.mark.parametrize("flags", [0, fftrw.FLAG_LEAVE_PERMUTED])
def test_stage_times(gpu_lib, dims, flags):
    # what the stages leave of the time between events around the call is the
    # events' own, in place as out of place; a copy that no stage holds (an odd
    # number of transposes) would be in it
    import torch
    plan = fftrw.Plan(dims, 8, None, flags=flags)
    assert plan.describe()[1].startswith("fused|")
    x = torch.zeros(dims, dtype=torch.complex64, device="cuda")
    y = torch.empty_like(x)
    rest = {}
    for name, out in (("in", x), ("out", y)):
        plan.set_timing(True)
        left = []
        for _ in range(8):
            span = _spans(lambda: plan.exec_fwd(x, out), 1)[0]
            stages = plan.timings()
            assert len(stages) == len(dims)
            left.append(span - sum(stages))
        rest[name] = min(left)
    copy = min(_spans(lambda: y.copy_(x))) - min(_spans(lambda: None))
    print(dims, rest, copy, flush=True)
    assert rest["in"] - rest["out"] < 0.5 * copy


@pytest.mark.parametrize("dims", [(32, 48, 40), (16, 15, 12, 10), (100, 96)])
def test_captured(gpu_lib, dims):
    import torch
    plan = fftrw.Plan(dims, 8, None)
    x = torch.randn(dims, dtype=torch.complex64, device="cuda")
    want = torch.empty_like(x)
    buf = x.clone()
    plan.exec_fwd(buf, buf)  # (code objects load outside the capture)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        plan.exec_fwd(buf, buf)
    for k in range(4):
        src = x * (k + 1)
        buf.copy_(src)
        graph.replay()
        torch.cuda.synchronize()
        plan.exec_fwd(src, want)
        torch.cuda.synchronize()
        assert torch.equal(buf, want), k
