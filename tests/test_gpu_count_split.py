"""Owner counts of fused plans whose rows are split over processes (level M):
exact for row lengths below, at and above the parts a row is counted in, and no
dearer than in the separate form, whose transposes count tile by tile."""
import math

import pytest

from paper_1302_6189_amd import fftrw

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,P", [((4096, 3), 4097), ((3, 4096), 12288), ((2048, 3000), 877714), ((5, 3, 2), 30),
                                    ((64, 60, 45), 5000), ((2, 125, 3, 96), 71999), ((2, 2, 2, 2, 2), 32),
                                    ((1, 48, 1, 36), 1728), ((32, 32, 32, 32, 2), 70000)])
@pytest.mark.parametrize("own", [0, fftrw.FLAG_OWN_MATCHED])
def test_counts(gpu_lib, dims, P, own):
    import torch
    if own and math.prod(dims) > 100000:
        pytest.skip("the matching of so many ranges takes the host long")
    order = fftrw.fft_order_at(len(dims), fftrw.fft_order_count(len(dims)) - 1)
    x = torch.zeros(math.prod(dims), dtype=torch.complex64, device="cuda")
    y = torch.empty_like(x)
    for extra in (0, fftrw.FLAG_LEAVE_PERMUTED):
        plan = fftrw.Plan(dims, P, order, flags=fftrw.FLAG_COUNT_MOVED | own | extra)
        sep = fftrw.Plan(dims, P, order, flags=fftrw.FLAG_COUNT_MOVED | own | extra | fftrw.FLAG_SEPARATE)
        for _ in range(2):  # the second exec finds the first one's counts
            plan.exec_fwd(x, y)
            sep.exec_fwd(x, y)
            analytic, moved = plan.stats()
            assert moved == sep.stats()[1]
            assert moved[:-1] == analytic[:-1] and (extra or moved == analytic)


def test_time(gpu_lib):
    # 6,144,000 processes, one per point: the fused form makes half the passes
    # of the separate one over memory, so with its counts it takes no longer
    import torch
    dims = (2048, 3000)
    T = math.prod(dims)
    x = torch.zeros(T, dtype=torch.complex64, device="cuda")
    y = torch.empty_like(x)
    best = {}
    for name, flags in (("fused", 0), ("separate", fftrw.FLAG_SEPARATE)):
        plan = fftrw.Plan(dims, T, fftrw.fft_order_at(2, 0), flags=fftrw.FLAG_COUNT_MOVED | flags)
        plan.exec_fwd(x, y)
        best[name] = math.inf
        for _ in range(5):
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            e0.record()
            for _ in range(5):
                plan.exec_fwd(x, y)
            e1.record()
            torch.cuda.synchronize()
            best[name] = min(best[name], e0.elapsed_time(e1) / 5)
    print(best, flush=True)
    assert best["fused"] < 1.25 * best["separate"]
