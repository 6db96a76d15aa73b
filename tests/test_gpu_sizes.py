"""Plans at the array sizes where the kernels change how they reach memory
(streaming or cached loads and stores, units renumbered over the XCDs), at
shapes that are no powers of two: fused against separate kernels bit for bit,
staged against fused, and sampled outputs against FP64 sums over the input."""
import math

import pytest

from paper_1302_6189_amd import fftrw

pytestmark = pytest.mark.gpu


def _sampled(x, points, sign):
    """Eq. (2) at the given outputs, every sum in FP64, the last axis first."""
    import torch
    out = []
    for k in points:
        v = x
        for r in range(x.dim() - 1, -1, -1):
            n = x.shape[r]
            j = torch.arange(n, device=x.device, dtype=torch.float64)
            w = torch.polar(torch.ones_like(j), sign * 2 * math.pi * torch.remainder(j * k[r], n) / n)
            rows = v.reshape(-1, n)
            v = torch.cat([(part.to(torch.complex128) * w).sum(1) for part in rows.split(max(1, (1 << 24) // n))])
        out.append(complex(v.item()))
    return out


# below and above 20, 64 and 256 MB and 1 GB; whole lines, whole axes and parts
# of lines per run; rows in registers and through LDS; one and several slices
# per group
CASES = [((96, 100, 90), 30, 7, False), ((100, 120, 300), 8, 1, False), ((125, 135, 150), 64, 4, True),
         ((45, 50, 60, 75), 100, 500, False), ((240, 240, 240), 48, 3, False), ((12, 15, 20, 50, 60), 1000, 4000000, False),
         ((320, 300, 375), 100, 6, False), ((480, 540, 512), 77, 2, False), ((1215, 1125, 100), 9, 5, False)]


@pytest.mark.parametrize("dims,P,oidx,double", CASES)
def test_fused(gpu_lib, dims, P, oidx, double):
    import torch
    tdt, dtype = (torch.complex128, fftrw.C128) if double else (torch.complex64, fftrw.C64)
    order = fftrw.fft_order_at(len(dims), oidx)
    gen = torch.Generator(device="cuda").manual_seed(oidx)
    x = torch.empty(dims, dtype=tdt, device="cuda")
    torch.view_as_real(x).uniform_(-1, 1, generator=gen)
    y, z = torch.empty_like(x), torch.empty_like(x)
    fused = fftrw.Plan(dims, P, order, dtype=dtype, flags=fftrw.FLAG_COUNT_MOVED)
    plain = fftrw.Plan(dims, P, order, dtype=dtype, flags=fftrw.FLAG_COUNT_MOVED | fftrw.FLAG_SEPARATE)
    assert fused.describe()[1].startswith("fused|")
    for run in ("exec_inv", "exec_fwd"):
        getattr(fused, run)(x, y)
        getattr(plain, run)(x, z)
        assert torch.equal(y, z), run
        analytic, moved = fused.stats()
        assert moved == analytic and plain.stats()[1] == analytic
        z.copy_(x)
        getattr(fused, run)(z, z)
        assert torch.equal(y, z), (run, "in place")
    points = [tuple((n * f).__floor__() for n, f in zip(dims, fs)) for fs in
              ((0, 0, 0, 0, 0), (.31, .77, .5, .9, .2), (.99, .01, .63, .4, .8), (.5, .999, .12, .7, .6))]
    rms = math.sqrt(math.prod(dims) * 2 / 3)
    for k, want in zip(points, _sampled(x, points, -1)):
        # single outputs err by a few times the relative L2 error (about 2e-7, 5e-16)
        assert abs(complex(y[k].item()) - want) < (1e-14 if double else 3e-6) * rms, k


@pytest.mark.parametrize("dims,P,oidx,double", [((200, 200, 200), 64, 0, False), ((320, 320, 320), 100, 3, False),
                                                ((360, 400, 384), 250, 1, False), ((100, 160, 128), 40, 5, True),
                                                ((36, 40, 45, 48), 60, 300, False)])
def test_staged(gpu_lib, dims, P, oidx, double):
    import torch
    tdt, dtype = (torch.complex128, fftrw.C128) if double else (torch.complex64, fftrw.C64)
    order = fftrw.fft_order_at(len(dims), oidx)
    gen = torch.Generator(device="cuda").manual_seed(oidx + 1)
    x = torch.empty(dims, dtype=tdt, device="cuda")
    torch.view_as_real(x).uniform_(-1, 1, generator=gen)
    y, z = torch.empty_like(x), torch.empty_like(x)
    staged = fftrw.Plan(dims, P, order, dtype=dtype, flags=fftrw.FLAG_STAGED)
    fused = fftrw.Plan(dims, P, order, dtype=dtype)
    for run in ("exec_fwd", "exec_inv"):
        getattr(staged, run)(x, y)
        getattr(fused, run)(x, z)
        assert torch.equal(y, z), run
        analytic, moved = staged.stats()
        assert moved == analytic
