"""Rows alone (a step by itself, plans of separate kernels): their kernels by
array size, row by row, as one block and straight from HBM, give the same bits;
short odd rows keep up with the even ones beside them."""
import math

import numpy as np
import pytest

from oracle import dft
from paper_1302_6189_amd import fftrw, inputs
from tests.gpu_util import to_dev, to_host

pytestmark = pytest.mark.gpu


def _step(dims, dtype, x, y, direction):
    plan = fftrw.Plan(dims, 1, fftrw.fft_order_at(len(dims), 0), dtype=dtype, flags=fftrw.FLAG_SEPARATE)
    plan.exec_fft_step(0, direction, x, y)
    plan.destroy()


# lengths of one lane, of lanes in pairs and not, of whole lines and not, odd
# and even, of one and several rows per group
@pytest.mark.parametrize("n", [2, 3, 4, 9, 15, 16, 20, 25, 27, 32, 48, 60, 64, 75, 90, 96, 100, 125, 128, 135, 250, 375,
                               625, 729, 1000, 1125, 2048, 2187, 3125, 4050, 4096])
@pytest.mark.parametrize("double", [False, True])
def test_sizes_agree(gpu_lib, n, double):
    import torch
    if double and n > 2048:
        pytest.skip("complex128 kernels end at 2048 points")
    dtype = fftrw.C128 if double else fftrw.C64
    tdt = torch.complex128 if double else torch.complex64
    esz = 16 if double else 8
    # a base of at most 1 MB, and arrays of it just above 4, 24 and 256 MB, the
    # last group of rows ragged
    rows = max(m for m in (27, 45, 81, 135, 243, 405, 729, 1215, 2187, 3645) if m == 27 or m * n * esz <= 1 << 20)
    x = inputs.gaussian((rows, n), n, np.complex128 if double else np.complex64)
    xd = to_dev(x)
    for direction in (-1, 1):
        want = torch.empty_like(xd)
        _step((rows, n), dtype, xd, want, direction)
        assert dft.rel_l2(to_host(want), dft.fft1d_rows(x, sign=direction)) < (1e-12 if double else 1e-5)
        for mb in (5, 30, 270):
            most = mb * (1 << 20) // (rows * n * esz) + 1
            a = min(m for m in range(most, 4 * most) if _smooth(m))
            dims = (a, rows, n) if a <= 4096 else (a // 64 + 1, 64, rows, n)
            while len(dims) == 4 and not _smooth(dims[0]):
                dims = (dims[0] + 1, *dims[1:])
            reps = math.prod(dims[:-2])
            big = xd.repeat(reps, 1)
            out = torch.empty(reps * rows, n, dtype=tdt, device="cuda")
            _step(dims, dtype, big, out, direction)
            assert bool((out.view(reps, rows, n) == want).all()), (mb, direction)
            _step(dims, dtype, big, big, direction)
            assert torch.equal(big, out), (mb, direction, "in place")
            del big, out


# rows of one lane that fit one group, whole and ragged, and one row more
@pytest.mark.parametrize("rows", [1, 27, 250, 256, 270])
@pytest.mark.parametrize("n", [2, 4, 9, 16])
def test_one_group(gpu_lib, rows, n):
    import torch
    x = inputs.gaussian((rows, n), rows * n, np.complex64)
    xd = to_dev(x)
    out = torch.empty_like(xd)
    _step((rows, n), fftrw.C64, xd, out, -1)
    assert dft.rel_l2(to_host(out), dft.fft1d_rows(x, sign=-1)) < 1e-5


def _smooth(n):
    for p in (2, 3, 5):
        while n % p == 0:
            n //= p
    return n == 1


def test_odd_rows_keep_up(gpu_lib):
    # 131 MB of 125-point rows and of 128-point rows: the same bytes, to 0.1%
    import torch
    best = {}
    x = torch.zeros(4096 * 4096, dtype=torch.complex64, device="cuda")
    y = torch.empty_like(x)
    plans = {d: fftrw.Plan(d, 1, fftrw.fft_order_at(3, 0), flags=fftrw.FLAG_SEPARATE)
             for d in ((32, 4096, 125), (32, 4000, 128))}
    for _ in range(5):
        for d, plan in plans.items():
            plan.exec_fft_step(0, -1, x, y)
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            e0.record()
            for _ in range(20):
                plan.exec_fft_step(0, -1, x, y)
            e1.record()
            torch.cuda.synchronize()
            best[d[2]] = min(best.get(d[2], math.inf), e0.elapsed_time(e1) / 20)
    print(best, flush=True)
    assert best[125] < 1.35 * best[128]
