"""Rounding errors of the row kernels against an 80-bit transform, at lengths
whose twiddles and butterfly constants once cost accuracy.  The bounds lie
between an emulation of the kernels (complex64: butterflies and twiddles as
they are) or of their twiddles (complex128) with and without the loss."""
import numpy as np
import pytest
import scipy.fft

from paper_1302_6189_amd import fftrw
from tests.gpu_util import empty_dev, to_dev, to_host

pytestmark = pytest.mark.gpu


def _error(n, dtype):
    rows = max(27, 32768 // n)
    rows = next(r for r in range(rows, 0, -1) if _smooth(r))
    plan = fftrw.Plan((rows, n), 1, fftrw.fft_order_at(2, 0), dtype=fftrw.C64 if dtype == np.complex64 else fftrw.C128,
                      flags=fftrw.FLAG_SEPARATE)
    sq = []
    for seed in range(6):
        g = np.random.default_rng(seed + 100 * n)
        x = (g.standard_normal((rows, n)) + 1j * g.standard_normal((rows, n))).astype(dtype)
        yd = empty_dev(x.shape, dtype)
        plan.exec_fft_step(0, -1, to_dev(x), yd)
        ref = scipy.fft.fft(x.astype(np.clongdouble), axis=1)
        d = (to_host(yd) - ref).astype(np.complex128)
        sq.append(np.linalg.norm(d) ** 2 / np.linalg.norm(ref.astype(np.complex128)) ** 2)
    return float(np.sqrt(np.mean(sq)))


def _smooth(n):
    for p in (2, 3, 5):
        while n % p == 0:
            n //= p
    return n == 1


# complex64 with rounded constants 0.963, 1.230, 1.357 and 1.210e-7, in two
# parts 0.918, 1.168, 1.290 and 1.177e-7; complex128 with rounded angles
# 2.17e-16 and 2.22e-16, exact 1.94e-16 and about 2.0e-16
@pytest.mark.parametrize("n,dtype,bound", [(81, np.complex64, 0.945e-7), (729, np.complex64, 1.20e-7),
                                           (2187, np.complex64, 1.32e-7), (4096, np.complex64, 1.195e-7),
                                           (81, np.complex128, 2.06e-16), (320, np.complex128, 2.11e-16)])
def test_rows(gpu_lib, n, dtype, bound):
    err = _error(n, dtype)
    print(n, np.dtype(dtype).name, f"{err:.4e}", flush=True)
    assert err < bound
