"""Split-precision plans with an axis the matrix cores do not take: every step
fuses with its transpose unless that axis is a power of two above 512."""
import math

import pytest

from oracle import dft, orders
from paper_1302_6189_amd import fftrw, inputs
from tests.gpu_util import empty_dev, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,P,oidx", [((256, 600, 256), 7, 3), ((256, 1500, 16), 64, 1), ((12, 512, 1000), 5, 6),
                                         ((256, 625), 9, 0), ((3750, 256), 4, 0), ((5, 2187, 256), 30, 2)])
@pytest.mark.parametrize("prec", [fftrw.PREC_SPLIT_F16, fftrw.PREC_SPLIT_BF16X3])
def test_long_axis(gpu_lib, dims, P, oidx, prec):
    import numpy as np
    order = fftrw.fft_order_at(len(dims), oidx)
    x = inputs.uniform(dims, 44, np.complex64)
    xd, a, b = to_dev(x), empty_dev(dims, np.complex64), empty_dev(dims, np.complex64)
    fused = fftrw.Plan(dims, P, order, precision=prec, flags=fftrw.FLAG_COUNT_MOVED)
    plain = fftrw.Plan(dims, P, order, precision=prec, flags=fftrw.FLAG_COUNT_MOVED | fftrw.FLAG_SEPARATE)
    desc = fused.describe()[1]
    assert desc.startswith("fused|") and "mfma:" in desc, desc
    for run in ("exec_fwd", "exec_inv"):
        getattr(fused, run)(xd, a)
        getattr(plain, run)(xd, b)
        assert np.array_equal(to_host(a), to_host(b)), run
        analytic, moved = fused.stats()
        assert moved == analytic
        wd = to_dev(x)
        getattr(fused, run)(wd, wd)
        assert np.array_equal(to_host(wd), to_host(a)), run
    if math.prod(dims) <= 1 << 23:
        fused.exec_fwd(xd, a)
        assert dft.rel_l2(to_host(a), dft.fftn_direct(x, orders.fft_axis_sequence(order))) < 1e-5
