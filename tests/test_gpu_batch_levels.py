"""GPU checks of the batch's level sweep at the sizes where its claims and
waits change form: levels of one unit, of fewer units than work-groups, of
single claims only and of chunks with a remainder, of more tasks than the
LDS table holds, and levels of very different sizes in one launch."""
import numpy as np
import pytest

from paper_1302_6189_amd import fftrw, inputs
from tests.gpu_util import empty_dev, to_dev, to_host

pytestmark = pytest.mark.gpu

SETS = {
    "one unit": [((2, 3, 2), 1)],
    "few units": [((16, 20, 12), 5)] * 3,
    "single claims": [((48, 50, 45), 15), ((64, 64, 64), 16)],
    "chunks": [((128, 96, 100), 30), ((125, 120, 81), 9), ((160, 64, 135), 64)],
    "many tasks": [((4, 5, 6), 3), ((8, 9, 10), 7), ((3, 4, 2, 5), 4)] * 90,
    "uneven levels": [((2, 3, 2), 1), ((96, 100, 64), 20), ((6, 5, 8, 4, 3), 12), ((10, 9, 12, 8), 30)],
}


@pytest.mark.parametrize("name", list(SETS))
def test_level_sweep(gpu_lib, name):
    items = SETS[name]
    xs = [inputs.uniform(d, 700 + i, np.complex64) for i, (d, _) in enumerate(items)]
    refs = [np.fft.fftn(x.astype(np.complex128)) for x in xs]
    b = fftrw.Batch(items, flags=fftrw.FLAG_COUNT_MOVED)
    ins = [to_dev(x) for x in xs]
    outs = [empty_dev(x.shape, np.complex64) for x in xs]
    back = [empty_dev(x.shape, np.complex64) for x in xs]
    for _ in range(3):
        for o in outs:
            o.zero_()
        b.exec_fwd(ins, outs)
        st = b.stats()
        assert st["error"] == 0 and st["moved"] == st["analytic"]
        for i, o in enumerate(outs):
            err = np.linalg.norm(to_host(o) - refs[i]) / np.linalg.norm(refs[i])
            assert err < 1e-5, (i, items[i], err)
    b.exec_inv(outs, back)
    for i, x in enumerate(xs):
        assert np.linalg.norm(to_host(back[i]) - x) / np.linalg.norm(x) < 1e-5, (i, items[i])
    assert b.stats()["error"] == 0
