"""The autotuner against the batch it tunes: a cache never makes a batch slower,
and what the file says is what runs."""
import json
import math

import numpy as np
import pytest

from oracle import dft, orders
from paper_1302_6189_amd import fftrw, inputs
from tests.gpu_util import empty_dev, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tuned(gpu_lib, tmp_path_factory):
    items = inputs.batch_items(256, seed=5)
    cache = str(tmp_path_factory.mktemp("tune") / "tune.json")
    fftrw.fft_autotune(items, cache)
    return items, cache


def _times(items, flags, caches, n=4):
    import torch
    sizes = [math.prod(d) for d, _ in items]
    x = torch.zeros(sum(sizes), dtype=torch.complex64, device="cuda")
    y = torch.empty_like(x)
    ins, outs = list(x.split(sizes)), list(y.split(sizes))
    batches = [fftrw.Batch(items, flags=flags, tune_cache=c) for c in caches]
    best = [math.inf] * len(caches)
    for _ in range(n):
        for k, b in enumerate(batches):
            b.exec_fwd(ins, outs)
            e0, e1 = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            e0.record()
            for _ in range(4):
                b.exec_fwd(ins, outs)
            e1.record()
            torch.cuda.synchronize()
            best[k] = min(best[k], e0.elapsed_time(e1) / 4)
    return best


@pytest.mark.parametrize("flags", [0, fftrw.FLAG_BATCH_NO_FUSE, fftrw.FLAG_LEAVE_PERMUTED])
def test_no_slower(tuned, flags):
    # two runs of one batch differ by less than 1%
    items, cache = tuned
    plain, with_cache = _times(items, flags, [None, cache])
    print(flags, f"untuned {plain:.3f} ms, tuned {with_cache:.3f} ms", flush=True)
    assert with_cache < 1.01 * plain


def test_lists_run_as_stored(gpu_lib, tmp_path):
    # every list the kernels accept, 6 among the radices and 16 as 4 x 4, in the
    # fused unit and the row blocks; a file without the radices it was timed
    # with keeps the built-in order where its list is the old built-in one
    items = [((96, 60, 36), 5), ((16, 48, 12), 3)]
    xs = [inputs.uniform(d, 31 + i, np.complex64) for i, (d, _) in enumerate(items)]
    cache = str(tmp_path / "tune.json")
    fftrw.fft_autotune(items, cache)
    with open(cache) as f:
        rec = json.load(f)
    assert rec["radices"] == [2, 3, 4, 5, 6, 8]
    lists = {96: [6, 16], 60: [2, 6, 5], 36: [6, 6], 16: [16], 48: [3, 16], 12: [2, 6]}
    rec["tiles"] = []
    rec["rows"] = [dict(r, radix=lists[r["n"]]) for r in rec["rows"]]
    rec["fused"] = [dict(r, radix=lists[r["n"]]) for r in rec["fused"]]

    def run(flags, data):
        with open(cache, "w") as f:
            json.dump(data, f)
        b = fftrw.Batch(items, flags=flags, tune_cache=cache)
        ins, outs = [to_dev(x) for x in xs], [empty_dev(x.shape, np.complex64) for x in xs]
        b.exec_fwd(ins, outs)
        assert b.stats()["error"] == 0
        return [to_host(o) for o in outs]

    plain = run(0, dict(rec, device="other"))
    fused, separate = run(0, rec), run(fftrw.FLAG_BATCH_NO_FUSE, rec)
    for i, (dims, P) in enumerate(items):
        order = fftrw.fft_order_search(dims, P)["best_order"]
        assert dft.rel_l2(fused[i], dft.fftn_direct(xs[i], orders.fft_axis_sequence(order))) < 1e-5
        assert np.array_equal(fused[i], separate[i]), i
    assert not np.array_equal(fused[0], plain[0])
    old = {k: v for k, v in rec.items() if k != "radices"}
    old_lists = {96: [8, 4, 3], 60: [4, 3, 5], 36: [4, 3, 3], 16: [16], 48: [16, 3], 12: [4, 3]}
    for key in ("rows", "fused"):
        old[key] = [dict(r, radix=old_lists[r["n"]]) for r in rec[key]]
    for a, b in zip(run(0, old), plain):
        assert np.array_equal(a, b)
