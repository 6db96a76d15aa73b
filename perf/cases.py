"""Timing cases of the transforms, through the package's public entry points.

A case is one of four calls a program makes:

* ``plan``     a ``fftrw.Plan`` kept by the program and executed (forward,
               inverse, or one of each; the pair also in place)
* ``staged``   the same with the explicit pack -> exchange -> unpack transposes
* ``noalloc``  ``fftrw.fft_exec_noalloc``, which plans on every call
* ``batch``    a ``fftrw.Batch`` of many uneven transforms in one launch

Sizes, process counts, orders and input distributions are those of the
benchmark, the order study and the tests: powers of two and other
2^a 3^b 5^c sizes, 2-D to 5-D, complex64 and complex128.  Inputs are drawn on
the GPU from the seed alone.
"""
from __future__ import annotations

import math

import torch

from paper_1302_6189_amd import fftrw, inputs

SMOOTH = sorted({2 ** a * 3 ** b * 5 ** c for a in range(13) for b in range(8) for c in range(6)
                 if 2 ** a * 3 ** b * 5 ** c <= 4096})
PRECISION = {"native": fftrw.PREC_NATIVE, "split_f16": fftrw.PREC_SPLIT_F16, "split_bf16": fftrw.PREC_SPLIT_BF16,
             "split_bf16x3": fftrw.PREC_SPLIT_BF16X3}


def _case(call, dims, P, dtype="c64", direction="fwd", precision="native", count=False, inplace=False,
          permuted=False, order=-1, values="uniform"):
    return {"call": call, "dims": "x".join(map(str, dims)), "P": P, "dtype": dtype, "direction": direction,
            "precision": precision, "count": count, "inplace": inplace, "permuted": permuted, "order": order,
            "values": values}


def listed():
    named = {
        # the smallest configuration of the library's own checks, FP64 data: launches and latency
        "cube32_c128": _case("plan", (32, 32, 32), 4, dtype="c128", count=True),
        # a serving loop that may not allocate: a small transform planned and run in one call
        "noalloc_cube64": _case("noalloc", (64, 64, 64), 16, order=0),
        # odd sizes in FP64, rows of 3s and 5s only, odd runs on every side
        "odd_75x81x125_c128": _case("plan", (75, 81, 125), 30, dtype="c128", direction="inv", values="gaussian"),
        # an ordinary grid of a solver: even sizes that are no powers of two
        "grid_192x160x144": _case("plan", (192, 160, 144), 48, direction="inv"),
        # the order study's 4-D and 5-D grids, process counts that do and do not divide
        "hyper_64p4": _case("plan", (64, 64, 64, 64), 256, values="gaussian"),
        "hyper_32p4x16": _case("plan", (32, 32, 32, 32, 16), 1000, direction="inv", count=True, values="gaussian"),
        # a 2-D field of long rows, filtered in place: forward, then inverse, in its own buffer
        "field_2048x3000_inplace": _case("plan", (2048, 3000), 64, direction="both", inplace=True),
        # 256-point rows on the matrix cores
        "cube256_split_f16": _case("plan", (256, 256, 256), 64, precision="split_f16", values="log_uniform"),
        # the distributed transposes executed as messages between process regions
        "staged_cube256": _case("staged", (256, 256, 256), 512),
        # a large grid that is no power of two
        "cube480": _case("plan", (480, 480, 480), 100),
        # 256 uneven 3-D to 5-D transforms in one launch, owner changes counted
        "batch256": {"call": "batch", "items": 256, "items_seed": 5, "direction": "fwd", "count": True},
        # the benchmark's step: forward and inverse of the largest grid, owner changes counted
        "cube512_pair": _case("plan", (512, 512, 512), 4096, direction="both", count=True),
    }
    return [dict(c, name=n) for n, c in named.items()]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _sizes(rng, M, lo, hi, most):
    """M smooth sizes of [lo, hi], spread over their logarithm, at most `most` points and at least 8^M."""
    while True:
        dims = tuple(min((s for s in SMOOTH if lo <= s <= hi), key=lambda s, t=_log_int(rng, lo, hi): abs(s - t))
                     for _ in range(M))
        if 8 ** M <= math.prod(dims) <= most:
            return dims


def draw(rng):
    call = rng.choice(["plan"] * 10 + ["staged", "staged", "noalloc", "batch"])
    direction = rng.choice(["fwd", "fwd", "inv", "both"])
    values = rng.choice(["uniform", "gaussian", "log_uniform"])
    dtype = rng.choice(["c64", "c64", "c128"])
    if call == "batch":
        return {"call": "batch", "items": _log_int(rng, 8, 256), "items_seed": rng.randrange(6, 1 << 16),
                "direction": rng.choice(["fwd", "inv"]), "count": rng.random() < 0.5}
    most = (1 << 26) // (1 if dtype == "c64" else 2)
    if call == "noalloc":
        dims = _sizes(rng, rng.choice([2, 3, 3, 4]), 8, 256, (1 << 23) // (1 if dtype == "c64" else 2))
        return _case("noalloc", dims, _log_int(rng, 1, 64), dtype, rng.choice(["fwd", "inv"]), order=0, values=values)
    if call == "staged":
        dims = _sizes(rng, 3, 16, 512, most // 2)
        return _case("staged", dims, _log_int(rng, 2, min(512, math.prod(dims) // max(dims))), dtype, direction,
                     values=values)
    M = rng.choice([2, 3, 3, 3, 4, 5])
    if M == 2:
        dims = _sizes(rng, 2, 32, 4096 if dtype == "c64" else 2048, most)
    else:
        dims = _sizes(rng, M, 8, (0, 0, 0, 512, 192, 64)[M], most)
    if rng.random() < 0.4:  # powers of two as often as they are used
        dims = tuple(1 << round(math.log2(n)) for n in dims)
        while math.prod(dims) > most:
            dims = tuple(max(8, n // 2) for n in dims)
    precision = "native"
    if M == 3 and dtype == "c64" and rng.random() < 0.25:
        precision = rng.choice(["split_f16", "split_bf16x3"])
        dims = (rng.choice([256, 512]), rng.choice([256, 512]), dims[2])
        if math.prod(dims) > most:
            dims = (dims[0], dims[1], 128)
    inplace = direction == "both" and rng.random() < 0.4
    return _case("plan", dims, _log_int(rng, 1, min(1000, math.prod(dims) // max(dims))), dtype, direction, precision,
                 count=rng.random() < 0.4, inplace=inplace, permuted=direction == "fwd" and rng.random() < 0.2,
                 order=rng.randrange(fftrw.fft_order_count(M)) if rng.random() < 0.3 else -1, values=values)


def _dims(case):
    return tuple(int(n) for n in case["dims"].split("x"))


def _fill(out, values, gen):
    """Complex values into `out`: re, im U[-1, 1), N(0, 1), or of log-uniform magnitude 1e-6..1 with random signs."""
    r = torch.view_as_real(out)
    if values == "gaussian":
        r.normal_(generator=gen)
    elif values == "uniform":
        r.uniform_(-1.0, 1.0, generator=gen)
    else:
        sign = torch.empty_like(r).uniform_(-1.0, 1.0, generator=gen).sign_()
        r.uniform_(-6.0, 0.0, generator=gen)
        torch.pow(10.0, r, out=r)
        r.mul_(sign)


def _order(case):
    """The case's transpose order: None (the plan's best), or a canonical index."""
    return None if case["order"] < 0 else fftrw.fft_order_at(len(_dims(case)), case["order"])


def _batch_items(case):
    return inputs.batch_items(case["items"], seed=case["items_seed"])


def _draw_inputs(case, seed, device="cuda"):
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    if case["call"] == "batch":
        x = torch.empty(sum(math.prod(d) for d, _ in _batch_items(case)), dtype=torch.complex64, device="cuda")
        _fill(x, "uniform", gen)
        return x
    dt = torch.complex64 if case["dtype"] == "c64" else torch.complex128
    x = torch.empty(_dims(case), dtype=dt, device="cuda")
    _fill(x, case["values"], gen)
    return x


def prepare(case, seed):
    x = _draw_inputs(case, seed)
    state = {"case": case, "x": x, "y": x if case.get("inplace") else torch.empty_like(x)}
    if case["call"] == "batch":
        items = _batch_items(case)
        state["plan"] = fftrw.Batch(items, flags=fftrw.FLAG_COUNT_MOVED if case["count"] else 0)
        sizes = [math.prod(d) for d, _ in items]
        state["ins"], state["outs"] = list(x.split(sizes)), list(state["y"].split(sizes))
        return state
    dims = _dims(case)
    dtype = fftrw.C64 if case["dtype"] == "c64" else fftrw.C128
    if case["call"] == "noalloc":
        state["args"] = (dims, case["P"], _order(case), -1 if case["direction"] == "fwd" else 1)
        state["dtype"] = dtype
        return state
    flags = (fftrw.FLAG_STAGED if case["call"] == "staged" else 0) | (fftrw.FLAG_COUNT_MOVED if case["count"] else 0) \
        | (fftrw.FLAG_LEAVE_PERMUTED if case["permuted"] else 0)
    state["plan"] = fftrw.Plan(dims, case["P"], _order(case), dtype=dtype, precision=PRECISION[case["precision"]],
                               flags=flags)
    if case["direction"] == "both":
        state["z"] = x if case["inplace"] else torch.empty_like(x)
    return state


def run(state):
    case, x, y = state["case"], state["x"], state["y"]
    if case["call"] == "batch":
        (state["plan"].exec_fwd if case["direction"] == "fwd" else state["plan"].exec_inv)(state["ins"], state["outs"])
        return y
    if case["call"] == "noalloc":
        fftrw.fft_exec_noalloc(*state["args"], x, y, dtype=state["dtype"])
        return y
    plan = state["plan"]
    if case["direction"] == "fwd":
        plan.exec_fwd(x, y)
        return y
    if case["direction"] == "inv":
        plan.exec_inv(x, y)
        return y
    z = state["z"]
    plan.exec_fwd(x, y)
    plan.exec_inv(y, z)
    return z if case["inplace"] else [y, z]


def work(case):
    if case["call"] == "batch":
        Ts, esz, calls = [math.prod(d) for d, _ in _batch_items(case)], 8, 1
    else:
        Ts, esz = [math.prod(_dims(case))], 8 if case["dtype"] == "c64" else 16
        calls = 2 if case["direction"] == "both" else 1
    return {"bytes": calls * sum(2 * T * esz for T in Ts), "flops": calls * sum(5 * T * math.log2(T) for T in Ts)}


def exact(case, seed):
    x = _draw_inputs(case, seed).cpu()
    if case["call"] == "batch":
        f = torch.fft.fftn if case["direction"] == "fwd" else torch.fft.ifftn
        items = _batch_items(case)
        parts = x.split([math.prod(d) for d, _ in items])
        return torch.cat([f(p.to(torch.complex128).reshape(d)).reshape(-1) for p, (d, _) in zip(parts, items)])
    x = x.to(torch.complex128)
    if case["direction"] == "both":
        return x if case["inplace"] else [torch.fft.fftn(x), x]
    if case["direction"] == "inv":
        return torch.fft.ifftn(x)
    y = torch.fft.fftn(x)
    if case["permuted"]:  # the output stays in the order's last layout
        dims, order = _dims(case), _order(case)
        if order is None:
            order = fftrw.fft_order_search(dims, case["P"])["best_order"]
        y = y.permute(order[-1]).contiguous().reshape(dims)
    return y
