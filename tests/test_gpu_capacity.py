"""Contexts with room for more particles than are loaded (needs an MI355X).

The chunks of the sorted passes are planned for the particles loaded, within the
chunk list that the capacity gives.  With the deterministic deposit a run with
spare capacity keeps the bits of one without, whatever was loaded before, clustered
in one tile (the most chunks of a tile) or not, alone and in an ensemble, and from
a state of another count.

And the rate: float64 particles in a sixteenth of the capacity step no slower than
in a context of their number (it was 1.9 times as slow with chunks planned for the
capacity; it is 1.00 now, bounded here by 1.25)."""

import numpy as np
import pytest
import torch

from paper_2410_18414_amd import pic, workloads

pytestmark = pytest.mark.gpu


def _load(ctx, w, i=None):
    if i is not None:
        pic.select_instance(ctx, i)
    pic.init_particles(ctx, torch.as_tensor(w["x"], device=ctx.device), torch.as_tensor(w["y"], device=ctx.device),
                       torch.as_tensor(np.ascontiguousarray(w["P"].T), device=ctx.device))


def _config(w, dtype, capacity, flags=pic.FLAG_DETERMINISTIC):
    return pic.make_config(w["nx"], w["ny"], w["lx"], w["ly"], w["dt"], degree=3, dtype=dtype, q=w["q"], m=w["m"],
                           max_particles=capacity, flags=flags)


def _result(ctx):
    return pic.get_particles(ctx), pic.get_history(ctx)


def _clustered(w):
    return dict(w, x=(2 + 0.5 * w["x"] / w["lx"]) * w["lx"] / w["nx"], y=(2 + 0.5 * w["y"] / w["ly"]) * w["ly"] / w["ny"])


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("spare", [1.5, 8, 100])
@pytest.mark.parametrize("clustered", [False, True])
def test_bits_of_the_exact_capacity(gpu_lib, dtype, spare, clustered):
    w = workloads.weibel(nx=40, ny=32, ppc=8, seed=41)
    small = {k: (w[k][:700] if k in ("x", "y", "P") else w[k]) for k in w}
    if clustered:
        w = _clustered(w)
    n = len(w["x"])
    # the capacity sets the deterministic scale (a power of two): the same step of it for both
    a = pic.Context(_config(w, dtype, int(spare * n)))
    _load(a, w)
    pic.step(a, 8)
    want = _result(a)
    b = pic.Context(_config(w, dtype, int(spare * n)))
    _load(b, small)                      # planned for 700
    pic.step(b, 3)
    few = pic.save_state(b)
    _load(b, w)                          # and for n
    pic.step(b, 5)
    saved = pic.save_state(b)
    pic.load_state(b, few)
    pic.step(b, 2)
    pic.load_state(b, saved)
    pic.step(b, 3)
    for g, r in zip(_result(b), want):
        assert torch.equal(g, r)
    if dtype == "f32":                   # float32: one scale for every capacity below 8M
        c = pic.Context(_config(w, dtype, n))
        _load(c, w)
        pic.step(c, 8)
        for g, r in zip(_result(c), want):
            assert torch.equal(g, r)


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_ensemble_with_spare_capacity(gpu_lib, dtype):
    ws = [workloads.weibel(nx=nx, ny=ny, ppc=ppc, seed=50 + i)
          for i, (nx, ny, ppc) in enumerate([(32, 32, 9), (40, 24, 30), (16, 16, 1), (64, 48, 4)])]
    ws[1] = _clustered(ws[1])
    caps = [len(w["x"]) * k for w, k in zip(ws, (1, 20, 300, 3))]
    e = pic.Context([_config(w, dtype, c) for w, c in zip(ws, caps)])
    for i in (2, 0, 3, 1):
        _load(e, ws[i], i)
    pic.step_batched(e, 7)
    for i, (w, c) in enumerate(zip(ws, caps)):
        a = pic.Context(_config(w, dtype, c))
        _load(a, w)
        pic.step(a, 7)
        pic.select_instance(e, i)
        for g, r in zip(_result(e), _result(a)):
            assert torch.equal(g, r), i


def test_spare_capacity_costs_no_time(gpu_lib):
    w = workloads.weibel(nx=64, ny=64, ppc=16, seed=61)
    times = []
    for spare in (16, 1):
        ctx = pic.Context(_config(w, "f64", spare * len(w["x"]), flags=0))
        _load(ctx, w)
        pic.step(ctx, pic.graph_period(ctx) + 1)
        best = np.inf
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(ctx.stream)
            pic.step(ctx, 54)
            b.record(ctx.stream)
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
        ctx.close()
    print("ms", times)
    assert times[0] <= 1.25 * times[1]
