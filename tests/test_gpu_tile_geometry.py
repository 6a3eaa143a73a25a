"""The compiled tile geometries on grids of any side (needs an MI355X).

A tile plan of the compiled shapes (16- or 8-cell tiles, slack 3) runs the
kernels whose window offsets are constants; any other slack runs the
runtime-geometry kernel.  With the deterministic deposit a run does not depend
on its window, so the two must agree bit for bit, on partial tiles, across
seams and sorts; and an ensemble that mixes powers of two with other sides
equals its instances run alone.
"""

import numpy as np
import pytest
import torch

from paper_2410_18414_amd import pic, workloads

pytestmark = pytest.mark.gpu


def _run(w, degree, dtype, slack, tile, flags=pic.FLAG_DETERMINISTIC, steps=13):
    ctx = _context([w], degree, dtype, slack, tile, flags)
    pic.step(ctx, steps)
    out = pic.get_particles(ctx), pic.get_history(ctx)
    ctx.close()
    return out


def _context(ws, degree, dtype, slack, tile, flags):
    cfgs = [pic.make_config(w["nx"], w["ny"], w["lx"], w["ly"], w["dt"], degree=degree, dtype=dtype, q=w["q"],
                            m=w["m"], max_particles=len(w["x"]), flags=flags, sort_interval=5, slack=slack,
                            tile_cells=tile) for w in ws]
    ctx = pic.Context(cfgs)
    for i, w in enumerate(ws):
        if len(ws) > 1:
            pic.select_instance(ctx, i)
        pic.init_particles(ctx, torch.as_tensor(w["x"]), torch.as_tensor(w["y"]),
                           torch.as_tensor(np.ascontiguousarray(w["P"].T)))
    return ctx


@pytest.mark.parametrize("nx,ny,tile,degree,dtype", [
    (37, 29, 16, 3, "f32"), (50, 27, 16, 3, "f64"), (17, 100, 16, 2, "f32"), (16, 18, 16, 5, "f64"),
    (9, 13, 8, 4, "f32"), (20, 11, 8, 1, "f64")])
def test_compiled_shape_equals_runtime_shape(gpu_lib, nx, ny, tile, degree, dtype):
    print("case", nx, ny, tile, degree, dtype, flush=True)
    w = workloads.weibel(nx=nx, ny=ny, ppc=6, seed=7, drift=0.3)
    a = _run(w, degree, dtype, 3, tile)
    b = _run(w, degree, dtype, 4, tile)
    assert torch.equal(a[0], b[0])
    assert torch.equal(a[1], b[1])


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_mixed_ensemble_equals_instances_alone(gpu_lib, dtype):
    ws = [workloads.weibel(nx=32, ny=32, ppc=6, seed=8), workloads.weibel(nx=37, ny=29, ppc=5, seed=9),
          workloads.weibel(nx=64, ny=16, ppc=3, seed=10)]
    ctx = _context(ws, 3, dtype, 0, 16, pic.FLAG_DETERMINISTIC)
    pic.step_batched(ctx, 13)
    for i, w in enumerate(ws):
        pic.select_instance(ctx, i)
        alone = _run(w, 3, dtype, 0, 16)
        assert torch.equal(pic.get_particles(ctx), alone[0]), i
        assert torch.equal(pic.get_history(ctx), alone[1]), i
    ctx.close()
