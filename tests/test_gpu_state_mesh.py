"""The mesh fields of a state saved in phase SOLVED (needs an MI355X).

A state saved after deposit_current and field_solve is loaded again after the
context has solved something else, and into a context that has solved nothing:
PIC_FIELD_MESH is the mesh the state was saved with, bit for bit (the export
copies the same values, or transforms the same spectra), and looking at it
leaves what the particles gather as it is (gather_push gives the same particles,
bit for bit: a particle's push is a sum of its own).  A solve in one launch
(32 x 24), one in three (40 x 36), alone and as an ensemble."""

import numpy as np
import pytest
import torch

from paper_2410_18414_amd import pic, workloads

pytestmark = pytest.mark.gpu


def _context(sides, dtype, scheme, load=True):
    ws = [workloads.cloud(nx=nx, ny=ny, ppc=3, seed=9 + i, drift=0.2, vth=0.05) for i, (nx, ny) in enumerate(sides)]
    ctx = pic.Context([pic.make_config(w["nx"], w["ny"], w["lx"], w["ly"], w["dt"], degree=2, scheme=scheme, dtype=dtype,
                                       q=w["q"], m=w["m"], max_particles=len(w["x"])) for w in ws])
    for i, w in enumerate(ws if load else []):
        pic.select_instance(ctx, i)
        pic.init_particles(ctx, torch.as_tensor(w["x"], device=ctx.device), torch.as_tensor(w["y"], device=ctx.device),
                           torch.as_tensor(np.ascontiguousarray(w["P"].T), device=ctx.device))
    return ctx


def _every(ctx, get):
    out = []
    for i in range(pic.instance_count(ctx)):
        pic.select_instance(ctx, i)
        out.append(get(ctx).clone())
    return out


@pytest.mark.parametrize("sides", [[(32, 24)], [(40, 36)], [(32, 24), (9, 8)], [(32, 24), (40, 36)]],
                         ids=["small", "large", "small-ensemble", "ensemble"])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("scheme", ["bdf", "cdf2"])
def test_loaded_mesh_is_the_saved_one(gpu_lib, sides, dtype, scheme):
    a = _context(sides, dtype, scheme)
    pic.step(a, 3)
    pic.deposit_current(a)
    pic.field_solve(a)
    saved = pic.save_state(a)
    mesh = _every(a, lambda c: pic.get_field(c, pic.FIELD_MESH))
    assert all(float(m.abs().max()) > 0 for m in mesh)
    pic.gather_push(a)
    parts = _every(a, pic.get_particles)
    pic.step(a, 4)
    pic.deposit_current(a)
    pic.field_solve(a)  # another solve's fields in the context
    for ctx in (a, _context(sides, dtype, scheme, load=False), _context(sides, dtype, scheme)):
        pic.load_state(ctx, saved)
        for m, want in zip(_every(ctx, lambda c: pic.get_field(c, pic.FIELD_MESH)), mesh):
            assert torch.equal(m, want)
        pic.gather_push(ctx)
        for p, want in zip(_every(ctx, pic.get_particles), parts):
            assert torch.equal(p, want)
        pic.step(ctx, 2)
        ctx.close()
