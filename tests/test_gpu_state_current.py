"""The current planes behind a loaded state (needs an MI355X).

pic_load_state replaces the whole state in any phase, so nothing the context had
deposited before may stay: a state loaded over a deposit that no solve has read,
and a naive-charge state (its rho plane starts from the ion background) loaded
into a context that has loaded no particles, or others, step as the context it was
saved from.  Bit for bit with the deterministic deposit; the naive mode and
float64 atomics within the summation order, 1e-10."""

import numpy as np
import pytest
import torch

from paper_2410_18414_amd import pic, workloads
from pic_harness import make_gpu, rel

pytestmark = pytest.mark.gpu


def _load(ctx, w):
    pic.init_particles(ctx, torch.as_tensor(w["x"], device=ctx.device), torch.as_tensor(w["y"], device=ctx.device),
                       torch.as_tensor(np.ascontiguousarray(w["P"].T), device=ctx.device))


@pytest.mark.parametrize("dtype,scheme,flags,tol", [
    ("f32", "bdf", pic.FLAG_DETERMINISTIC, 0.0), ("f64", "dirk3", pic.FLAG_DETERMINISTIC | pic.FLAG_DIRK_SUBSTEP, 0.0),
    ("f64", "bdf", 0, 1e-10), ("f64", "bdf", pic.FLAG_NAIVE_RHO, 1e-10), ("f64", "dirk2", pic.FLAG_NAIVE_RHO, 1e-10)])
@pytest.mark.parametrize("trust", [False, True])
@pytest.mark.parametrize("nx,ny", [(24, 20), (40, 36), (9, 13)])
def test_load_leaves_no_deposit(gpu_lib, nx, ny, dtype, scheme, flags, tol, trust):
    w = workloads.cloud(nx=nx, ny=ny, ppc=3, seed=5, drift=0.2, vth=0.05)
    other = workloads.cloud(nx=nx, ny=ny, ppc=3, seed=6, drift=-0.3, vth=0.1)
    a = make_gpu(w, 2, scheme, dtype, flags=flags)
    pic.step(a, 3)
    saved = pic.save_state(a)
    pic.step(a, 2)
    want = pic.get_particles(a), pic.get_history(a)
    pic.deposit_current(a)             # in the planes when the state is loaded
    fresh = pic.Context(a.cfgs)
    others = pic.Context(a.cfgs)
    _load(others, other)
    pic.step(others, 1)
    pic.deposit_current(others)
    for ctx in (a, fresh, others):
        pic.load_state(ctx, saved, trust_header=trust)
        pic.step(ctx, 2)
        got = pic.get_particles(ctx), pic.get_history(ctx)
        for g, r in zip(got, want):
            if tol:
                assert rel(g.cpu().numpy(), r.cpu().numpy()) <= tol
            else:
                assert torch.equal(g, r)
        ctx.close()
