"""The push adjoint's scatter by matrix instructions (needs an MI355X): the
gradient of the field energy by the sorted passes -- compiled and runtime tile
shapes, and windows that leave no room for the staging arrays, which scatter by
LDS atomics -- against the untiled passes, which add every product to global
memory.  Degrees 1 to 3 (4, 9 and 16 nodes of the 16-row products), beams that
leave their windows between sorts, and counts that leave partial waves.

Tolerance 1e-11 normwise: the runs differ by the order of float64 sums over
steps (the state to about 1e-14), and 1e-10 is what the gradient is held to
against autograd.
"""

import numpy as np
import pytest
import torch

from paper_2410_18414_amd import adjoint, pic, workloads
from pic_harness import rel

pytestmark = pytest.mark.gpu


def _gradient(w, degree, n, flags=0, **plan):
    cfg = pic.make_config(w["nx"], w["ny"], w["lx"], w["ly"], w["dt"], degree=degree, scheme="bdf", bdf_order=2,
                          dtype="f64", q=w["q"], m=w["m"], max_particles=n, flags=pic.FLAG_ADJOINT | flags, **plan)
    ctx = pic.Context(cfg)
    x, y = (torch.as_tensor(w[k][:n], device="cuda").requires_grad_(True) for k in ("x", "y"))
    P = torch.as_tensor(np.ascontiguousarray(w["P"][:n].T), device="cuda").requires_grad_(True)
    adjoint.field_energy(ctx, x, y, P, 7, every=3).backward()
    ctx.close()
    return [t.grad.cpu().numpy() for t in (x, y, P)]


@pytest.mark.parametrize("degree", [1, 2, 3])
@pytest.mark.parametrize("n", [1, 63, 2000])
def test_sorted_gradient_equals_untiled(gpu_lib, degree, n):
    w = workloads.weibel(nx=32, ny=32, ppc=2, seed=17, drift=0.6)
    ref = _gradient(w, degree, n, flags=pic.FLAG_NO_SORT)
    plans = [dict(), dict(tile_cells=8), dict(tile_cells=8, slack=2), dict(slack=4), dict(sort_interval=9, chunk=640)]
    for plan in plans:
        print("case", degree, n, plan, flush=True)
        for got, want in zip(_gradient(w, degree, n, **plan), ref):
            assert rel(got, want) <= 1e-11, plan
