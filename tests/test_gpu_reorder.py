"""The bucket reorderings of large particle sets (needs an MI355X): the
first sort of loaded particles by way of tile buckets, and the export to the
original order by way of buckets of original indices.

P_z is constant in 2-D, so every particle carries a label through the run: it
must come back in its place, bit for bit.  The other values are compared with
the unsorted passes, whose particles never move (1e-10 float64, 1e-4 float32:
the parity tolerances of the step).
"""

import numpy as np
import pytest
import torch

from paper_2410_18414_amd import pic, workloads
from pic_harness import DT_TOL, rel, rel_periodic

pytestmark = pytest.mark.gpu


def _context(w, dtype, tile=0, flags=0, count=1):
    cfg = [pic.make_config(w["nx"], w["ny"], w["lx"], w["ly"], w["dt"], degree=2, dtype=dtype, q=w["q"], m=w["m"],
                           max_particles=len(w["x"]) + 5, flags=flags, tile_cells=tile) for _ in range(count)]
    ctx = pic.Context(cfg)
    for i in range(count):
        if count > 1:
            pic.select_instance(ctx, i)
        pic.init_particles(ctx, torch.as_tensor(w["x"]), torch.as_tensor(w["y"]),
                           torch.as_tensor(np.ascontiguousarray(w["P"].T)))
    return ctx


def _check(got, want, w, dtype):
    z = torch.as_tensor(w["P"][:, 2], device="cuda")
    assert torch.equal(got[4], z.float().double() if dtype == "f32" else z)
    got, want = got.cpu().numpy(), want.cpu().numpy()
    for a, L in ((0, w["lx"]), (1, w["ly"])):
        assert rel_periodic(got[a], want[a], L) <= DT_TOL[dtype]
    for a in (slice(2, 4), slice(5, 8), slice(8, 11)):
        assert rel(got[a], want[a]) <= DT_TOL[dtype]


# (grid, ppc, tile edge): the smallest sets that take the bucket passes (sort
# 2^18, export 2^19 particles), one particle more, tiles in groups (4096
# tiles), partial tiles, 2 million
@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("nx,ny,ppc,tile,cut", [(128, 128, 16, 0, 0), (64, 64, 129, 8, 4095), (256, 256, 8, 4, 0),
                                               (150, 97, 40, 0, 1), (256, 256, 32, 0, 3)])
def test_large_sets_keep_their_order(gpu_lib, nx, ny, ppc, tile, cut, dtype):
    print("case", nx, ny, ppc, tile, cut, dtype, flush=True)
    w = workloads.weibel(nx=nx, ny=ny, ppc=ppc, seed=21, drift=0.2)
    for k in ("x", "y", "P"):
        w[k] = w[k][:len(w[k]) - cut]
    a, b = _context(w, dtype, tile), _context(w, dtype, tile, pic.FLAG_NO_SORT)
    _check(pic.get_particles(a), pic.get_particles(b), w, dtype)
    for n in (1, 8):
        pic.step(a, n)
        pic.step(b, n)
        _check(pic.get_particles(a), pic.get_particles(b), w, dtype)
    pic.set_particles(a, pic.get_particles(b))  # back to the original order: sorted anew
    pic.step(a, 2)
    pic.step(b, 2)
    _check(pic.get_particles(a), pic.get_particles(b), w, dtype)
    a.close()
    b.close()


def test_ensemble_is_sorted_together(gpu_lib):
    """Four instances below the threshold each and above it together, from a cloud (uneven buckets)."""
    w = workloads.cloud(nx=64, ny=64, ppc=17, seed=22)
    w["P"][:, 2] = np.arange(len(w["x"])) * 1e-9 * w["m"]
    ctx, alone = _context(w, "f64", count=4), _context(w, "f64", flags=pic.FLAG_NO_SORT)
    pic.step_batched(ctx, 9)
    pic.step(alone, 9)
    for i in range(4):
        pic.select_instance(ctx, i)
        _check(pic.get_particles(ctx), pic.get_particles(alone), w, "f64")
    ctx.close()
    alone.close()
