"""The counting sort at the edges of its passes (needs an MI355X): waves and
blocks of the count pass that are partly empty (one particle per thread, and four
from 3 x 2^19 particles on), tiles of 16 to 1024 cells in the cell scan's lanes
and passes of four per lane, and one to several passes of the tile scan's 256
tiles.

P_z is constant in 2-D: it labels a particle and must come back in its place, bit
for bit.  The other values are compared with the unsorted passes (1e-10 float64,
1e-4 float32: the parity tolerances of the step)."""

import numpy as np
import pytest
import torch

from paper_2410_18414_amd import pic, workloads
from pic_harness import DT_TOL, rel, rel_periodic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,tile,n", [(32, 32, 16, 1), (32, 32, 16, 63), (32, 32, 16, 65), (32, 32, 8, 256),
                                          (32, 32, 16, 257), (64, 64, 4, 4095), (64, 64, 32, 4096), (64, 64, 16, 4097),
                                          (40, 24, 4, 2000), (64, 68, 4, 3001), (128, 130, 4, 5000),
                                          (128, 128, 0, 3 * (1 << 19) - 1), (128, 128, 0, 3 * (1 << 19)),
                                          (128, 128, 0, 3 * (1 << 19) + 1025)])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_sorted_steps_equal_unsorted(gpu_lib, nx, ny, tile, n, dtype):
    if dtype == "f64" and tile == 32:
        tile = 16  # float64 windows of 32 x 32 tiles do not fit the LDS
    print("case", nx, ny, tile, n, dtype, flush=True)
    w = workloads.weibel(nx=nx, ny=ny, ppc=-(-n // (nx * ny)), seed=3, drift=0.2)
    pick = np.random.default_rng(4).permutation(len(w["x"]))[:n]
    for k in ("x", "y", "P"):
        w[k] = w[k][pick]
    got, want = [], []
    for out, flags in ((got, 0), (want, pic.FLAG_NO_SORT)):
        cfg = pic.make_config(nx, ny, w["lx"], w["ly"], w["dt"], degree=2, dtype=dtype, q=w["q"], m=w["m"],
                              max_particles=n, flags=flags, tile_cells=0 if flags else tile,
                              sort_interval=0 if flags else 2)
        c = pic.Context(cfg)
        pic.init_particles(c, torch.as_tensor(w["x"]), torch.as_tensor(w["y"]),
                           torch.as_tensor(np.ascontiguousarray(w["P"].T)))
        pic.step(c, 6)
        out.append(pic.get_particles(c).cpu().numpy())
        c.close()
    got, want = got[0], want[0]
    z = w["P"][:, 2]
    assert np.array_equal(got[4], z.astype(np.float32) if dtype == "f32" else z)
    for a, L in ((0, w["lx"]), (1, w["ly"])):
        assert rel_periodic(got[a], want[a], L) <= DT_TOL[dtype]
    for a in (slice(2, 4), slice(5, 8), slice(8, 11)):
        assert rel(got[a], want[a]) <= DT_TOL[dtype]
