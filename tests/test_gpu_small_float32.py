"""What float32 particles gather after a one-launch solve (needs an MI355X).

k_solve_small stores the float64 planes of the mesh export and the float32 record
that the particles read separately.  From a history of random real fields, so that
every one of the eleven gathered fields is as large as the others, one step's
momenta and velocities against the oracle's (1e-4 normwise, the float32 parity
tolerance, per component and step increment), and the exported mesh to the same;
even and odd sides, the smallest and the longest columns, every stepper family."""

import numpy as np
import pytest
import torch

from paper_2410_18414_amd import pic, workloads
from pic_harness import DT_TOL, flat_to_hist, make_gpu, make_oracle, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(8, 8), (9, 8), (32, 32), (31, 33), (8, 128), (25, 40)])
@pytest.mark.parametrize("scheme,k", [("bdf", 2), ("cdf2", 1), ("dirk3", 1)])
def test_gathered_fields_match_oracle(gpu_lib, nx, ny, scheme, k):
    w = workloads.weibel(nx=nx, ny=ny, ppc=3, seed=11)
    o = make_oracle(w, 3, scheme, k)
    g = make_gpu(w, 3, scheme, "f32", bdf_order=k)
    rng = np.random.default_rng(nx * 1000 + ny)
    nf = pic.history_fields(g.cfg)
    flat = np.fft.rfft2(0.02 * rng.standard_normal((nf, ny, nx)))
    o.hist = flat_to_hist(o.p, flat)
    pic.set_history(g, torch.as_tensor(flat))
    P0 = pic.get_particles(g).cpu().numpy()[2:5]
    o.deposit()
    fields = o.solve()
    pic.deposit_current(g)
    pic.field_solve(g)
    mesh = pic.get_field(g, pic.FIELD_MESH).cpu().numpy()
    for f in range(12):
        assert rel(mesh[f], fields[f]) <= DT_TOL["f32"], f
    o.gather_push()
    pic.gather_push(g)
    a = pic.get_particles(g).cpu().numpy()
    dP, ref = a[2:5] - P0, o.part["P"].T - w["P"].T
    for c in range(2):  # P_z is constant
        assert rel(dP[c], ref[c]) <= DT_TOL["f32"], c
    for c in range(3):
        assert rel(a[5 + c], o.part["v"].T[c]) <= DT_TOL["f32"], c
    g.close()
