"""The one-launch field solve of small grids (needs an MI355X).

Two solves from random particles against the oracle's, float64, at the grids
where it can go wrong: the smallest, the most modes it takes (5 x 128), the
largest areas (32 x 32, 33 x 31), odd sides (rows and columns paired with
nothing, pairs of rows that belong to two components), and the first size beyond
it; every family of steppers, and the naive mode.  The spectral history and the
twelve mesh fields within 1e-10 normwise (the parity tolerance of the step); the
second solve shows that J was cleared.  Float32: the exported mesh fields are the
ones the particles gather (their float32 rounding, 2^-24 of each value), and an
ensemble of small grids is solved in one launch as the instances alone are."""

import numpy as np
import pytest
import torch

from paper_2410_18414_amd import pic, workloads
from pic_harness import hist_to_flat, make_gpu, make_oracle, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(8, 8), (9, 8), (8, 9), (9, 13), (8, 128), (128, 8), (32, 32), (31, 33), (33, 31),
                                   (16, 64), (25, 40), (33, 32)])
@pytest.mark.parametrize("scheme,k,naive", [("bdf", 1, False), ("bdf", 6, False), ("cdf2", 1, False),
                                            ("dirk3", 1, False), ("bdf", 2, True), ("dirk2", 1, True)])
def test_solve_matches_oracle(gpu_lib, nx, ny, scheme, k, naive):
    print("case", nx, ny, scheme, k, naive, flush=True)
    w = workloads.cloud(nx=nx, ny=ny, ppc=2, seed=7, drift=0.2, vth=0.05)
    o = make_oracle(w, 2, scheme, k, naive=naive)
    g = make_gpu(w, 2, scheme, "f64", bdf_order=k, flags=pic.FLAG_NAIVE_RHO if naive else 0)
    for _ in range(2):
        o.deposit()
        fields = o.solve()
        pic.deposit_current(g)
        pic.field_solve(g)
        mesh = pic.get_field(g, pic.FIELD_MESH).cpu().numpy()
        for f in range(12):
            assert rel(mesh[f], fields[f]) <= 1e-10, f
        assert rel(pic.get_history(g).cpu().numpy(), hist_to_flat(o.p, o.hist)) <= 1e-10
        o.gather_push()
        pic.gather_push(g)
    g.close()


def test_float32_mesh_and_ensemble(gpu_lib):
    ws = [workloads.cloud(nx=nx, ny=ny, ppc=3, seed=8, drift=0.2, vth=0.05) for nx, ny in ((32, 32), (11, 24), (8, 128))]
    cfgs = [pic.make_config(w["nx"], w["ny"], w["lx"], w["ly"], w["dt"], degree=2, scheme="bdf", bdf_order=2,
                            dtype="f32", q=w["q"], m=w["m"], max_particles=len(w["x"])) for w in ws]
    b = pic.Context(cfgs)
    alone = [make_gpu(w, 2, "bdf", "f32", bdf_order=2) for w in ws]
    for i, w in enumerate(ws):
        pic.select_instance(b, i)
        pic.init_particles(b, torch.as_tensor(w["x"], device=b.device), torch.as_tensor(w["y"], device=b.device),
                           torch.as_tensor(np.ascontiguousarray(w["P"].T), device=b.device))
    pic.step_batched(b, 5)
    pic.deposit_current(b)
    pic.field_solve(b)
    for i, a in enumerate(alone):
        pic.step(a, 5)
        pic.deposit_current(a)
        pic.field_solve(a)
        pic.select_instance(b, i)
        ma, mb = (pic.get_field(c, pic.FIELD_MESH).cpu().numpy() for c in (a, b))
        assert np.isfinite(ma).all() and np.abs(ma).max() > 0
        # float32 particles, the same fixed-point sums up to the order of the
        # windows' float64 additions, which particles' float32 roundings carry on
        assert rel(mb, ma) <= 1e-5, i
        a.close()
    b.close()
