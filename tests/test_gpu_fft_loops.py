"""LDS FFTs of powers of two with more than one butterfly per thread (needs an
MI355X): the passes of the general lengths, with reciprocals for divisions.

Row transforms take them at 1024 with four rows to a block (ny >= 344) and at 512
with eight (ny >= 683); one deposit and solve against the oracle, float64, the
spectral history and the mesh within 1e-10 normwise (the parity tolerance of the
step).  The adjoint's columns, up to eight to a block, take them from 256 on; one
adjoint step against the oracle's vector-Jacobian product, 1e-10 normwise."""

import numpy as np
import pytest
import torch

from oracle import adjoint as oadj
from oracle import pic as opic
from paper_2410_18414_amd import pic, workloads
from pic_harness import hist_to_flat, make_gpu, make_oracle, oracle_params, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(1024, 352), (512, 688)])
def test_rows_match_oracle(gpu_lib, nx, ny):
    w = workloads.weibel(nx=nx, ny=ny, ppc=1, seed=5)
    w = dict(w, x=w["x"][::5], y=w["y"][::5], P=w["P"][::5])
    o = make_oracle(w, 1, "bdf", 1)
    g = make_gpu(w, 1, "bdf", "f64", bdf_order=1)
    o.deposit()
    fields = o.solve()
    pic.deposit_current(g)
    pic.field_solve(g)
    mesh = pic.get_field(g, pic.FIELD_MESH).cpu().numpy()
    for f in range(12):
        assert rel(mesh[f], fields[f]) <= 1e-10, f
    assert rel(pic.get_history(g).cpu().numpy(), hist_to_flat(o.p, o.hist)) <= 1e-10
    g.close()


@pytest.mark.parametrize("nx,ny", [(8, 256), (8, 512), (1024, 16)])
def test_adjoint_columns_match_oracle(gpu_lib, nx, ny):
    w = workloads.weibel(nx=nx, ny=ny, ppc=2, seed=31)
    p = oracle_params(w, 3, "bdf", 2)
    s = opic.State(p, w["x"], w["y"], w["P"])
    s.step(2)
    rng = np.random.default_rng(3)
    part = {k: s.part[k] for k in ("x", "y", "P", "v", "vprev")}
    lp = {k: rng.standard_normal(np.shape(part[k])) for k in part}
    flat = hist_to_flat(p, s.hist)
    lh = rng.standard_normal(flat.shape) + 1j * rng.standard_normal(flat.shape)
    ref_p, ref_h = oadj.step_vjp(p, part, s.hist, lp, lh)
    ctx = make_gpu(w, 3, "bdf", "f64", flags=pic.FLAG_ADJOINT)

    def stack(d):
        return np.concatenate([d["x"][None], d["y"][None], d["P"].T, d["v"].T, d["vprev"].T])

    def dev(a):
        return torch.as_tensor(np.ascontiguousarray(a), device=ctx.device)
    pic.set_particles(ctx, dev(stack(part)))
    pic.set_history(ctx, dev(flat))
    lam, lam_h = dev(stack(lp)), dev(lh)
    pic.step_adjoint(ctx, lam, lam_h)
    got = lam.cpu().numpy()
    ref = stack({k: np.asarray(v) for k, v in ref_p.items()})
    for k in (slice(0, 1), slice(1, 2), slice(2, 5), slice(5, 8), slice(8, 11)):
        assert rel(got[k], ref[k]) <= 1e-10, k
    assert rel(lam_h.cpu().numpy(), ref_h) <= 1e-10
    ctx.close()
