"""Diagnostics at the edges of their block partials (needs an MI355X): one field
block, a few, and the full 64 with a remainder; one particle, one block of
particles and one more, and the full 256 blocks.  Scales, energy and kinetic
energy against the oracle, pic_diagnostics against pic_diagnostics_all.

Tolerance: the state itself may differ by 1e-10 normwise (the step's float64
tolerance), squares double it and the sums add rounding far below: 1e-9.
"""

import numpy as np
import pytest

from oracle import diagnostics as odiag
from paper_2410_18414_amd import pic, workloads
from pic_harness import make_gpu, make_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,n", [(8, 8, 1), (30, 32, 256), (33, 31, 257), (64, 64, 65536), (256, 250, 65537)])
@pytest.mark.parametrize("scheme", ["bdf", "cdf2", "dirk2"])
def test_diagnostics_of_any_size(gpu_lib, nx, ny, n, scheme):
    print("case", nx, ny, n, scheme, flush=True)
    w = workloads.weibel(nx=nx, ny=ny, ppc=-(-n // (nx * ny)), seed=3)
    for k in ("x", "y", "P"):
        w[k] = w[k][:n]
    o, g = make_oracle(w, 2, scheme), make_gpu(w, 2, scheme, "f64")
    o.step(3)
    pic.step(g, 3)
    got, ref = pic.diagnostics(g), odiag.residuals(o)
    v2 = (o.part["v"] ** 2).sum(1)
    ref["kinetic"] = float(((1.0 / np.sqrt(1.0 - v2) - 1.0) * w["m"]).sum())
    for k in ("gauge_scale", "gauss_scale", "energy", "kinetic"):
        assert abs(got[k] - ref[k]) <= 1e-9 * abs(ref[k]), (k, got[k], ref[k])
    both = dict(zip(pic.DIAG_NAMES, pic.diagnostics_all(g).cpu().numpy()[0]))
    for k in ("gauge_scale", "gauss_scale", "energy", "kinetic", "nonfinite"):
        assert abs(got[k] - both[k]) <= 1e-12 * abs(got[k]), k
    g.close()


@pytest.mark.parametrize("n", [2 * 65536 - 1, 4 * 65536, 4 * 65536 + 1, 7 * 65536 + 129])
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_particle_sums_over_whole_and_partial_batches(gpu_lib, n, dtype):
    """Four particles of a thread are loaded together: counts around one, two and
    four strides of the full 256 blocks.  The kinetic energy against numpy's of
    the exported velocities (n sums of positive terms: n 2^-53 < 1e-10)."""
    print("case", n, dtype, flush=True)
    w = workloads.weibel(nx=64, ny=64, ppc=-(-n // 4096), seed=5)
    for k in ("x", "y", "P"):
        w[k] = w[k][:n]
    g = make_gpu(w, 2, "bdf", dtype)
    pic.step(g, 2)
    v = pic.get_particles(g)[5:8].cpu().numpy()
    got = pic.diagnostics(g)
    want = float(((1.0 / np.sqrt(1.0 - (v ** 2).sum(0)) - 1.0) * w["m"]).sum())
    assert abs(got["kinetic"] - want) <= 1e-10 * want
    assert got["nonfinite"] == 0
    g.close()
