"""The LDS FFT over its lengths, through the field solve (needs an MI355X).

One deposit and solve from random particles against the oracle's, float64: the
spectral history and the twelve mesh fields within 1e-10 normwise (the parity
tolerance of the step; the transforms themselves are accurate to about 1e-15).
Lengths: every power of two (one butterfly per thread, and the looped passes of
the row kernel at 1024), butterflies of 3 and 5, and the passes of any odd
radix -- one (7, 127, 509), a second one with twiddles (11 x 13), a repeated one
(7 x 7), and mixtures.
"""

import numpy as np
import pytest
import torch

from paper_2410_18414_amd import pic, workloads
from pic_harness import hist_to_flat, make_gpu, make_oracle, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(8, 16), (16, 8), (32, 64), (64, 32), (128, 256), (256, 128), (512, 8), (8, 512),
                                   (1024, 16), (16, 1024), (9, 25), (14, 49), (49, 22), (15, 127), (127, 20),
                                   (143, 9), (10, 143), (254, 21), (12, 509), (509, 12), (30, 60), (968, 8), (9, 972)])
def test_solve_matches_oracle(gpu_lib, nx, ny):
    print("case", nx, ny, flush=True)
    w = workloads.weibel(nx=nx, ny=ny, ppc=2, seed=5)
    o = make_oracle(w, 3, "bdf", 2)
    g = make_gpu(w, 3, "bdf", "f64")
    o.deposit()
    fields = o.solve()
    pic.deposit_current(g)
    pic.field_solve(g)
    mesh = pic.get_field(g, pic.FIELD_MESH).cpu().numpy()
    for f in range(12):
        assert rel(mesh[f], fields[f]) <= 1e-10, f
    assert rel(pic.get_history(g).cpu().numpy(), hist_to_flat(o.p, o.hist)) <= 1e-10
    g.close()
