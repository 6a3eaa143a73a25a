"""The float32 fixed-point deposit at the edge of its scale (needs an MI355X).

A chunk of `count` particles sits on one mesh node (linear splines: the whole
weight there) and moves at the speed of light: the largest window sum a chunk
can hold.  Counts around the powers of two where the scale changes, and above
2^14 where the rule rounds up.  The mesh total of J_x must be n q c / (dx dy).

Tolerance: a contribution is rounded by at most half a unit at each of the four
nodes it touches, and the scale leaves a full contribution at least 2^(29 - l)
units, l = ceil(log2(count)) at most and not below 9: 2 / 2^(29 - l), plus 2e-6
for the float32 products (a dozen roundings of 2^-24).
"""

import math

import pytest
import torch

from paper_2410_18414_amd import pic

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [1, 511, 512, 513, 1023, 1024, 2047, 2048, 16383, 16384, 16385, 40000, 65535])
@pytest.mark.parametrize("det", [False, True])
def test_largest_sum_of_a_chunk(gpu_lib, count, det):
    nx = ny = 16
    cfg = pic.make_config(nx, ny, 16.0, 16.0, 0.5, degree=1, dtype="f32", q=-1.0 / count, m=1.0 / count,
                          max_particles=count, chunk=max(64, count), flags=pic.FLAG_DETERMINISTIC if det else 0)
    ctx = pic.Context(cfg)
    x = torch.full((count,), 4.5, dtype=torch.float64)
    y = torch.full((count,), 9.0, dtype=torch.float64)
    P = torch.zeros(3, count, dtype=torch.float64)
    P[0] = 1e6 / count  # v = c (1 - 5e-13): c in float32
    pic.init_particles(ctx, x, y, P)
    pic.deposit_current(ctx)
    J = pic.get_field(ctx, pic.FIELD_J).cpu()
    level = max(9, math.ceil(math.log2(count))) if count > 1 else 9
    assert abs(float(J[0].sum()) + 1.0) <= 2.0 / 2 ** (29 - level) + 2e-6
    assert float(J[0, 9, 5]) < -0.999
    assert float(J[1:].abs().max()) == 0.0
    ctx.close()
