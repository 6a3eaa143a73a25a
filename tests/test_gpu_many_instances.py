"""Blocks find their instance in ensembles around and beyond the 64 that one
round of loads tells apart (needs an MI355X).

Every member has its own grid and particle count (some with one particle, so a
kind of block has as many as another kind has few); after sorted and unsorted
steps each member equals the same instance alone to the step's parity
tolerance, 1e-10 in float64."""

import numpy as np
import pytest
import torch

from paper_2410_18414_amd import pic, workloads
from pic_harness import make_gpu, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [2, 63, 64, 65, 129])
@pytest.mark.parametrize("extra", [0, pic.FLAG_NO_SORT], ids=["tiled", "untiled"])
def test_members_equal_instances_alone(gpu_lib, count, extra):
    ws = []
    for i in range(count):
        # 40 x 40: the members' solves in three launches instead of one
        w = workloads.cloud(nx=40 if extra and i == count // 2 else 8 + i % 5, ny=40 if i == count // 2 else 8 + i % 3, ppc=2, seed=i, drift=0.2, vth=0.05)
        n = 1 if i % 7 == 3 else len(w["x"]) - i % 11
        ws.append(dict(w, x=w["x"][:n], y=w["y"][:n], P=w["P"][:n]))
    cfgs = [pic.make_config(w["nx"], w["ny"], w["lx"], w["ly"], w["dt"], degree=2, scheme="bdf", bdf_order=1,
                            dtype="f64", q=w["q"], m=w["m"], max_particles=len(w["x"]), flags=extra) for w in ws]
    b = pic.Context(cfgs)
    for i, w in enumerate(ws):
        pic.select_instance(b, i)
        pic.init_particles(b, torch.as_tensor(w["x"], device=b.device), torch.as_tensor(w["y"], device=b.device),
                           torch.as_tensor(np.ascontiguousarray(w["P"].T), device=b.device))
    pic.step_batched(b, 8)
    for i in sorted({0, 1, count // 2, count - 2, count - 1} | set(range(0, count, 16))):
        w = ws[i]
        a = make_gpu(w, 2, "bdf", "f64", bdf_order=1, flags=extra)
        pic.step(a, 8)
        pic.select_instance(b, i)
        assert rel(pic.get_history(b).cpu().numpy(), pic.get_history(a).cpu().numpy()) <= 1e-10, i
        pa, pb = (pic.get_particles(c) for c in (a, b))
        for k in range(2):
            d = (pa[k] - pb[k]).abs()
            box = (w["lx"], w["ly"])[k]
            assert torch.minimum(d, box - d).max().item() <= 1e-10 * box, (i, k)
        a.close()
    b.close()


def test_row_groups_of_ensembles_keep_the_bits(gpu_lib):
    """The row transforms of an ensemble take more rows per block than those of an
    instance alone (up to 16, the last group partial): with the deterministic
    deposit every member keeps the bits of the instance alone."""
    sides = [(64, 97), (33, 100), (128, 50), (48, 112), (512, 48), (512, 16), (16, 96), (8, 49)]
    ws = [workloads.cloud(nx=sides[i % 8][0], ny=sides[i % 8][1], ppc=1, seed=i, drift=0.2, vth=0.05) for i in range(64)]
    flags = pic.FLAG_DETERMINISTIC
    cfgs = [pic.make_config(w["nx"], w["ny"], w["lx"], w["ly"], w["dt"], degree=2, scheme="bdf", bdf_order=2,
                            dtype="f32", q=w["q"], m=w["m"], max_particles=len(w["x"]), flags=flags) for w in ws]
    b = pic.Context(cfgs)
    for i, w in enumerate(ws):
        pic.select_instance(b, i)
        pic.init_particles(b, torch.as_tensor(w["x"], device=b.device), torch.as_tensor(w["y"], device=b.device),
                           torch.as_tensor(np.ascontiguousarray(w["P"].T), device=b.device))
    pic.step_batched(b, 6)
    for i in list(range(8)) + [63]:
        a = make_gpu(ws[i], 2, "bdf", "f32", bdf_order=2, flags=flags)
        pic.step(a, 6)
        pic.select_instance(b, i)
        assert torch.equal(pic.get_history(b), pic.get_history(a)), i
        assert torch.equal(pic.get_particles(b), pic.get_particles(a)), i
        a.close()
    b.close()
