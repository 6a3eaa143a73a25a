"""The default chunk of small particle sets, on the CPU.

A chunk size shows in the workspace a configuration asks for (the chunk list has
room for ntiles + ceil(capacity / chunk) chunks of every member).  Sets of at most
8192 particles take chunks of 128 only while those leave a workgroup per CU: a set
alone and few members do, members of a large ensemble take longer chunks, as
larger members do."""

import ctypes

import pytest

from paper_2410_18414_amd import pic


def _bytes(count, nx, n, dtype, chunk):
    cfgs = [pic.make_config(nx, nx, 0.1 * nx, 0.1 * nx, 0.02, dtype=dtype, max_particles=n, chunk=chunk)] * count
    arr = (pic.ConfigStruct * count)(*cfgs)
    return pic.load().pic_batch_workspace_bytes(arr, ctypes.c_int32(count))


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("count,nx,n,short", [(1, 32, 4096, True), (1, 64, 8192, True), (8, 32, 4096, True),
                                              (9, 32, 4096, False), (64, 32, 4096, False), (64, 32, 8192, False),
                                              (1024, 16, 4096, False), (256, 64, 8000, False)])
def test_chunks_of_128_leave_at_most_a_workgroup_per_cu(count, nx, n, short, dtype):
    planned, small = _bytes(count, nx, n, dtype, 0), _bytes(count, nx, n, dtype, 128)
    assert planned > 0
    if short:
        assert planned == small
    else:
        assert planned < small
