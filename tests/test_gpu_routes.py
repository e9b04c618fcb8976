"""Which kernels the automatic layout takes, at the edges of its rules, and that
they agree with the march of one workgroup per column there.

The plane kernels reduce the source's sums in their z kernel, so a solve by them
has no launch in the group of reductions (pp_plan_kernel_times); the separate y
transforms around the z-systems round differently from the march, so equal bits
mean that the march ran."""

import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

H = (1.0, 1.0, 1.0)
TOL = {"f64": 1e-12, "f32": 1e-5}


def _run(shape, bc, dtype, batch, zsplit, faces=False):
    import torch
    from paper_1909_05423_amd import Plan, _lib
    tdt = torch.float32 if dtype == "f32" else torch.float64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(sum(shape) + batch)
    draw = lambda s: torch.randn(s, generator=gen, device="cuda", dtype=tdt)   # noqa: E731
    plan = Plan(shape, bc, H, dtype=dtype, batch=batch, zsplit=zsplit)
    f = draw((batch,) + shape)
    g = [None if k == "P" else draw(plan.face_shape(i)) for i, k in enumerate(bc)] if faces else None
    lib = _lib.load()
    lib.pp_plan_set_timing(plan._handle, 1)
    u = plan.solve(f, faces=g)
    n = (ctypes.c_int * 4)()
    lib.pp_plan_kernel_times(plan._handle, None, n, 1)
    return u, n[3] == 0


def _close(a, b, dtype):
    return float((a.double() - b.double()).abs().max()) <= TOL[dtype] * float(b.double().abs().max())


# (shape, batch, the plane kernels run).  Planes of more than 8192 values from twelve
# on, of 4096 or more from 32 on where rows of 256 come in whole blocks; every size
# of workgroup, full and ragged (in float 1024 threads from 8193 values of row pairs on)
PLANES = [("f64", (31, 32, 256), 1, False), ("f64", (32, 32, 256), 1, True), ("f64", (3, 8, 256), 1, True),
          ("f64", (11, 72, 162), 3, False), ("f64", (12, 72, 162), 1, True), ("f64", (3, 54, 81), 1, True),
          ("f64", (13, 128, 128), 1, True), ("f32", (11, 162, 192), 1, False), ("f32", (12, 162, 192), 1, True),
          ("f32", (31, 128, 256), 2, False), ("f32", (32, 128, 256), 1, True), ("f32", (12, 243, 128), 2, True),
          ("f32", (13, 128, 128), 1, True), ("f32", (1, 64, 64), 1, True), ("f32", (12, 162, 216), 1, False)]


@pytest.mark.parametrize("faces", [False, True])
@pytest.mark.parametrize("bc", ["DDNNDN", "PPDDDD"])
@pytest.mark.parametrize("dtype,shape,batch,planes", PLANES)
def test_planes(dtype, shape, batch, planes, bc, faces):
    from gpu_util import banner
    banner(f"route planes {dtype} {shape} x {batch} {bc} faces={faces}")
    u, took = _run(shape, bc, dtype, batch, "auto", faces)
    v, march = _run(shape, bc, dtype, batch, "off", faces)
    assert took == planes and not march
    assert _close(u, v, dtype)


# (shape, batch, the y transforms run by themselves): 20 planes, 900 pairs a plane, the
# most pairs; lines of 512 as others
LINES = [("f32", (9, 128, 256), 2, False), ("f32", (19, 18, 288), 1, False), ("f32", (20, 18, 288), 1, True),
         ("f64", (25, 192, 384), 1, False), ("f64", (48, 192, 384), 1, True), ("f64", (200, 512, 144), 1, True),
         ("f32", (70, 512, 216), 1, True), ("f64", (70, 512, 192), 1, False), ("f32", (32, 512, 128), 1, False),
         ("f32", (80, 256, 486), 1, False)]


@pytest.mark.parametrize("bc", ["NNPPPP", "PPNNPP"])
@pytest.mark.parametrize("dtype,shape,batch,lines", LINES)
def test_separate_y_transforms(dtype, shape, batch, lines, bc):
    import torch
    from gpu_util import banner
    banner(f"route lines {dtype} {shape} x {batch} {bc}")
    u, _ = _run(shape, bc, dtype, batch, "auto")
    v, _ = _run(shape, bc, dtype, batch, "off")
    assert torch.equal(u, v) != lines
    assert _close(u, v, dtype)
