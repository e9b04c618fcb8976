"""Workspace of plans with rows over 512 and many batch entries: the partial
records of the x kernels are bounded by their grid, so what comes on top of the
spectra and the tables stays small, and calls on the fixed workspace fit it."""

import ctypes

import numpy as np
import pytest

from paper_1909_05423_amd import _lib


def _bytes(shape, dtype, batch, bc="PPPPNN"):
    lib = _lib.load()
    nz, ny, nx = shape
    p = ctypes.c_void_p()
    assert lib.pp_plan_create(nx, ny, nz, bc.encode(), (ctypes.c_double * 3)(1.0, 1.0, 1.0), dtype, batch,
                              ctypes.byref(p)) == 0
    n = lib.pp_plan_workspace_bytes(p)
    lib.pp_plan_destroy(p)
    return n


# (bytes: what the plan needs with one record per line of a workgroup and row block)
@pytest.mark.parametrize("shape,dtype,batch,most", [((16, 16, 1152), _lib.PP_F32, 64, 98312704),
                                                    ((8, 8, 1024), _lib.PP_F64, 1000, 1292714240),
                                                    ((1, 2, 2048), _lib.PP_F64, 512, 42140672),
                                                    ((3, 6, 576), _lib.PP_F32_REFINED, 200, 45839360)])
def test_records_do_not_grow_with_the_wavefronts_of_a_line(shape, dtype, batch, most):
    assert _bytes(shape, dtype, batch) <= most


def test_records_of_many_batch_entries_are_bounded_by_the_grid():
    # beyond 1024 workgroups the region grows with the batch, no longer with its square
    spectra = 8 * 8 * 1024 * 8
    one, two = (_bytes((8, 8, 1024), _lib.PP_F64, b) - b * spectra for b in (1000, 2000))
    assert two < 2.1 * one


@pytest.mark.parametrize("nz", [2270, 2280, 2290])
def test_low_parts_of_pivots_do_not_take_a_plan_past_the_fixed_workspace(nz):
    # (within 2 MB of it; the low parts of the pivots of these columns take 3 to 5)
    lib = _lib.load()
    p = ctypes.c_void_p()
    assert lib.pp_plan_create(96, 128, nz, b"DDDDDD", (ctypes.c_double * 3)(1.0, 1.0, 0.2), _lib.PP_F32, 1,
                              ctypes.byref(p)) == 0
    n = lib.pp_plan_workspace_bytes(p)
    lib.pp_plan_destroy(p)
    assert n <= _lib.NOALLOC_SCRATCH_BYTES


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_noalloc_solve_of_long_rows_and_a_batch(dtype):
    import torch
    from paper_1909_05423_amd import Plan
    from gpu_util import banner, rel_max, to_dev
    shape, batch = (16, 16, 1152), (64 if dtype == "f32" else 24)
    banner(f"noalloc long rows {dtype} {shape} x {batch}")
    tdt = torch.float32 if dtype == "f32" else torch.float64
    f = to_dev(np.random.default_rng(9).standard_normal((batch,) + shape), tdt)
    plan = Plan(shape, "PPPPNN", (1.0, 1.0, 1.0), dtype=dtype, batch=batch)
    out = torch.empty_like(f)
    plan.solve_noalloc(f, out)
    u = plan.solve(f)
    torch.cuda.synchronize()
    assert torch.equal(out, u)
    one = Plan(shape, "PPPPNN", (1.0, 1.0, 1.0), dtype=dtype)
    for b in (0, batch - 1):
        ref = one.solve(f[b].contiguous())
        assert rel_max(u[b].double().cpu().numpy(), ref.double().cpu().numpy()) < (1e-5 if dtype == "f32" else 1e-12)
