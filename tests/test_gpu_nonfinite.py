"""Non-finite values on the GPU are reported, never returned as a solution."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [1e60, 1e200])
@pytest.mark.parametrize("shape,bc", [((4, 8, 8), "DDDDDD"), ((4, 8, 8), "PPPPNN"), ((3, 6, 576), "PPNNPP")])
def test_refined_solve_past_the_float_range_is_reported(shape, bc, size):
    """A finite source whose spectra overflow float leaves a solution of NaN
    throughout, of which no maximum is left to compare a correction with."""
    from paper_1909_05423_amd import Plan, _lib
    from gpu_util import banner, to_dev
    banner(f"refined overflow {shape} {bc} {size}")
    f = np.random.default_rng(3).standard_normal(shape) * size
    plan = Plan(shape, bc, (1.0, 1.0, 1.0), dtype="f32_refined")
    with pytest.raises(_lib.PPError) as ei:
        plan.solve(to_dev(f))
    assert ei.value.status == -8


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("dtype", ["f64", "f32", "f32_refined"])
@pytest.mark.parametrize("entry", [0, 1, 2])
@pytest.mark.parametrize("shape,zsplit", [((6, 8, 12), "auto"), ((6, 8, 12), "off"), ((24, 8, 288), "auto"),
                                          ((3, 8, 768), "auto")])
def test_nonfinite_source_in_any_batch_entry_is_reported(shape, zsplit, entry, dtype, bad):
    """By the plane kernels, the march, the separate y transforms and shared rows."""
    import torch
    from paper_1909_05423_amd import Plan, _lib
    from gpu_util import banner, to_dev
    banner(f"nonfinite {dtype} {shape} {zsplit} entry {entry} {bad}")
    for bc in ("PPPPPP", "DDNNDN"):
        f = np.random.default_rng(4).standard_normal((3,) + shape)
        f[entry, 2, 3, 4] = bad
        plan = Plan(shape, bc, (1.0, 1.0, 1.0), dtype=dtype, batch=3, zsplit="off" if dtype == "f32_refined" else zsplit)
        with pytest.raises(_lib.PPError) as ei:
            plan.solve(to_dev(f, torch.float32 if dtype == "f32" else torch.float64))
            plan.last_info()
        assert ei.value.status == -8
        torch.cuda.synchronize()
