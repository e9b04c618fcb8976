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
