"""GPU parity of the double z march on y lines of exactly 384 (whole chunks of
eight planes: the exact-count form; others: the general one), whole, split,
segmented and with periodic z, against the CPU oracle at 1e-12."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zsplit,shape", [("off", (8, 384, 6)), ("off", (9, 384, 6)), ("off", (24, 384, 4)),
                                          ("on", (16, 384, 4)), ("on", (32, 384, 4)), ("seg", (48, 384, 4))])
@pytest.mark.parametrize("bc", ["PPDDDN", "DDNNDD", "PPPPNN", "NNPPPP"])
def test_lines_of_384(bc, zsplit, shape):
    import torch
    from paper_1909_05423_amd import Plan
    from gpu_util import banner, rel_max, to_dev
    if bc[4] == "P" and zsplit != "off":
        zsplit = "off"   # periodic z has one layout
    banner(f"lines of 384 {bc} {zsplit} {shape}")
    nz, ny, nx = shape
    h = (1.0 / nx, 1.0 / ny, 1.0 / nz)
    f = np.random.default_rng(61 + nz).standard_normal((2,) + shape)
    u = Plan(shape, bc, h, dtype="f64", batch=2, zsplit=zsplit).solve(to_dev(f))
    torch.cuda.synchronize()
    for b in range(2):
        assert rel_max(u[b].cpu().numpy(), oracle.solve(f[b], bc, h, "mean")) < 1e-12, (bc, zsplit, shape)
