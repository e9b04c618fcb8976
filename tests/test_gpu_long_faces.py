"""Float face values on rows over 512: rows shared by two and four wavefronts, whole
and ragged blocks, against the CPU oracle.

Spacings of order 1 and face values of order 1 keep the lifted 2 g / h^2 of the size
of f, so that its rounding to float is as f's own and the float bound holds."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", ["DDNNDN", "NNDDND", "PPDDDD"])
@pytest.mark.parametrize("shape", [(3, 6, 576), (3, 8, 768), (3, 9, 768), (2, 16, 1024), (2, 6, 1152), (2, 8, 2048)],
                         ids=lambda s: "x".join(map(str, s)))
def test_float_faces_on_long_rows(shape, bc):
    import torch
    from paper_1909_05423_amd import Plan
    from gpu_util import banner, rel_max, to_dev
    banner(f"float faces on long rows {bc} {shape}")
    nz, ny, nx = shape
    rng = np.random.default_rng(nx + ny)
    draw = lambda s: rng.standard_normal(s).astype(np.float32).astype(np.float64)   # noqa: E731
    h = (1.0, 1.0, 1.0)
    f = draw(shape)
    dims = [(nz, ny), (nz, ny), (nz, nx), (nz, nx), (ny, nx), (ny, nx)]
    faces = [None if k == "P" else draw(d) for k, d in zip(bc, dims)]
    plan = Plan(shape, bc, h, dtype="f32")
    u = plan.solve(to_dev(f[None], torch.float32), faces=[None if g is None else to_dev(g[None], torch.float32) for g in faces])
    torch.cuda.synchronize()
    assert rel_max(u[0].double().cpu().numpy(), oracle.solve(f, bc, h, "mean", faces=faces)) < 1e-5
