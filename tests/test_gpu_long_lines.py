"""GPU parity on lines over 512: x rows shared by two or four wavefronts and y
lines whose planes are shared by wavefronts in the z march, against the CPU
oracle.  Unit-cube spacings, as the other parity tests of long lines; relative
max-norm 1e-12 in double and for the refined solve, 1e-5 in float.
"""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5, "f32_refined": 1e-12}

# rows: two wavefronts (576; 729 odd; 768 and 1024 the exact-count forms, with and
# without whole row blocks), four (1152, 1458; 1728 and 2048 fewer rows per block in double)
ROWS = [(3, 6, 576), (2, 4, 729), (3, 8, 768), (3, 9, 768), (2, 6, 1024), (3, 6, 1152), (2, 9, 1458), (2, 8, 1728),
        (2, 12, 2048)]
# lines: the forms up to 1024, 1536 and 2048, each below and at its length, z whole
# chunks (4, 2 or 8 planes) and ragged
LINES = [(9, 729, 4), (8, 768, 6), (5, 1152, 4), (8, 1536, 3), (3, 1536, 4), (5, 1944, 2), (4, 2048, 4)]


def _check(shape, bc, dtype, faces=False, adjoint=False):
    import torch
    from paper_1909_05423_amd import Plan
    from gpu_util import banner, rel_max, to_dev
    banner(f"long lines {dtype} {bc} {shape} faces={faces}")
    nz, ny, nx = shape
    h = (1.0 / nx, 1.0 / ny, 1.0 / nz)
    rng = np.random.default_rng(nx * 7 + ny * 3 + nz)
    tdt = torch.float32 if dtype == "f32" else torch.float64

    def draw(s):
        a = rng.standard_normal(s)
        return a.astype(np.float32).astype(np.float64) if dtype == "f32" else a

    f = draw(shape)
    plan = Plan(shape, bc, h, dtype=dtype)
    fd = to_dev(f[None], tdt)
    if faces:
        dims = [(nz, ny), (nz, ny), (nz, nx), (nz, nx), (ny, nx), (ny, nx)]
        g = [None if k == "P" else draw(d) for k, d in zip(bc, dims)]
        u = plan.solve(fd, faces=[None if x is None else to_dev(x[None], tdt) for x in g])
        uo = oracle.solve(f, bc, h, "mean", faces=g)
    elif adjoint:
        u = plan.adjoint(fd)
        uo = oracle.solve_adjoint(f, bc, h, "mean")
    else:
        u = plan.solve(fd)
        uo = oracle.solve(f, bc, h, "mean")
    torch.cuda.synchronize()
    assert rel_max(u[0].double().cpu().numpy(), uo) < TOL[dtype], (dtype, bc, shape)


@pytest.mark.parametrize("dtype", ["f64", "f32", "f32_refined"])
@pytest.mark.parametrize("bc", ["PPPPNN", "DDNNDD", "NNPPDN"])
@pytest.mark.parametrize("shape", ROWS, ids=lambda s: "x".join(map(str, s)))
def test_long_rows(shape, bc, dtype):
    _check(shape, bc, dtype)


@pytest.mark.parametrize("dtype", ["f64", "f32", "f32_refined"])
@pytest.mark.parametrize("bc", ["PPPPNN", "DDNNDD", "NNDDPP", "PPPPPP"])
@pytest.mark.parametrize("shape", LINES, ids=lambda s: "x".join(map(str, s)))
def test_long_y_lines(shape, bc, dtype):
    _check(shape, bc, dtype)


# (in double: a face value enters the source as 2 g / h^2, whose float rounding
# at h = 1/1152 alone is 1.2e-5 of u)
@pytest.mark.parametrize("dtype", ["f64"])
@pytest.mark.parametrize("shape", [(3, 9, 768), (2, 6, 1152), (3, 1152, 4)], ids=lambda s: "x".join(map(str, s)))
def test_long_lines_faces_and_adjoint(shape, dtype):
    _check(shape, "DDNNDN", dtype, faces=True)
    _check(shape, "NNPPNN", dtype, adjoint=True)


@pytest.mark.parametrize("bc", ["NNPPPP", "DDDDPP", "PPPPNN"])
def test_refined_lines_of_1024_read_no_stale_workspace(bc):
    """The mixed march on lines of 1024, periodic z among them, on a workspace
    filled with NaN before the first solve."""
    import torch
    from paper_1909_05423_amd import Plan
    from gpu_util import banner, rel_max, to_dev
    for shape in [(16, 1024, 8), (16, 1024, 48)]:
        banner(f"refined lines of 1024 {bc} {shape}")
        h = (1.0 / shape[2], 1.0 / shape[1], 1.0 / shape[0])
        f = np.random.default_rng(67).standard_normal(shape)
        plan = Plan(shape, bc, h, dtype="f32_refined")
        plan.workspace.fill_(255)
        u = plan.solve(to_dev(f[None]))
        torch.cuda.synchronize()
        assert rel_max(u[0].cpu().numpy(), oracle.solve(f, bc, h, "mean")) < 1e-12, (bc, shape)
