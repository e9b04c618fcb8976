"""GPU parity of the small-plane kernels (x and y transforms of a z plane in one
workgroup, z-systems in one pass over segments) against the CPU oracle and
against the march of one workgroup per column on the same inputs.

Tolerances as the other parity tests (relative max-norm): 1e-12 in double, 1e-5
in float.
"""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5}

# (nz, ny, nx): one value; odd x and y; the smallest workgroup full (2048
# values a plane in double) and one over; the middle and the largest workgroup,
# full and ragged; lines of 243 and 256 (three and two stages); z at the edges
# of a thread's rows (8, 16) and of a segment's workgroup
SHAPES = [(1, 1, 1), (5, 27, 9), (9, 64, 64), (8, 54, 81), (17, 64, 128), (7, 96, 144), (3, 128, 128), (6, 16, 243),
          (4, 256, 24), (128, 8, 12), (129, 9, 8), (257, 4, 6)]


def _solve(f, bc, h, dtype, zsplit="auto", gauge="mean", batch=1, adjoint=False, faces=None):
    import torch
    from paper_1909_05423_amd import Plan
    from gpu_util import to_dev
    plan = Plan(f.shape[-3:], bc, h, dtype=dtype, batch=batch, gauge=gauge, zsplit=zsplit)
    tdt = torch.float32 if dtype == "f32" else torch.float64
    fd = to_dev(f.reshape((batch,) + f.shape[-3:]), tdt)
    if faces is not None:
        u = plan.solve(fd, faces=[None if g is None else to_dev(g[None], tdt) for g in faces])
    else:
        u = plan.adjoint(fd) if adjoint else plan.solve(fd)
    torch.cuda.synchronize()
    return u.double().cpu().numpy().reshape(f.shape), plan


def _input(rng, shape, dtype):
    f = rng.standard_normal(shape)
    return f.astype(np.float32).astype(np.float64) if dtype == "f32" else f


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("bc", ["PPPPDN", "NNDDDD", "DDNNND", "PPNNNN", "DDPPPP"])
def test_plane_vs_oracle_and_march(dtype, bc):
    from gpu_util import banner, rel_max
    rng = np.random.default_rng(sum(map(ord, bc + dtype)))
    for shape in SHAPES:
        if bc[4] == "P" and shape[0] < 3:
            continue
        banner(f"plane {dtype} {bc} {shape}")
        h = (1.0 / shape[2], 1.0 / shape[1], 1.0 / shape[0])
        f = _input(rng, shape, dtype)
        u, _ = _solve(f, bc, h, dtype)
        u1, _ = _solve(f, bc, h, dtype, zsplit="off")
        uo = oracle.solve(f, bc, h, "mean")
        assert rel_max(u, uo) < TOL[dtype], (dtype, bc, shape)
        assert rel_max(u1, uo) < TOL[dtype], (dtype, bc, shape)


@pytest.mark.parametrize("gauge", ["mean", "pin", "pin_raw"])
@pytest.mark.parametrize("bc", ["PPPPNN", "NNPPPP", "NNNNNN"])
def test_plane_singular_gauges_batch_adjoint(bc, gauge):
    from gpu_util import banner, rel_max
    rng = np.random.default_rng(41)
    for shape in [(33, 12, 16), (18, 9, 27)]:
        banner(f"plane gauge {gauge} {bc} {shape}")
        h = tuple(rng.uniform(0.5, 2.0, 3))
        f = rng.standard_normal((3,) + shape) + np.array([0.3, -1.0, 2.0])[:, None, None, None]
        u, plan = _solve(f, bc, h, "f64", gauge=gauge, batch=3)
        _, means, _ = plan.last_info()
        a, _ = _solve(f, bc, h, "f64", gauge=gauge, batch=3, adjoint=True)
        for b in range(3):
            assert rel_max(u[b], oracle.solve(f[b], bc, h, gauge)) < 1e-12, (b, shape)
            assert rel_max(a[b], oracle.solve_adjoint(f[b], bc, h, gauge)) < 1e-12, (b, shape)
            expect = f[b].mean() if gauge != "pin_raw" else 0.0
            assert abs(means[b] - expect) < 1e-13 * max(1.0, abs(f[b]).max())


@pytest.mark.parametrize("zsplit", ["auto", "off"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("bc", ["DDNNDN", "PPDDNN", "NNPPND"])
def test_plane_and_march_face_values(dtype, bc, zsplit):
    """Face values on every non-periodic face, by the plane kernels and by the x
    kernels and the march."""
    from gpu_util import banner, rel_max
    rng = np.random.default_rng(43)
    for shape in [(6, 9, 16), (5, 96, 144)]:
        banner(f"plane faces {dtype} {bc} {shape} {zsplit}")
        nz, ny, nx = shape
        h = (1.0 / nx, 1.0 / ny, 1.0 / nz)
        f = _input(rng, shape, dtype)
        dims = [(nz, ny), (nz, ny), (nz, nx), (nz, nx), (ny, nx), (ny, nx)]
        faces = [None if k == "P" else _input(rng, d, dtype) for k, d in zip(bc, dims)]
        u, _ = _solve(f, bc, h, dtype, zsplit=zsplit, faces=faces)
        uo = oracle.solve(f, bc, h, "mean", faces=faces)
        assert rel_max(u, uo) < TOL[dtype], (dtype, bc, shape)


@pytest.mark.parametrize("bc", ["DDPPNN", "DDPPPP"])
def test_plane_z_in_chunks(bc):
    """More planes than one workgroup's segments hold (the z-systems in chunks)."""
    from gpu_util import banner, rel_max
    rng = np.random.default_rng(47)
    for dtype, shape in [("f64", (1025, 4, 8)), ("f64", (2100, 6, 4)), ("f32", (1025, 4, 8))]:
        h = (1.0 / 64, 1.0 / 64, 1.0 / 64)
        f = _input(rng, shape, dtype)
        banner(f"plane chunks {dtype} {bc} {shape}")
        u, _ = _solve(f, bc, h, dtype)
        assert rel_max(u, oracle.solve(f, bc, h, "mean")) < TOL[dtype], (dtype, shape)


# (nz, ny, nx) off the small-plane rule (a line over 256) whose march would be one
# workgroup per column with few columns: y transforms by themselves.  Groups of
# lines whole and ragged, odd lines, one line of 512 per quarter group, z in one
# pass and in chunks
LINES = [(5, 8, 288), (3, 9, 324), (4, 288, 8), (3, 512, 4), (6, 243, 288), (17, 4, 512), (1025, 2, 288)]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("bc", ["PPPPPP", "NNDDPP", "DDNNPP", "NNPPPP", "PPNNPP"])
def test_separate_y_transforms_vs_oracle_and_march(dtype, bc):
    from gpu_util import banner, rel_max
    rng = np.random.default_rng(1 + sum(map(ord, bc + dtype)))
    for shape in LINES:
        banner(f"lines {dtype} {bc} {shape}")
        h = (1.0 / shape[2], 1.0 / shape[1], 1.0 / shape[0])
        if shape[0] > 1000:
            h = (1.0 / 64, 1.0 / 64, 1.0 / 64)
        f = _input(rng, shape, dtype)
        u, _ = _solve(f, bc, h, dtype)
        u1, _ = _solve(f, bc, h, dtype, zsplit="off")
        uo = oracle.solve(f, bc, h, "mean")
        assert rel_max(u, uo) < TOL[dtype], (dtype, bc, shape)
        assert rel_max(u1, uo) < TOL[dtype], (dtype, bc, shape)


@pytest.mark.parametrize("gauge", ["mean", "pin", "pin_raw"])
def test_separate_y_transforms_near_singular_batch(gauge):
    """Double columns too close to singular to split (long z, Neumann), per batch entry."""
    from gpu_util import banner, rel_max
    rng = np.random.default_rng(53)
    shape, bc = (700, 4, 288), "NNPPNN"
    h = (1.0 / 64, 1.0 / 64, 1.0 / 64)
    f = rng.standard_normal((2,) + shape) + np.array([0.5, -1.0])[:, None, None, None]
    banner(f"lines near-singular {gauge} {shape}")
    u, plan = _solve(f, bc, h, "f64", gauge=gauge, batch=2)
    _, means, _ = plan.last_info()
    for b in range(2):
        assert rel_max(u[b], oracle.solve(f[b], bc, h, gauge)) < 1e-12, (b, gauge)
        expect = f[b].mean() if gauge != "pin_raw" else 0.0
        assert abs(means[b] - expect) < 1e-13 * max(1.0, abs(f[b]).max())
