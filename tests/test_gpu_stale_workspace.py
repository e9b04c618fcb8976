"""Solves on a workspace filled with NaN bytes and on one filled with zeros give the
same bits (no kernel reads workspace that the solve did not write first), for the
kernel forms by line length, layout and z faces."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5, "f32_refined": 1e-12}

# shape, dtypes, layout: general x kernels and the single march on short lines; rows
# shared by two and four wavefronts (exact-count and general); marches on lines of 384,
# 512, up to 1024 (planes shared by two wavefronts), 1536 and 2048, z whole chunks and
# ragged; the split and the segmented march; y transforms by themselves; z in chunks
CASES = [((9, 12, 18), "f64 f32", "off"), ((16, 48, 36), "f64 f32", "off"), ((3, 8, 768), "f64 f32 f32_refined", "auto"),
         ((3, 9, 576), "f64 f32 f32_refined", "auto"), ((3, 8, 1024), "f64 f32", "auto"), ((3, 6, 1152), "f64 f32 f32_refined", "auto"),
         ((24, 384, 6), "f64 f32 f32_refined", "off"), ((25, 384, 6), "f64 f32 f32_refined", "off"),
         ((16, 512, 6), "f64 f32 f32_refined", "off"), ((17, 486, 6), "f64 f32 f32_refined", "off"),
         ((16, 1024, 6), "f64 f32 f32_refined", "off"), ((9, 972, 4), "f64 f32 f32_refined", "off"),
         ((8, 1536, 4), "f64 f32", "off"), ((7, 1152, 4), "f64 f32", "off"), ((8, 2048, 4), "f64 f32", "off"),
         ((5, 1944, 4), "f64 f32", "off"), ((32, 1024, 6), "f64 f32 f32_refined", "on"), ((48, 384, 4), "f64 f32", "seg"),
         ((40, 768, 4), "f64 f32", "seg"), ((24, 8, 288), "f64 f32", "auto"), ((1025, 2, 288), "f64", "auto"),
         ((1025, 4, 8), "f64 f32", "auto"), ((200, 8, 12), "f64 f32", "auto"), ((33, 128, 64), "f64 f32", "auto")]


@pytest.mark.parametrize("bc", ["PPPPNN", "DDNNDN", "NNPPPP"])
@pytest.mark.parametrize("shape,dtypes,zsplit", CASES, ids=lambda v: str(v))
def test_workspace_contents_do_not_reach_the_result(shape, dtypes, zsplit, bc):
    import torch
    from paper_1909_05423_amd import Plan
    from gpu_util import banner, rel_max, to_dev
    if bc[4] == "P" and zsplit in ("on", "seg"):
        zsplit = "off"   # periodic z has one layout
    h = (1.0 / shape[2], 1.0 / shape[1], 1.0 / 64)
    f = np.random.default_rng(71).standard_normal(shape).astype(np.float32).astype(np.float64)
    for dtype in dtypes.split():
        banner(f"stale workspace {dtype} {bc} {shape} {zsplit}")
        us = []
        for fill in (255, 0):
            plan = Plan(shape, bc, h, dtype=dtype, zsplit=zsplit)
            plan.workspace.fill_(fill)
            u = plan.solve(to_dev(f[None], torch.float32 if dtype == "f32" else torch.float64))
            torch.cuda.synchronize()
            us.append(u[0].double().cpu().numpy())
        assert np.all(np.isfinite(us[0])), (dtype, bc, shape)
        # (the split and segmented marches add the zero mode's mean by atomics)
        if zsplit in ("on", "seg") and bc == "PPPPNN":
            assert rel_max(us[0], us[1]) < TOL[dtype]
        else:
            assert np.array_equal(us[0], us[1]), (dtype, bc, shape)
        if shape[0] < 1000:
            assert rel_max(us[0], oracle.solve(f, bc, h, "mean")) < TOL[dtype], (dtype, bc, shape)
