"""The windowed 3-D march (line windows, ray parts, the sample range of the
polar wedge) against the FP64 oracle where its shape changes: the ends of the
channel blocks and one more, ragged tiles, partial last steps, uneven and
falling channels, and inclinations on both sides of the one from which the
wedge's range is the whole chord, with grids that reach the poles or lie on one
side of the midplane.

Bar: max |dI| <= 1e-5 of the peak, the 3-D march's own bar.
"""
import math
from dataclasses import replace

import numpy as np
import pytest
import torch

import oracle
from synth import disk3d as S3

pytestmark = pytest.mark.gpu

TOL = 1e-5


def check(prob):
    import paper_2509_03623_amd as rt
    ref = oracle.render3(prob)
    print(f"[gpu] windows3 {prob.camera.nx}x{prob.camera.ny}x{len(prob.v_kms)} ns={prob.nsamp} "
          f"incl={prob.camera.incl_deg}", flush=True)
    got = rt.render3d(rt.scene3d_from_problem(prob))
    torch.cuda.synchronize()
    assert ref.max() > 0
    assert np.abs(got.cpu().numpy().astype(np.float64) - ref).max() <= TOL * ref.max()


def problem(nx=17, ny=13, nch=9, nsamp=70, incl=38.0, dv=None, seed=61):
    return S3.make_problem3(S3.Grid3Spec(26, 14, 18), seed=seed, nx=nx, ny=ny, nch=nch, dv=dv or 5.0 / nch,
                            nsamp=nsamp, incl=incl, pa=25.0)


@pytest.mark.parametrize("nch", [1, 16, 17, 32, 33, 48, 49, 64, 65, 96, 97, 128, 129, 257])
def test_channel_blocks(nch):
    check(problem(nch=nch))


@pytest.mark.parametrize("nx,ny,nsamp", [(5, 3, 1), (9, 9, 33), (21, 10, 65), (33, 18, 129), (130, 97, 35)])
def test_ray_parts_and_tiles(nx, ny, nsamp):
    check(problem(nx=nx, ny=ny, nsamp=nsamp))


@pytest.mark.parametrize("order", ["uneven", "falling", "repeated"])
@pytest.mark.parametrize("nch", [11, 70])
def test_channel_orders(order, nch):
    prob = problem(nch=nch)
    v = prob.v_kms.copy()
    rng = np.random.Generator(np.random.PCG64(5))
    v = {"uneven": lambda: v + 0.3 * (v[1] - v[0]) * rng.uniform(-1, 1, nch), "falling": lambda: v[::-1].copy(),
         "repeated": lambda: np.full(nch, 0.4)}[order]()
    check(replace(prob, v_kms=v))


@pytest.mark.parametrize("incl", [0.0, 20.0, 60.0, 75.0, 90.0, 120.0, 180.0])
@pytest.mark.parametrize("wedge", ["disk", "poles", "above", "thin"])
def test_polar_wedges(incl, wedge):
    prob = problem(incl=incl)
    lo, hi = {"disk": (None, None), "poles": (0.0, math.pi), "above": (0.9, 1.3),
              "thin": (0.5 * math.pi - 0.25, 0.5 * math.pi + 0.25)}[wedge]
    if lo is not None:
        prob = replace(prob, grid=replace(prob.grid, th_min=lo, th_max=hi))
    check(prob)


@pytest.mark.parametrize("half,nsamp", [(1e-4, 1 << 17), (1e-3, 1 << 19)])
def test_thinnest_wedges(half, nsamp):
    """A wedge whose crossing is a few samples of the ray: the windowed march finds
    every crossing that the march over the whole chord does (bar: the march's own)."""
    import paper_2509_03623_amd as rt
    from paper_2509_03623_amd import _lib as L
    grid = replace(S3.Grid3Spec(20, 6, 8), th_min=0.5 * math.pi - half, th_max=0.5 * math.pi + half)
    n = 40 if nsamp < 1 << 18 else 20
    prob = S3.uniform_problem3(grid, nx=n, ny=n, nch=3, nsamp=nsamp, incl=55.0, pa=30.0, fov_au=2.0 * grid.r_max_au)
    sc = rt.scene3d_from_problem(prob)
    print(f"[gpu] windows3 wedge {half} ns={nsamp}", flush=True)
    got = rt.render3d(sc)
    rt.set_option(L.RT_OPT_CHANNEL_BLOCK, 8)
    try:
        want = rt.render3d(sc)
    finally:
        rt.set_option(L.RT_OPT_CHANNEL_BLOCK, 0)
    peak = float(want.max())
    assert peak > 0 and float((got - want).abs().max()) <= TOL * peak
