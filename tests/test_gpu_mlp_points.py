"""Which points the network kernels take: the forward evaluates the points the
march reads (rays that meet the grid, inside its taper), in queues of 64 per
wave, and the backward the points whose dL/do counts.  Sizes around a queue's
64 points and a tile's edges, images mostly beyond the grid, and cotangents of
any scale.  Bars as in the network's own tests: FP32 cube 1e-5 of the peak and
gradients 1e-3 in L2; BF16 cube 1e-2 in L2 and gradient cosine 0.99.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from oracle import torch_ref

pytestmark = pytest.mark.gpu


def problem(**kw):
    args = dict(nx=16, ny=14, nch=8, nsamp=48, nr=40, nz=20, seed=6, dv=0.3, mlp_seed=4)
    args.update(kw)
    prob = synth.small_problem(**args)
    return prob.replace(intensity_scale=synth.disk.rj_kelvin_scale(prob.line))


def both(prob, fp32, cot):
    import paper_2509_03623_amd as rt
    print(f"[gpu] network points {prob.camera.nx}x{prob.camera.ny} ns={prob.nsamp} fov={prob.camera.fov_au:.0f} "
          f"fp32={fp32}", flush=True)
    sc = rt.scene_from_problem(prob, mlp_precision=rt.RT_MLP_FP32 if fp32 else rt.RT_MLP_BF16)
    cube = rt.render(sc)
    g = rt.render_adjoint(sc, torch.as_tensor(np.ascontiguousarray(cot, np.float32), device="cuda"),
                          want=("temp_k", "mlp_w"))
    torch.cuda.synchronize()
    return cube.cpu().numpy().astype(np.float64), {k: v.cpu().numpy().astype(np.float64) for k, v in g.items()}


@pytest.mark.parametrize("fp32", [True, False])
@pytest.mark.parametrize("kw", [dict(nx=3, ny=3, nsamp=7), dict(nx=8, ny=8, nsamp=1), dict(nx=9, ny=7, nsamp=65),
                                dict(nx=16, ny=16, nsamp=40, fov=6000.0), dict(nx=33, ny=5, nsamp=31, incl=80.0)])
def test_sizes(kw, fp32):
    prob = problem(**kw)
    ref = oracle.render(prob)
    leaves = torch_ref.as_leaves(prob)
    rng = np.random.Generator(np.random.PCG64(3))
    cot = 1.0 + 0.5 * rng.standard_normal(ref.shape)
    (torch_ref.cube(prob, leaves) * torch.tensor(cot)).sum().backward()
    cube, g = both(prob, fp32, cot)
    assert ref.max() > 0
    if fp32:
        assert np.abs(cube - ref).max() <= 1e-5 * ref.max()
    else:
        assert np.linalg.norm(cube - ref) <= 1e-2 * np.linalg.norm(ref)
    for k, v in g.items():
        r = leaves[k].grad.numpy().ravel()
        if fp32:
            assert np.linalg.norm(v.ravel() - r) <= 1e-3 * np.linalg.norm(r), k
        else:
            assert np.dot(v.ravel(), r) >= 0.99 * np.linalg.norm(v) * np.linalg.norm(r), k


@pytest.mark.parametrize("fp32", [True, False])
@pytest.mark.parametrize("power", [-60, 50])
def test_cotangent_scale(power, fp32):
    """A cotangent times a power of two gives the gradient times it: the points
    left out go with the largest dL/do (1e-5: the order of atomic additions)."""
    prob = problem()
    cot = np.random.Generator(np.random.PCG64(8)).standard_normal((8, 14, 16))
    _, a = both(prob, fp32, cot)
    _, b = both(prob, fp32, cot * 2.0 ** power)
    for k in a:
        scale = np.abs(a[k]).max()
        assert scale > 0
        assert np.abs(b[k] * 2.0 ** -power - a[k]).max() <= 1e-5 * scale


@pytest.mark.parametrize("fp32", [True, False])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_not_finite(bad, fp32):
    """A cotangent that is not finite at a bright voxel shows in the gradient."""
    prob = problem()
    ref = oracle.render(prob)
    cot = np.ones_like(ref)
    cot[np.unravel_index(int(np.argmax(ref)), ref.shape)] = bad
    _, g = both(prob, fp32, cot)
    assert not np.isfinite(g["mlp_w"]).all()


@pytest.mark.parametrize("fp32", [True, False])
def test_no_cotangent(fp32):
    _, g = both(problem(), fp32, np.zeros((8, 14, 16)))
    assert np.all(g["mlp_w"] == 0.0) and np.all(g["temp_k"] == 0.0)


def tail_neuron_weights(seed, zt):
    """A network whose last neuron of every layer is silent (0 in float) below
    zt of the grid's height and of order 1 above, and acts on the temperature."""
    from synth.mlp import MLP_DEPTH, MLP_WIDTH, layer_shapes, make_mlp_weights
    flat = make_mlp_weights(seed)
    n, off, parts = MLP_WIDTH - 1, 0, []
    for li, (o, i) in enumerate(layer_shapes()):
        W = flat[off:off + o * i].reshape(o, i).copy()
        b = flat[off + o * i:off + o * i + o].copy()
        off += o * i + o
        if li:
            W[:, n] = 0.0
        if li < MLP_DEPTH:
            W[n] = 0.0
            W[n, 48 if li == 0 else n] = (-2000.0, 1.0, 1.0, 0.02)[li]       # feature 48: cos(pi z)
            b[n] = (2000.0 * np.cos(np.pi * zt), -150.0, -150.0, 0.0)[li]
        else:
            W[2, n] = 0.01
        parts += [W.ravel(), b]
    return np.concatenate(parts).astype(np.float32), off - 3 - MLP_WIDTH + n


@pytest.mark.parametrize("fp32", [True, False])
def test_neuron_that_only_the_faintest_points_drive(fp32):
    """The gradient of a weight whose neuron is silent wherever dL/do is large
    comes whole from points with 1e-17 of the largest.  Bars: FP32 as above;
    BF16 0.3, its features' 2^-9 times the 2000 of the first weight being about
    a twentieth of the neuron's range."""
    prob = problem(nz=96)
    w, at = tail_neuron_weights(4, 0.8)
    prob = prob.replace(mlp_w=w)
    cot = np.ones((8, 14, 16))
    leaves = torch_ref.as_leaves(prob)
    torch_ref.cube(prob, leaves).sum().backward()
    ref = leaves["mlp_w"].grad.numpy()
    assert 1e-30 < abs(ref[at]) < 1e-15 * np.abs(ref).max()
    _, g = both(prob, fp32, cot)
    assert abs(g["mlp_w"].ravel()[at] - ref[at]) <= (1e-3 if fp32 else 0.3) * abs(ref[at])
