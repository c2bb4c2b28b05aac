"""Rays that miss the grid share waves with rays that meet it: they stay exactly
dark whatever stands where they would cross the grid's midplane (nodes no ray of
theirs samples, network outputs nobody wrote), and the rays that meet the grid
stay what the FP64 oracle makes them.
"""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


def poison_pool(nbytes):
    """NaN in the device memory that the library's next allocations of nbytes
    to nbytes + 2 MB on this stream get: blocks of those sizes, filled and
    handed back to the stream-ordered pool that its scratch comes from."""
    from paper_2509_03623_amd import _lib as L
    hip, st = L.lib(), C.c_void_p(torch.cuda.current_stream().cuda_stream)
    blocks = []
    for more in (1 << 18, 1 << 19, 1 << 20, 2 << 20):
        p = C.c_void_p()
        n = (nbytes + more + 255) // 256 * 256
        assert hip.hipMallocAsync(C.byref(p), C.c_size_t(n), st) == 0
        assert hip.hipMemsetD32Async(p, C.c_int(0x7FC00000), C.c_size_t(n // 4), st) == 0
        blocks.append(p)
    for p in blocks:
        assert hip.hipFreeAsync(p, st) == 0


def inclined(**kw):
    """An image whose rays miss the grid at its top and bottom, inside the grid's radius."""
    args = dict(nx=18, ny=19, nch=24, nsamp=40, nr=48, nz=24, seed=51, dv=0.4, incl=55.0)
    args.update(kw)
    return synth.small_problem(**args)


def check_dark(prob, cube, live):
    ref = oracle.render(prob)
    assert 0 < live.sum() < live.size
    assert np.all(ref[:, ~live] == 0.0)
    assert np.all(cube[:, ~live] == 0.0)
    return ref


@pytest.mark.parametrize("field,bad", [("temp_k", np.nan), ("ln_nh2", np.nan), ("ln_nh2", np.inf), ("vphi_kms", np.nan)])
@pytest.mark.parametrize("nch,order", [(24, ""), (70, ""), (24, "uneven")])
def test_bad_nodes_in_the_outer_rows(field, bad, nch, order):
    import paper_2509_03623_amd as rt
    prob = inclined(nch=nch, dv=9.6 / nch)
    t = getattr(prob, field).copy()
    t[44:] = bad
    prob = prob.replace(**{field: t})
    if order:
        prob = prob.replace(v_kms=prob.v_kms + 0.02 * np.sin(np.arange(nch) * 1.7))
    sc = rt.scene_from_problem(prob)
    print(f"[gpu] missed rays {field} {bad} {nch} {order}", flush=True)
    cube = rt.render(sc).cpu().numpy().astype(np.float64)
    ref = check_dark(prob, cube, sc.live_mask())
    finite = np.isfinite(ref).all(0)
    assert finite.any()
    assert np.abs(cube - ref)[:, finite].max() <= 1e-5 * ref[:, finite].max()


@pytest.mark.parametrize("fp32", [True, False])
@pytest.mark.parametrize("incl", [30.0, 55.0, 80.0])
def test_network_outputs_nobody_wrote(incl, fp32):
    import paper_2509_03623_amd as rt
    prob = inclined(nx=35, ny=38, nsamp=64, incl=incl, mlp_seed=4)
    sc = rt.scene_from_problem(prob, mlp_precision=rt.RT_MLP_FP32 if fp32 else rt.RT_MLP_BF16)
    live = sc.live_mask()
    print(f"[gpu] missed rays, network incl={incl} fp32={fp32}", flush=True)
    for _ in range(2):
        poison_pool(16 * sc.nx * sc.ny * sc.nsamp)
        cube = rt.render(sc).cpu().numpy().astype(np.float64)
        ref = check_dark(prob, cube, live)
        assert np.isfinite(cube).all()
        if fp32:
            assert np.abs(cube - ref).max() <= 1e-5 * ref.max()
        else:
            assert np.linalg.norm(cube - ref) <= 1e-2 * np.linalg.norm(ref)


@pytest.mark.parametrize("order", ["", "uneven"])
def test_bad_nodes_in_a_served_batch(order):
    import paper_2509_03623_amd as rt
    probs = []
    for field, bad, nch in [("temp_k", np.nan, 24), ("ln_nh2", np.inf, 24), ("vphi_kms", np.nan, 40), ("", 0.0, 24)]:
        prob = inclined(nch=nch, dv=9.6 / nch)
        if field:
            t = getattr(prob, field).copy()
            t[44:] = bad
            prob = prob.replace(**{field: t})
        if order:
            prob = prob.replace(v_kms=prob.v_kms + 0.02 * np.sin(np.arange(nch) * 1.7))
        probs.append(prob)
    scenes = [rt.scene_from_problem(p) for p in probs]
    cubes = [torch.full((s.nch, s.ny, s.nx), float("nan"), device="cuda") for s in scenes]
    torch.cuda.synchronize()
    print(f"[gpu] missed rays, served {order}", flush=True)
    with rt.Server(max_slots=8, streams=2) as sv:
        tickets = [sv.submit(s, c) for s, c in zip(scenes, cubes)]
        assert all(sv.wait(t)["state"] == "done" for t in tickets)
    torch.cuda.synchronize()
    for p, s, c in zip(probs, scenes, cubes):
        cube = c.cpu().numpy().astype(np.float64)
        ref = check_dark(p, cube, s.live_mask())
        finite = np.isfinite(ref).all(0)
        assert np.abs(cube - ref)[:, finite].max() <= 1e-5 * ref[:, finite].max()
