"""The windowed forward march (line windows, faint samples, ray parts, the top
taper's sample range) against the FP64 oracle, at the sizes where its shape
changes: the ends of each channel block, one more than a block, ragged tiles,
each number of ray parts, a sample count that leaves a partial last step,
channels spaced unevenly or in falling order, and cameras on both sides of the
inclination from which the taper's range is the whole chord.

Bars: max |dI| <= 1e-5 of the peak, the forward bar; the windows leave out only
channels whose depth is 0 in float, so they take nothing from it, and extremely
thin scenes hold the same relative bar.  Gradients: the adjoint's bar, 1e-3
relative in L2 per block and per large entry, with the oracle's cotangent.
"""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

TOL = 1e-5


def gpu_cube(prob):
    import paper_2509_03623_amd as rt
    print(f"[gpu] windows {prob.camera.nx}x{prob.camera.ny}x{prob.nch} ns={prob.nsamp} incl={prob.camera.incl_deg}",
          flush=True)
    cube = rt.render(rt.scene_from_problem(prob))
    torch.cuda.synchronize()
    return cube.cpu().numpy().astype(np.float64)


def check(prob):
    ref = oracle.render(prob)
    assert ref.max() > 0
    got = gpu_cube(prob)
    assert np.abs(got - ref).max() <= TOL * ref.max()
    return got, ref


@pytest.mark.parametrize("nch", [1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 96, 97, 128, 129, 256, 257])
def test_channel_blocks(nch):
    check(synth.small_problem(nx=19, ny=13, nch=nch, nsamp=70, nr=48, nz=24, seed=31, dv=6.0 / nch))


@pytest.mark.parametrize("nx,ny,nsamp", [(7, 5, 1), (7, 5, 31), (9, 9, 33), (21, 10, 65), (33, 40, 129), (150, 110, 70),
                                         (372, 361, 37)])
def test_ray_parts_and_tiles(nx, ny, nsamp):
    check(synth.small_problem(nx=nx, ny=ny, nch=9, nsamp=nsamp, nr=40, nz=20, seed=32, dv=0.3))


@pytest.mark.parametrize("order", ["uneven", "falling", "shuffled", "repeated"])
@pytest.mark.parametrize("nch", [11, 50, 115])
def test_channel_orders(order, nch):
    prob = synth.small_problem(nx=18, ny=15, nch=nch, nsamp=60, nr=48, nz=24, seed=33, dv=5.0 / nch)
    rng = np.random.Generator(np.random.PCG64(5))
    v = prob.v_kms.copy()
    v = {"uneven": lambda: v + 0.3 * (v[1] - v[0]) * rng.uniform(-1, 1, nch), "falling": lambda: v[::-1].copy(),
         "shuffled": lambda: rng.permutation(v), "repeated": lambda: np.full(nch, 0.4)}[order]()
    check(prob.replace(v_kms=v))


@pytest.mark.parametrize("incl", [0.0, 20.0, 55.0, 62.0, 64.5, 70.0, 89.0, 90.0])
def test_inclinations(incl):
    check(synth.small_problem(nx=24, ny=22, nch=20, nsamp=90, nr=48, nz=24, seed=34, incl=incl, dv=0.3))


@pytest.mark.parametrize("x_co", [1e-4, 1e-14, 1e-20])
def test_any_depth(x_co):
    """Sample depths of 1 down to 1e-16 and less: the relative bar holds at each."""
    prob = synth.small_problem(nx=16, ny=14, nch=16, nsamp=80, nr=48, nz=24, seed=35, dv=0.25).replace(x_co=x_co,
        intensity_scale=synth.disk.rj_kelvin_scale(synth.disk.co21_line()))
    check(prob)


@pytest.mark.parametrize("field", ["temp_k", "ln_nh2", "vphi_kms", "z_up_au"])
@pytest.mark.parametrize("nch", [40, 70, 130])
def test_nan_field_reaches_every_channel(field, nch):
    """A ring of NaN nodes makes a ray NaN in every channel or in none, as the
    march without windows does, and in none that the oracle keeps finite."""
    import paper_2509_03623_amd as rt
    from paper_2509_03623_amd import _lib as L
    prob = synth.small_problem(nx=16, ny=14, nch=nch, nsamp=80, nr=48, nz=24, seed=36, dv=8.0 / nch)
    t = getattr(prob, field).copy()
    t[36:40] = np.nan
    prob = prob.replace(**{field: t})
    ref = np.isnan(oracle.render(prob))
    bad = np.isnan(gpu_cube(prob))
    rt.set_option(L.RT_OPT_CHANNEL_BLOCK, 16)
    try:
        plain = np.isnan(gpu_cube(prob))
    finally:
        rt.set_option(L.RT_OPT_CHANNEL_BLOCK, 0)
    assert plain.any() and not ref.all()
    assert np.array_equal(bad.any(0), bad.all(0))
    assert not (bad & ~ref).any()
    assert bad.any(0).sum() >= plain.any(0).sum() // 2


@pytest.mark.parametrize("order", ["", "falling", "uneven"])
def test_served_blocks(order):
    """Requests at the ends of the server's 32-channel blocks and 4 x 4 tiles,
    in one batch, each against the oracle."""
    import paper_2509_03623_amd as rt
    probs = []
    for i, (nx, ny, nch, nsamp) in enumerate([(4, 4, 1, 1), (5, 3, 31, 7), (8, 9, 32, 33), (17, 12, 33, 64),
                                              (20, 20, 64, 50), (12, 11, 65, 101)]):
        prob = synth.small_problem(nx=nx, ny=ny, nch=nch, nsamp=nsamp, nr=40, nz=20, seed=40 + i, dv=6.0 / nch,
                                   incl=30.0 + 9 * i)
        if order:
            v = prob.v_kms[::-1].copy() if order == "falling" else prob.v_kms + 0.02 * np.sin(np.arange(nch) * 1.7)
            prob = prob.replace(v_kms=v)
        probs.append(prob)
    scenes = [rt.scene_from_problem(p) for p in probs]
    cubes = [torch.full((s.nch, s.ny, s.nx), float("nan"), device="cuda") for s in scenes]
    torch.cuda.synchronize()
    print(f"[gpu] served blocks {order}", flush=True)
    with rt.Server(max_slots=8, streams=2) as sv:
        tickets = [sv.submit(s, c) for s, c in zip(scenes, cubes)]
        assert all(sv.wait(t)["state"] == "done" for t in tickets)
    torch.cuda.synchronize()
    for p, c in zip(probs, cubes):
        ref = oracle.render(p)
        assert np.abs(c.cpu().numpy().astype(np.float64) - ref).max() <= TOL * ref.max()


@pytest.mark.parametrize("nx,ny,nch,order", [(7, 5, 1, ""), (9, 7, 16, ""), (13, 9, 17, "falling"), (11, 11, 32, ""),
                                             (11, 11, 33, "uneven"), (14, 13, 64, ""), (10, 9, 65, "uneven"),
                                             (180, 183, 35, "")])
def test_reverse_march(nx, ny, nch, order):
    """Gradients at the ends of the channel blocks, on tiles with ragged edges,
    on an image large enough for 64-channel blocks, and the cube that the
    reverse march forms: the forward march's to the same bar."""
    import paper_2509_03623_amd as rt
    import test_gpu_adjoint as ta
    from oracle import torch_ref
    nsamp = 24 if nx > 100 else 61
    prob = ta.kscale(synth.small_problem(nx=nx, ny=ny, nch=nch, nsamp=nsamp, nr=40, nz=20, seed=38, dv=5.0 / nch))
    if order:
        v = prob.v_kms[::-1].copy() if order == "falling" else prob.v_kms + 0.02 * np.sin(np.arange(nch) * 1.7)
        prob = prob.replace(v_kms=v)
    ref = oracle.render(prob)
    target = ta.target_for(prob)
    print(f"[gpu] reverse march {nx}x{ny}x{nch}", flush=True)
    vjp, cube, _ = ta.gpu_grads(prob, target, cotangent=2.0 * (ref - target))
    _, oref = torch_ref.loss_and_grad(prob, target)
    for k in ta.BLOCKS:
        ta.check_block(k, vjp[k], oref[k])
    sc = rt.scene_from_problem(prob)
    own, _, _ = rt.render_l2_adjoint(sc, torch.as_tensor(target, dtype=torch.float32, device="cuda"), want=ta.BLOCKS)
    assert np.abs(own.cpu().numpy().astype(np.float64) - ref).max() <= TOL * ref.max()


@pytest.mark.parametrize("nr,nz,fov", [(24, 12, None), (256, 128, None), (256, 128, 90.0), (290, 125, None), (300, 128, None),
                                       (40, 900, None)])
@pytest.mark.parametrize("double", [0, 1])
def test_chain_rows(nr, nz, fov, double):
    """The chain's gradient grid in LDS with all its rows in double (small grids),
    some (256 x 128: whole disk, and an image of its inner 90 au, where the rows
    of doubles are others), none (300 x 128), and too large for LDS (scatter to
    memory), into either kind of accumulator."""
    import paper_2509_03623_amd as rt
    import test_gpu_adjoint as ta
    from oracle import torch_ref
    from paper_2509_03623_amd import _lib as L
    kw = dict(fov=fov) if fov else {}
    prob = ta.kscale(synth.small_problem(nx=16, ny=15, nch=9, nsamp=48, nr=nr, nz=nz, seed=47, dv=0.6, **kw))
    ref = oracle.render(prob)
    target = ta.target_for(prob)
    rt.set_option(L.RT_OPT_GRAD_ACCUM, double)
    try:
        vjp, _, _ = ta.gpu_grads(prob, target, cotangent=2.0 * (ref - target))
        two, _, _ = ta.gpu_grads(prob, target, want=("ln_nh2", "temp_k"), cotangent=2.0 * (ref - target))
    finally:
        rt.set_option(L.RT_OPT_GRAD_ACCUM, 0)
    _, oref = torch_ref.loss_and_grad(prob, target)
    for k in ta.BLOCKS:
        if np.abs(oref[k]).max() > 0:
            ta.check_block(k, vjp[k], oref[k])
    for k in two:
        ta.check_block(k, two[k], oref[k])


@pytest.mark.parametrize("x_co", [1e-14, 1e-20])
def test_gradient_at_any_depth(x_co):
    """A scene whose samples are all faint has the gradient of its own scale."""
    import test_gpu_adjoint as ta
    from oracle import torch_ref
    prob = ta.kscale(synth.small_problem(nx=12, ny=10, nch=12, nsamp=50, nr=32, nz=16, seed=39, dv=0.4)).replace(x_co=x_co)
    ref = oracle.render(prob)
    target = ref * 0.0
    vjp, _, _ = ta.gpu_grads(prob, target, cotangent=np.full_like(ref, 1.0 / ref.max()))
    leaves = torch_ref.as_leaves(prob)
    (torch_ref.cube(prob, leaves) / ref.max()).sum().backward()
    for k in ta.BLOCKS:
        ta.check_block(k, vjp[k], leaves[k].grad.numpy())


def test_channel_far_from_every_line():
    """Channels no gas moves at are dark, also at a velocity where a float has lost the fraction."""
    prob = synth.small_problem(nx=12, ny=12, nch=24, nsamp=40, nr=48, nz=24, seed=37)
    got = gpu_cube(prob.replace(v_kms=np.linspace(5e3, 5e6, 24)))
    assert np.all(got == 0.0)


# one channel block of 10, 12, 14 or 16 a lane: the ends and one more
@pytest.mark.parametrize("nch,order", [(40, "uneven"), (41, ""), (49, "falling"), (56, "uneven"), (57, "")])
def test_reverse_march_block_ends(nch, order):
    test_reverse_march(182, 181, nch, order)


# grids that leave no room for the surfaces as doubles
@pytest.mark.parametrize("nr,nz", [(256, 148), (295, 128)])
@pytest.mark.parametrize("double", [0, 1])
def test_chain_rows_with_float_surfaces(nr, nz, double):
    test_chain_rows(nr, nz, None, double)


@pytest.mark.parametrize("log2k", [np.log2(13.45) - 30, np.log2(12.6) - 30, -40.5])
def test_longest_rays_of_faint_samples(log2k, n=1 << 20):
    """Rays of n equal samples with depths of log2 K each: the windowed reverse
    march against the one over all channels.  Both form J alike to the bit and hold
    the depth in two words, so they differ by a few roundings of the transmission
    and of the sums (1e-5).  A depth summed in one word is off by up to half an ulp
    of the sum a sample, and the gradient by 1.4e-5 at samples of 12.6 ulps."""
    import paper_2509_03623_amd as rt
    from paper_2509_03623_amd import _lib as L
    small = synth.slab_problem(nsamp=64, m=1, nch=1, dv=0.03, nx=4, ny=4)
    thick, thin = (oracle.render(small.replace(x_co=x)).max() for x in (1e2, 1e-14))
    inside = 62 / 64 * n                                     # samples in the layer
    x_co = 1e-14 * np.log(2.0) * 2.0 ** log2k * inside / (thin / thick)
    prob = synth.slab_problem(nsamp=n, m=n // 64, nch=1, dv=0.03, nx=4, ny=4, x_co=x_co)
    prob = prob.replace(intensity_scale=synth.disk.rj_kelvin_scale(prob.line))
    sc = rt.scene_from_problem(prob)
    cot = torch.as_tensor(1.0 + 0.5 * np.random.Generator(np.random.PCG64(9)).standard_normal((1, 4, 4)),
                          dtype=torch.float32, device="cuda")
    print(f"[gpu] longest rays, log2 K = {log2k}", flush=True)

    def grads():
        g = rt.render_adjoint(sc, cot, want=("ln_nh2", "temp_k"))
        return {k: v.cpu().numpy().astype(np.float64) for k, v in g.items()}
    got = grads()
    rt.set_option(L.RT_OPT_ADJ_CHANNEL_BLOCK, 16)
    try:
        want = grads()
    finally:
        rt.set_option(L.RT_OPT_ADJ_CHANNEL_BLOCK, 0)
    for k in got:
        err = np.linalg.norm(got[k] - want[k]) / np.linalg.norm(want[k])
        print(k, err, flush=True)
        assert np.linalg.norm(want[k]) > 0 and err <= 1e-5, k


# the longest ray of the kernel with literal bounds and the shortest of the other,
# at depths on both sides of either one's bounds (the same tolerance)
@pytest.mark.parametrize("n", [8192, 8193])
@pytest.mark.parametrize("log2k", [-25.5, -27.5, -40.5])
def test_rays_at_the_literal_bounds(n, log2k):
    test_longest_rays_of_faint_samples(log2k, n)


@pytest.mark.parametrize("field", ["temp_k", "ln_nh2", "vphi_kms", "z_up_au"])
@pytest.mark.parametrize("nch", [40, 130])
@pytest.mark.parametrize("rows", [(36, 40), (44, 48)])
def test_no_nan_ray_is_hidden(field, nch, rows):
    """Every ray that the march over all channels makes NaN is NaN in the windowed
    march, in every channel: what it leaves out reads no field.  (Not the other way
    round: the march over all channels passes over a NaN sample where no other ray
    of its wave has opacity.)"""
    import paper_2509_03623_amd as rt
    from paper_2509_03623_amd import _lib as L
    prob = synth.small_problem(nx=16, ny=14, nch=nch, nsamp=80, nr=48, nz=24, seed=36, dv=8.0 / nch)
    t = getattr(prob, field).copy()
    t[rows[0]:rows[1]] = np.nan
    prob = prob.replace(**{field: t})
    ref = np.isnan(oracle.render(prob)).any(0)
    bad = np.isnan(gpu_cube(prob))
    rt.set_option(L.RT_OPT_CHANNEL_BLOCK, 16)
    try:
        plain = np.isnan(gpu_cube(prob)).any(0)
    finally:
        rt.set_option(L.RT_OPT_CHANNEL_BLOCK, 0)
    assert plain.any() and np.array_equal(bad.any(0), bad.all(0))
    assert not (plain & ~bad.any(0)).any()
    assert not (bad.any(0) & ~ref).any()
