"""The points that the network kernels evaluate are the points that the march
reads, to the last one: both decide by a float taper that a differently rounded
position would put on the other side of 0.  Random views at sizes where some
samples lie within a rounding of the taper's edge, each render over scratch
memory filled with NaN: an output that is read and was not written shows.
"""
import numpy as np
import pytest
import torch

import synth
from test_gpu_missed_rays import poison_pool

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp32,n,nsamp,views", [(False, 256, 512, 24), (True, 96, 512, 12)])
def test_every_output_read_was_written(fp32, n, nsamp, views):
    import paper_2509_03623_amd as rt
    rng = np.random.Generator(np.random.PCG64(77))
    for i in range(views):
        nr, nz = int(rng.integers(20, 200)), int(rng.integers(10, 100))
        prob = synth.small_problem(nx=n, ny=n, nch=2, nsamp=nsamp, nr=nr, nz=nz, seed=60 + i, dv=1.0,
                                   incl=float(rng.uniform(5.0, 80.0)), pa=float(rng.uniform(-180.0, 180.0)), mlp_seed=4)
        sc = rt.scene_from_problem(prob, mlp_precision=rt.RT_MLP_FP32 if fp32 else rt.RT_MLP_BF16)
        print(f"[gpu] network points view {i} {nr}x{nz} incl={prob.camera.incl_deg:.1f} fp32={fp32}", flush=True)
        poison_pool(16 * n * n * nsamp)
        cube = rt.render(sc)
        assert bool(torch.isfinite(cube).all()) and float(cube.max()) > 0.0
