"""Beam convolution (rt_beam_convolve) over every support radius and the
boundaries of its tiles: rows of whole, aligned float4 and others, one pixel
more or less than a tile, and images narrower than the halo, against the FP64
oracle.  Bar: max |d| <= 1e-5 of the peak, the convolution's own."""
import numpy as np
import pytest
import torch

from oracle import beam as OB

pytestmark = pytest.mark.gpu

TOL = 1e-5


def check(shape, beam, seed, shift=0):
    import paper_2509_03623_amd as rt
    rng = np.random.Generator(np.random.PCG64(seed))
    c = (rng.random(shape) * (rng.random(shape) > 0.7)).astype(np.float32)
    buf = torch.zeros(c.size + shift, device="cuda")
    x = buf[shift:].view(shape)                # shift: an address that is no multiple of 16
    x.copy_(torch.tensor(c))
    print(f"[gpu] beam tiles {shape} {beam} shift {shift}", flush=True)
    got = rt.beam_convolve(x, *beam)
    torch.cuda.synchronize()
    ref = OB.convolve(c.astype(np.float64), *beam)
    assert np.abs(got.cpu().numpy() - ref).max() <= TOL * np.abs(ref).max()


@pytest.mark.parametrize("radius", range(1, 25))
def test_every_radius(radius):
    bmaj = 2.3548 * (radius - 0.4) / 3.0
    for shape in ((1, 70, 68), (2, 13, 67)):
        check(shape, (bmaj, 0.8 * bmaj, 25.0), radius)


@pytest.mark.parametrize("ny,nx", [(63, 64), (64, 60), (65, 65), (1, 129), (130, 1), (3, 4), (128, 132)])
@pytest.mark.parametrize("shift", [0, 1])
def test_tile_edges(ny, nx, shift):
    check((2, ny, nx), (5.0, 3.0, -40.0), 30, shift)


# one and two rows a lane: 256 tiles and one more, at the smallest radius with both forms and the largest
@pytest.mark.parametrize("radius", [7, 8, 24])
@pytest.mark.parametrize("nch", [256, 257])
@pytest.mark.parametrize("ny,nx", [(31, 64), (33, 61)])
def test_few_tiles_and_one_more(radius, nch, ny, nx):
    check((nch, ny, nx), (2.3548 * (radius - 0.4) / 3.0, 3.0, -40.0), 31)
