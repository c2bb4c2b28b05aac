"""Which grids the gradient's chain passes keep in LDS: every grid that fits as
floats with its two surface vectors beside it (the scatter to memory is for
larger ones).  Host-side, no GPU work."""
import ctypes as C

import pytest

from paper_2509_03623_amd import _lib as L

# 160 KB less the partition table's 511 records of 16 bytes and a kilobyte
ROOM = 160 * 1024 - 16 * 511 - 1024


def fits(nr, nz):
    f = L.lib()["_ZN2rt14chain_lds_fitsEii"]
    f.restype = C.c_bool
    return bool(f(C.c_int(nr), C.c_int(nz)))


@pytest.mark.parametrize("nr,nz", [(256, 128), (256, 148), (512, 73), (384, 98), (128, 300), (200, 190), (295, 128),
                                   (300, 126), (256, 149), (300, 128), (2, 19000), (19000, 2)])
def test_grids_that_fit_as_floats(nr, nz):
    assert fits(nr, nz) == (4 * nr * nz + 8 * nr <= ROOM)
