"""How many slices a batch holds (host only): the budget pays for a slice's grids
T, ext and yh, and for the parts of shared spreading tiles only where they
outgrow T, whose memory they use while it is dead.
"""

import ctypes

import numpy as np
import pytest


@pytest.mark.parametrize("n,angles,slices", [(512, 720, 16), (640, 600, 20), (1024, 901, 8)])
def test_parts_do_not_cut_batches_short(n, angles, slices):
    from paper_2304_12934_amd._lib import NR_OK, NrNufft, NrSlice, lib
    arr = (NrSlice * slices)(*[NrSlice(n, n, angles, z * n * n, z * angles * n, 0) for z in range(slices)])
    ang = np.linspace(0, np.pi, angles, endpoint=False)
    h = ctypes.c_void_p()
    assert lib().nr_plan_create(arr, slices, ang.ctypes.data_as(ctypes.POINTER(ctypes.c_double)),
                                ctypes.byref(NrNufft(2.0, 7, 0.0)), ctypes.byref(h)) == NR_OK
    info = (ctypes.c_int64 * 8)()
    assert lib().nr_plan_info(h, 0, info, 8) == NR_OK
    lib().nr_plan_destroy(h)
    G = 2 * n
    # G/2 + 1 grid rows and 8 for the halo, G columns and 8; rows of T in fours
    grids = 8 * ((n + 9) * (G + 8) + angles * (n // 2 + 1) + (n + 4) // 4 * 4 * n)
    # the default budget of 160 MiB holds this many slices' grids; parts that
    # outgrow T (sixteen slices of 512^2) still fit beside them here
    assert info[5] == min(slices, (160 << 20) // grids)
