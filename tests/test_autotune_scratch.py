"""nr_autotune_scratch_bytes (host only): no candidate of the autotuner's search
space needs a larger workspace than the scratch it asks for, also where tiles
are cut into many items whose sums take scratch.
"""

import ctypes
import itertools

import numpy as np
import pytest


@pytest.mark.parametrize("n,angles,slices,own", [(512, 720, 16, {}), (1024, 901, 1, {}), (1024, 901, 3, {"streams": 8}),
                                                 (512, 1500, 2, {"chunk": 64, "batch_mb": 37})])
def test_every_candidate_fits_the_scratch(n, angles, slices, own):
    from paper_2304_12934_amd._lib import NR_OK, NrNufft, NrSlice, lib
    L = lib()
    arr = (NrSlice * slices)(*[NrSlice(n, n, angles, z * n * n, z * angles * n, 0) for z in range(slices)])
    ang = np.linspace(0, np.pi, angles, endpoint=False)
    h = ctypes.c_void_p()
    assert L.nr_plan_create(arr, slices, ang.ctypes.data_as(ctypes.POINTER(ctypes.c_double)),
                            ctypes.byref(NrNufft(2.0, 7, 0.0)), ctypes.byref(h)) == NR_OK
    for key, v in own.items():
        assert L.nr_plan_tune(h, key.encode(), v) == NR_OK
    before, need, ws, v = ctypes.c_size_t(), ctypes.c_size_t(), ctypes.c_size_t(), ctypes.c_int64()
    assert L.nr_plan_workspace_bytes(h, ctypes.byref(before)) == NR_OK
    assert L.nr_autotune_scratch_bytes(h, ctypes.byref(need)) == NR_OK
    # the plan keeps its setting and its layout
    assert L.nr_plan_workspace_bytes(h, ctypes.byref(ws)) == NR_OK and ws.value == before.value
    space = {"chunk": [256, 512, 1024], "batch_mb": [1, 160, 640, 1400, 2048], "streams": [1, 2, 3, 6]}
    for key, values in space.items():
        assert L.nr_plan_get_tune(h, key.encode(), ctypes.byref(v)) == NR_OK
        values.append(v.value)
    room = need.value - 4 * slices * (2 * n * n + angles * n) - 3 * 256
    for chunk, (tw, th), mb, streams in itertools.product(space["chunk"], ((64, 32), (32, 32), (64, 64), (128, 32)),
                                                          space["batch_mb"], space["streams"]):
        for key, v in (("chunk", chunk), ("tile_w", tw), ("tile_h", th), ("batch_mb", mb), ("streams", streams)):
            assert L.nr_plan_tune(h, key.encode(), v) == NR_OK
        assert L.nr_plan_workspace_bytes(h, ctypes.byref(ws)) == NR_OK
        assert ws.value <= room, (chunk, tw, th, mb, streams)
    L.nr_plan_destroy(h)
