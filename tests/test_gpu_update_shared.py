"""mbir_update where two of x, x_prev and y are one buffer (a caller that does
not keep x_prev passes x for it): y <- x' + beta (x' - x), x_prev <- x, x <- x'
in this order, element by element.

Tolerance: x' and y are a few float32 operations on values below 8 (2^-21 each
way, twice that through the momentum).
"""

import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("same", [("x", "xp"), ("x", "y"), ("xp", "y")])
@pytest.mark.parametrize("count", [5, 4099])
def test_update_of_shared_buffers(same, count):
    from paper_2304_12934_amd._lib import NR_MBIR_STATE_DOUBLES, NrMbir, check, lib
    print(f"case: mbir_update of {count} elements, {same[0]} = {same[1]}", flush=True)
    dev = torch.device("cuda", 0)
    rng = np.random.default_rng(count)
    host = {k: rng.standard_normal(count).astype(np.float32) for k in ("x", "xp", "y", "g")}
    host[same[1]] = host[same[0]]
    buf = {k: torch.as_tensor(v, device=dev) for k, v in host.items()}
    buf[same[1]] = buf[same[0]]
    state = torch.zeros(NR_MBIR_STATE_DOUBLES, dtype=torch.float64, device=dev)
    state[0] = 5.0
    params = NrMbir(0.25, 0, 0, 0)
    p = {k: ctypes.c_void_p(v.data_ptr()) for k, v in buf.items()}
    check(lib().mbir_update(ctypes.byref(params), p["x"], p["xp"], p["y"], p["g"], count,
                            ctypes.c_void_p(state.data_ptr()),
                            ctypes.c_void_p(torch.cuda.current_stream(dev).cuda_stream)), "mbir_update")
    torch.cuda.synchronize()
    h = {k: v.astype(np.float64) for k, v in host.items()}
    xn = h["y"] - 0.25 * h["g"]
    beta = (5.0 - 1) / (0.5 * (1 + np.sqrt(101.0)))
    want = {"y": xn + beta * (xn - h["x"])}
    want["xp"] = h["x"]
    want["x"] = xn
    for k in ("y", "xp", "x"):            # the later store stays
        if k == same[0] or k == same[1]:
            last = "x" if "x" in same else "xp"
            assert np.max(np.abs(buf[k].cpu().numpy() - want[last])) <= 2.0 ** -20
        else:
            assert np.max(np.abs(buf[k].cpu().numpy() - want[k])) <= 2.0 ** -20
