"""The MBIR update on buffers that do and do not lie on 16 bytes and on element
counts that are no multiple of the four elements a thread takes at once.

Tolerance: x' and y are a few float32 operations on values below 8 (2^-21 each
way); the dot product is formed in float64 from float32 terms.
"""

import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count,shift", [(1, 0), (3, 0), (1027, 0), (1024, 1), (262147, 3), (1 << 22, 0)])
def test_update_against_float64(count, shift):
    from paper_2304_12934_amd._lib import NR_MBIR_STATE_DOUBLES, NrMbir, check, lib
    print(f"case: mbir_update of {count} elements, {4 * shift} bytes off", flush=True)
    dev = torch.device("cuda", 0)
    rng = np.random.default_rng(count + shift)
    host = {k: rng.standard_normal(count).astype(np.float32) for k in ("x", "xp", "y", "g")}
    buf = {k: torch.zeros(count + 8, dtype=torch.float32, device=dev) for k in host}
    view = {k: buf[k][shift:shift + count] for k in buf}
    for k in host:
        view[k].copy_(torch.as_tensor(host[k]))
    state = torch.zeros(NR_MBIR_STATE_DOUBLES, dtype=torch.float64, device=dev)
    state[0] = 5.0
    params = NrMbir(0.25, 1, 0, 0)
    ptr = {k: ctypes.c_void_p(view[k].data_ptr()) for k in view}
    stream = ctypes.c_void_p(torch.cuda.current_stream(dev).cuda_stream)
    check(lib().mbir_update(ctypes.byref(params), ptr["x"], ptr["xp"], ptr["y"], ptr["g"], count,
                            ctypes.c_void_p(state.data_ptr()), stream), "mbir_update")
    torch.cuda.synchronize()
    h = {k: v.astype(np.float64) for k, v in host.items()}
    xn = h["y"] - 0.25 * h["g"]
    dot = float(np.sum(h["g"] * (xn - h["x"])))
    t = 1.0 if dot > 0 else 5.0
    beta = (t - 1) / (0.5 * (1 + np.sqrt(1 + 4 * t * t)))
    st = state.cpu().numpy()
    assert abs(st[1] - dot) <= 2.0 ** -22 * float(np.sum(np.abs(h["g"]) * (np.abs(xn) + np.abs(h["x"]))))
    assert st[2] == 0.0 and abs(st[4] - beta) < 1e-12
    got = {k: view[k].cpu().numpy() for k in view}
    assert np.max(np.abs(got["x"] - xn)) <= 2.0 ** -21
    assert np.max(np.abs(got["y"] - (xn + beta * (xn - h["x"])))) <= 2.0 ** -20
    assert np.array_equal(got["xp"], host["x"])
    for k in buf:   # nothing outside the views was written
        assert float(buf[k][:shift].abs().sum() + buf[k][shift + count:].abs().sum()) == 0.0
    view["g"][count // 2] = float("inf")
    check(lib().mbir_update(ctypes.byref(params), ptr["x"], ptr["xp"], ptr["y"], ptr["g"], count,
                            ctypes.c_void_p(state.data_ptr()), stream), "mbir_update")
    assert float(state[2].item()) == 1.0
