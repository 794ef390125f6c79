"""The lengths whose adjoint takes other radices than its forward (640, 1024,
1280, 2048 and 2560 points), in a launch of several slices and one of a single
slice, against the FP64 oracle; and the pair <Af, y> = <f, A*y>.

Tolerances: float32 relative L2 <= 1e-5 (kernel width 7 on a 2x grid), the bound
of every parity test of the projector; the inner products, each off by no more
than that bound times ||Af|| ||y||, agree to 1e-5 of it.
"""

import numpy as np
import pytest
import torch

from oracle import radon as ora

pytestmark = pytest.mark.gpu
TOL = 1e-5


@pytest.mark.parametrize("n,z", [(320, 3), (512, 1), (640, 1), (1024, 1), (1280, 2)])
def test_adjoint_with_its_own_radices(n, z):
    from paper_2304_12934_amd import Plan
    print(f"case: {z} x {n}^2, 5 angles", flush=True)
    rng = np.random.default_rng(n)
    ang = np.array([0.0, 0.4, 1.1, 2.0, 2.9])
    f = rng.standard_normal((z, n, n)).astype(np.float32)
    y = rng.standard_normal((z, 5, n)).astype(np.float32)
    dev = torch.device("cuda", 0)
    with Plan.uniform_stack(n, n, ang, z, device=dev) as plan:
        s = plan.fwd(torch.as_tensor(f, device=dev)).cpu().numpy().astype(np.float64)
        g = plan.adj(torch.as_tensor(y, device=dev)).cpu().numpy().astype(np.float64)
    for k in (0, z - 1):
        ref = ora.radon_adj(y[k], ang, n)
        assert np.linalg.norm(g[k] - ref) < TOL * np.linalg.norm(ref)
    a, b = float((s * y).sum()), float((f * g).sum())
    assert abs(a - b) < 1e-5 * np.linalg.norm(s) * np.linalg.norm(y)
