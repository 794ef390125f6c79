"""Every form of the grid and radial transforms against the FP64 oracle: the
lengths whose last radix splits the kept outputs unevenly (5 * 2^a), those that
exchange their passes in two halves (4096 and 5120 points) and the smallest.

Tolerance: float32 relative L2 <= 1e-5 (kernel width 7 on a 2x grid), the bound
of every parity test of the projector.
"""

import numpy as np
import pytest
import torch

from oracle import radon as ora

pytestmark = pytest.mark.gpu
TOL = 1e-5


def rel(a, b):
    return float(np.linalg.norm(np.asarray(a, dtype=np.float64) - b) / np.linalg.norm(b))


@pytest.mark.parametrize("n,nd,z", [(8, 16, 2), (40, 80, 3), (80, 160, 1), (640, 640, 2), (1024, 1280, 1), (1280, 1280, 1),
                                    (2048, 2048, 2), (2560, 2560, 1)])
def test_transform_lengths_against_oracle(n, nd, z):
    from paper_2304_12934_amd import Plan
    print(f"case: {z} x {n}^2, {nd} bins, 3 angles", flush=True)
    rng = np.random.default_rng(n + nd)
    ang = np.array([0.3, 1.9, 2.7])
    f = rng.uniform(0, 1, (z, n, n)).astype(np.float32)
    y = rng.standard_normal((z, 3, nd)).astype(np.float32)
    dev = torch.device("cuda", 0)
    with Plan.uniform_stack(n, nd, ang, z, device=dev) as plan:
        s = plan.fwd(torch.as_tensor(f, device=dev)).cpu().numpy()
        g = plan.adj(torch.as_tensor(y, device=dev)).cpu().numpy()
    k = z - 1
    assert rel(s[k], ora.radon_fwd(f[k], ang, nd)) < TOL
    assert rel(g[k], ora.radon_adj(y[k], ang, n)) < TOL
