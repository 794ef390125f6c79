"""radon_normal on both sides of the size up to which a batch's radial stages are
joined (2^22 points of radial lines): its sinogram and gradient are the three
separate calls', the same arithmetic on the same float32 values (equal bit for
bit).
"""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("angles", [3200, 3300])   # 1600 and 1656 pairs of 2560 points: 4.10 and 4.24 M
def test_normal_around_the_joining_size(angles):
    from paper_2304_12934_amd import Plan
    print(f"case: normal over one 64^2 slice, 2560 bins, {angles} angles", flush=True)
    rng = np.random.default_rng(angles)
    dev = torch.device("cuda", 0)
    with Plan.uniform_stack(64, 2560, rng.uniform(0, np.pi, angles), 1, device=dev) as plan:
        vol = torch.as_tensor(rng.uniform(0, 1, plan.vol_shape()), dtype=torch.float32, device=dev)
        b = torch.as_tensor(rng.standard_normal(plan.sino_shape()), dtype=torch.float32, device=dev)
        r, g = plan.normal(vol, b)
        s = plan.fwd(vol) - b
        a = plan.adj(s)
    assert torch.equal(r, s)
    assert torch.equal(g, a)
