"""The persistent launch on small stacks, whose forward leaves the lines in a CU's
L1 that the adjoint's stages overwrite: the gradient is that of the launches per
stage, repeatedly.

Tolerance: the units are the same arithmetic; 1e-6 relative L2 allows for float32
rounding alone.
"""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("geoms", [[(128, 256, 2, 0.0)] * 6, [(64, 512, 8, -0.1), (256, 256, 25, 54.6)],
                                   [(128, 128, 181, 0.0)] * 2, [(512, 256, 80, 0.0), (256, 256, 6, 0.0), (128, 128, 19, 0.0)],
                                   [(512, 512, 180, 0.0)] * 4])
def test_small_stacks(geoms):
    from paper_2304_12934_amd import Plan, SliceGeometry
    print(f"case: persistent radon_normal over {geoms}", flush=True)
    rng = np.random.default_rng(len(geoms))
    slices = [SliceGeometry(n, nd, np.sort(rng.uniform(0, np.pi, na)), c) for n, nd, na, c in geoms]
    dev = torch.device("cuda", 0)
    with Plan(slices, device=dev) as plan:
        vol = torch.as_tensor(rng.uniform(0, 1, plan.vol_numel), dtype=torch.float32, device=dev)
        b = torch.as_tensor(rng.standard_normal(plan.sino_numel), dtype=torch.float32, device=dev)
        r, g = plan.normal(vol, b)
    with Plan(slices, device=dev, tuning={"persistent": 1}) as plan:
        for _ in range(5):
            rp, gp = plan.normal(vol, b)
            plan.check()
            assert torch.equal(rp.reshape(-1), r.reshape(-1))
            assert float((gp.reshape(-1) - g.reshape(-1)).norm() / g.norm()) <= 1e-6
