"""radon_normal joins the forward's and the adjoint's radial stages: its sinogram
and gradient against the three separate calls, which are the same arithmetic on
the same float32 values (equal bit for bit), over detector lengths with an odd
angle count, an axis offset, no data and mixed stacks.
"""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("geoms,with_b", [([(64, 80, 45, 0.0)], True), ([(128, 128, 7, 1.25)] * 3, True),
                                          ([(40, 16, 1, 0.0), (32, 640, 31, -2.5), (128, 1280, 12, 0.0)], True),
                                          ([(512, 512, 101, 0.0)] * 2, False)])
def test_normal_is_the_three_calls(geoms, with_b):
    from paper_2304_12934_amd import Plan, SliceGeometry
    print(f"case: normal over {geoms}, data {with_b}", flush=True)
    rng = np.random.default_rng(len(geoms))
    dev = torch.device("cuda", 0)
    with Plan([SliceGeometry(n, nd, rng.uniform(0, np.pi, na), c) for n, nd, na, c in geoms], device=dev) as plan:
        vol = torch.as_tensor(rng.uniform(0, 1, plan.vol_numel), dtype=torch.float32, device=dev)
        b = torch.as_tensor(rng.standard_normal(plan.sino_numel), dtype=torch.float32, device=dev) if with_b else None
        r, g = plan.normal(vol, b)
        s = plan.fwd(vol).reshape(-1)
        if with_b:
            s = s - b
        a = plan.adj(s)
    assert torch.equal(r.reshape(-1), s)
    assert torch.equal(g.reshape(-1), a.reshape(-1))
