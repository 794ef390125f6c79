"""Adding up the parts of spreading tiles that many items share: small slices
under long detectors, whose few tiles hold most of the points.
"""

import numpy as np
import pytest
import torch

from oracle import radon as ora

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [(64, 32), (32, 32), (64, 64), (128, 32)])
@pytest.mark.parametrize("angles", [110, 300])
def test_tiles_of_few_and_many_parts(tile, angles):
    """Tiles of a handful to dozens of parts, on both sides of the 16 up to which
    a thread adds every part of its cells: float32 relative L2 <= 1e-5."""
    from paper_2304_12934_amd import Plan
    print(f"case: one 64^2 slice, {angles} x 640, tile {tile}", flush=True)
    rng = np.random.default_rng(angles)
    ang = rng.uniform(0, np.pi, angles)
    y = rng.standard_normal((1, angles, 640)).astype(np.float32)
    dev = torch.device("cuda", 0)
    with Plan.uniform_stack(64, 640, ang, 1, device=dev, tuning={"tile_w": tile[0], "tile_h": tile[1]}) as plan:
        g = [plan.adj(torch.as_tensor(y, device=dev)).cpu().numpy() for _ in range(2)]
    ref = ora.radon_adj(y[0], ang, 64)
    assert np.linalg.norm(g[0][0] - ref) <= 1e-5 * np.linalg.norm(ref)
    assert np.array_equal(g[0], g[1])


def test_adding_up_parts_is_a_small_share_of_the_spreading():
    """A tile of hundreds of parts is no serial chain: 2 % of the spreading's time
    (18 % when one workgroup in four per tile added them one after the other)."""
    from paper_2304_12934_amd import Plan
    print("case: one 64^2 slice, 3200 x 2560, time of the stages", flush=True)
    dev = torch.device("cuda", 0)
    with Plan.uniform_stack(64, 2560, np.linspace(0, np.pi, 3200, endpoint=False), 1, device=dev) as plan:
        y = torch.randn(plan.sino_shape(), device=dev)
        plan.adj(y)
        plan.profile(True)
        plan.adj(y)
        plan.profile_read()
        for _ in range(5):
            plan.adj(y)
        ms = {k: v[0] for k, v in plan.profile_read().items()}
    assert ms["spread_shared"] < 0.08 * ms["spread"]


def test_persistent_launch_adds_many_parts():
    """The persistent kernel runs the same units: gradient as from the launches
    per stage, up to float32 rounding (transforms of other thread counts)."""
    from paper_2304_12934_amd import Plan
    print("case: two 64^2 slices, 500 x 512, persistent and per stage", flush=True)
    dev = torch.device("cuda", 0)
    ang = np.linspace(0, np.pi, 500, endpoint=False)
    out = []
    for persistent in (0, 1):
        with Plan.uniform_stack(64, 512, ang, 2, device=dev, tuning={"persistent": persistent}) as plan:
            vol = torch.as_tensor(np.random.default_rng(3).uniform(0, 1, (2, 64, 64)), dtype=torch.float32, device=dev)
            out.append(plan.normal(vol)[1])
            plan.check()
    assert float((out[1] - out[0]).norm() / out[0].norm()) <= 1e-6
