"""The tiled interpolation and the spreading items at the sizes where their
work is split differently: tiles at the grid's edges for every kernel width,
stacks of mixed sizes in one launch, plans with few points (small items, tiles
shared by several) and launches of one and of two items per workgroup.
"""

import numpy as np
import pytest
import torch

from oracle import radon as ora

pytestmark = pytest.mark.gpu


def rel(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("width", [6, 7, 8])
def test_tiles_equal_direct_sums_in_a_mixed_stack(width):
    """The same sums in the same order as the gathers straight from the grid;
    only the 1/N_t scale is rounded apart (one float32 rounding: 2^-24)."""
    from paper_2304_12934_amd import Plan, SliceGeometry
    print(f"case: mixed stack, width {width}, tiled and direct", flush=True)
    rng = np.random.default_rng(width)
    geoms = [SliceGeometry(n, nd, rng.uniform(0, np.pi, na)) for n, nd, na in
             ((128, 128, 50), (64, 80, 33), (256, 320, 201), (8, 16, 3), (128, 128, 50))]
    dev = torch.device("cuda", 0)
    out = []
    for mode in (0, 1):
        with Plan(geoms, width=width, device=dev, tuning={"interp_mode": mode}) as plan:
            vol = torch.as_tensor(np.random.default_rng(7).uniform(0, 1, plan.vol_numel), dtype=torch.float32, device=dev)
            out.append(plan.fwd(vol).cpu().numpy())
    assert rel(out[0], out[1]) < 2.0 ** -22


@pytest.mark.parametrize("n,na,z", [(128, 120, 1), (128, 400, 4), (512, 700, 3)])
def test_item_sizes_against_oracle(n, na, z):
    """Few points (items of 256, shared tiles), more (1024 per spreading item,
    256 or 512 per interpolation item) and many: float32 relative L2 <= 1e-5."""
    from paper_2304_12934_amd import Plan
    print(f"case: {z} x {n}^2, {na} angles", flush=True)
    rng = np.random.default_rng(n + na)
    ang = np.sort(rng.uniform(0, np.pi, na))
    f = rng.uniform(0, 1, (z, n, n)).astype(np.float32)
    y = rng.standard_normal((z, na, n)).astype(np.float32)
    dev = torch.device("cuda", 0)
    with Plan.uniform_stack(n, n, ang, z, device=dev) as plan:
        s = plan.fwd(torch.as_tensor(f, device=dev)).cpu().numpy()
        g = plan.adj(torch.as_tensor(y, device=dev)).cpu().numpy()
    some = rng.choice(na, 12, replace=False)
    assert rel(s[z - 1][some], ora.radon_fwd(f[z - 1], ang[some], n)) < 1e-5
    if n <= 128:
        assert rel(g[z - 1], ora.radon_adj(y[z - 1], ang, n)) < 1e-5
    else:
        pix = rng.integers(n // 8, n - n // 8, (64, 2))
        assert rel([g[z - 1][iy, ix] for iy, ix in pix], ora.radon_adj_entries(y[z - 1], ang, n, pix)) < 1e-5


@pytest.mark.parametrize("width", [6, 7, 8])
def test_two_items_per_workgroup_equal_one(width):
    """A launch of at least 8192 interpolation and spreading items (two per
    workgroup) against launches of one slice each (one per workgroup) over the
    same items: every item's arithmetic is the same, so the forward is equal bit
    for bit, and the adjoint differs by no more than float32 rounding."""
    from paper_2304_12934_amd import Plan
    n, na, z = 1024, 200, 12
    print(f"case: {z} x {n}^2, {na} angles, width {width}, two items and one per workgroup", flush=True)
    ang = np.linspace(0, np.pi, na, endpoint=False)
    # interpolation items: tiles of 32 x 64 cells holding first taps (radius j G / N_t of the half plane)
    j = np.arange(n // 2 + 1) * 2.0
    u, v = np.abs(np.outer(np.sin(ang), j)), np.outer(np.cos(ang), j)
    assert z * len(np.unique(np.floor(u / 32) * 1000 + np.floor(v / 64))) >= 9000
    dev = torch.device("cuda", 0)
    vol = torch.as_tensor(np.random.default_rng(width).uniform(0, 1, (z, n, n)), dtype=torch.float32, device=dev)
    sino = torch.as_tensor(np.random.default_rng(9).standard_normal((z, na, n)), dtype=torch.float32, device=dev)
    out = []
    for tuning in ({"batch_mb": 2048, "streams": 1}, {"batch": 1, "streams": 1}):
        with Plan.uniform_stack(n, n, ang, z, width=width, device=dev, tuning=tuning) as plan:
            info = plan.info()
            assert info["batches"] == (1 if "batch_mb" in tuning else z)
            assert z * info["spread_items"] >= 9000
            out.append((plan.fwd(vol), plan.adj(sino)))
    assert torch.equal(out[0][0], out[1][0])
    assert float((out[0][1] - out[1][1]).norm() / out[1][1].norm()) <= 1e-6
