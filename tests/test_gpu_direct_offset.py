"""The direct interpolation (interp_mode 1) of slices whose rotation axis lies off
centre: the sums and the phase of the tiled one; only the 1/N_t scale is rounded
apart (one float32 rounding, 2^-24, and one more through the phase).
"""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [6, 7, 8])
def test_direct_interpolation_off_centre(width):
    from paper_2304_12934_amd import Plan, SliceGeometry
    print(f"case: direct and tiled interpolation off centre, width {width}", flush=True)
    rng = np.random.default_rng(width)
    geoms = [SliceGeometry(n, nd, rng.uniform(0, np.pi, na), c)
             for n, nd, na, c in ((128, 160, 31, 1.25), (64, 80, 1, -3.5), (256, 256, 40, 0.0))]
    dev = torch.device("cuda", 0)
    out = []
    for mode in (0, 1):
        with Plan(geoms, width=width, device=dev, tuning={"interp_mode": mode}) as plan:
            vol = torch.as_tensor(np.random.default_rng(1).uniform(0, 1, plan.vol_numel), dtype=torch.float32, device=dev)
            out.append(plan.fwd(vol).reshape(-1).double())
    assert float((out[0] - out[1]).norm() / out[0].norm()) < 2.0 ** -22
