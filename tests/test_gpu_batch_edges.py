"""A batch's selection and post tiles at their edges: heights and widths around a tile
and a thread's rows, with and without the median, against single pairs, bit for bit.
"""
import numpy as np
import pytest

from test_gpu_batch import dev, nat  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("median", [3, 0])
def test_tiles_match_single_pairs(nat, median):  # noqa: F811
    import torch
    rng = np.random.default_rng(3)
    params, L, R = [], [], []
    for W, H in [(1, 1), (5, 2), (64, 15), (65, 16), (63, 17), (130, 33), (2, 19)]:
        left = rng.integers(0, 256, (H, W)).astype(np.uint8)
        L.append(dev(left))
        R.append(dev(np.roll(left, -1, 1)))
        params.append(dict(width=W, height=H, max_disp=16, census_w=7, census_h=9, census_mode=0, p1=7, p2=86,
                           uniqueness_pct=10, lr_max_diff=1, num_paths=8, median=median, subpixel=1, focal_px=400.0,
                           baseline_m=0.055))
    b = nat.Batch(params)
    outs = b.outputs()
    b.compute(L, R, outs)
    torch.cuda.synchronize()
    for i, (p, l, r, o) in enumerate(zip(params, L, R, outs)):
        ss = nat.SimSense(p)
        for k, t in zip(("depth", "disp", "flags"), ss(l, r)):
            assert torch.equal(o[k], t), (i, k)
        ss.close()
    b.close()
