"""The aggregation's lines, segments and pairs at the sizes where they can go wrong:
the summed path costs of every pixel and disparity against the oracle, bit for bit
(all values are integers).
"""
import numpy as np
import pytest

from synth import PairSpec, make_pair

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nat():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2201_11924_amd.native as n
    return n


def check(orc, nat, W, H, D, tunings=((0, 3),), **kw):
    import torch
    p = dict(width=W, height=H, max_disp=D, census_w=7, census_h=9, census_mode=0, p1=7, p2=86, uniqueness_pct=10,
             lr_max_diff=1, num_paths=8, median=3, subpixel=1, focal_px=400.0, baseline_m=0.055)
    p.update(kw)
    spec = PairSpec(W, H, planes=3, dmin=0, dmax=max(0.0, min(D - 1, W - 1) * 0.8), noise="gauss", sigma=3.0)
    pr = make_pair(spec, W * 7919 + H * 31 + D)
    left, right = orc.ir_noise(pr.left, pr.gamma_l, pr.n_l), orc.ir_noise(pr.right, pr.gamma_r, pr.n_r)
    ref = orc.sgm(p, left, right, keep_volume=True)
    L, R = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (left, right))
    ss = nat.SimSense(p)
    for lanes, blocks in tunings:
        ss.set_tuning(lanes, blocks)
        for rep in range(2):  # the scratch still holds the first pass's values in the second
            out = ss.compute_all(L, R, volume=True)
            S = out["volume"].cpu().numpy().view(np.uint16).astype(np.uint32)
            assert np.array_equal(S, ref.S), (W, H, D, lanes, blocks, rep, int((S != ref.S).sum()))
            assert np.array_equal(out["flags"].cpu().numpy(), ref.flags)
    ss.close()


# line lengths around a segment of 8 steps, a load ring of 16 and its look-ahead of 28;
# widths around the 4 and 8 lines of a wave and a block
@pytest.mark.parametrize("W,H", [(1, 1), (2, 9), (9, 2), (7, 8), (8, 7), (16, 17), (17, 16), (31, 33), (33, 15),
                                 (61, 64), (130, 29)])
@pytest.mark.parametrize("paths", [4, 8])
def test_line_lengths(orc, nat, W, H, paths):
    check(orc, nat, W, H, 20, num_paths=paths)


# every count of disparities per lane, whole and with padding, lanes in use and idle,
# for all lane counts; pairs stored as sums, and values too large for that (p2), which
# run one direction per buffer and the last one over the cost volume
@pytest.mark.parametrize("D,lanes", [(16, (16,)), (11, (16,)), (32, (16, 32)), (64, (16, 32, 64)), (50, (0, 64)),
                                     (96, (16, 32)), (81, (0,)), (128, (16, 32, 64)), (113, (0, 32)),
                                     (192, (16, 32, 64)), (179, (0,)), (256, (16, 32, 64)), (201, (16, 64))])
@pytest.mark.parametrize("kw", [{}, dict(p2=200), dict(census_mode=1, p2=65), dict(census_mode=1, p2=66)])
def test_disparities_per_lane(orc, nat, D, lanes, kw):
    check(orc, nat, 150, 37, D, tunings=[(hl, 3) for hl in lanes] + [(lanes[0], 0)], **kw)


@pytest.mark.parametrize("D", [16, 32, 64, 96, 128, 192, 256])
@pytest.mark.parametrize("paths", [2, 4, 8])
def test_block_costs(orc, nat, D, paths):
    check(orc, nat, 70, 43, D - 3, num_paths=paths, block_w=3, block_h=3, p1=63, p2=774)
    check(orc, nat, 33, 18, D, num_paths=paths, block_w=3, block_h=1, p1=0, p2=8191 - 93)


@pytest.mark.parametrize("W,H,D", [(1411, 771, 256), (1410, 770, 250), (1280, 720, 256)])
def test_large_volumes(orc, nat, W, H, D):
    """Cost volumes over and under the size from which the horizontal directions are
    stored as their sum, whole and with padding disparities; 16-byte path-value stores
    with the memory pipe busy."""
    check(orc, nat, W, H, D, tunings=((16, 3),))
