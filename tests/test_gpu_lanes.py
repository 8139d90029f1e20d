"""Lanes per horizontal line: the default about the sizes where it changes, against the
oracle's summed costs, bit for bit.
"""
import pytest

from test_gpu_aggregate import check, nat  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H", [512, 513, 1024, 1025])
@pytest.mark.parametrize("D,kw", [(90, {}), (128, dict(p2=200)), (192, {}), (175, dict(census_mode=1, p2=60))])
def test_default_of_rows_alone(orc, nat, H, D, kw):  # noqa: F811
    check(orc, nat, 45, H, D, num_paths=2, **kw)


@pytest.mark.parametrize("W,H", [(1900, 1097), (1903, 1098)])
def test_default_of_four_paths_from_words(orc, nat, W, H):  # noqa: F811
    check(orc, nat, W, H, 128, num_paths=4, p2=200)


@pytest.mark.parametrize("D,lanes", [(60, (16, 32, 64)), (90, (16, 32)), (128, (16, 32, 64))])
def test_autotune_times_each_launch_once(nat, D, lanes):  # noqa: F811
    """Candidates that launch the same thing report one time: a handle's blocks_per_cu above
    0, a batch's all, and 32 and 64 lanes of 64 disparities."""
    import torch
    p = dict(width=130, height=70, max_disp=D, census_w=7, census_h=9, census_mode=0, p1=7, p2=86, uniqueness_pct=10,
             lr_max_diff=1, num_paths=8, median=3, subpixel=1, focal_px=400.0, baseline_m=0.055)
    left = torch.randint(0, 256, (70, 130), dtype=torch.uint8, device="cuda")
    right = torch.roll(left, -3, 1)
    ss = nat.SimSense(p)
    want = [t.clone() for t in ss(left, right)]
    best, ms = ss.autotune(left, right, reps=3)
    got = ss(left, right)
    ss.close()
    assert len(ms) == 5 * len(lanes) and best["horizontal_lanes"] in lanes
    assert all(len(set(ms[i + 1:i + 5])) == 1 for i in range(0, len(ms), 5)), ms
    assert D != 60 or ms[5:10] == ms[10:15]
    assert all(torch.equal(g, w) for g, w in zip(got, want))
    b = nat.Batch([p, p])
    outs = b.outputs()
    best, ms = b.autotune([left] * 2, [right] * 2, outs, reps=3)
    b.compute([left] * 2, [right] * 2, outs)
    torch.cuda.synchronize()
    assert len(ms) == 4 * len(lanes) and best["horizontal_lanes"] in lanes
    assert all(len(set(ms[i:i + 4])) == 1 for i in range(0, len(ms), 4)), ms
    assert D != 60 or ms[4:8] == ms[8:12]
    assert all(torch.equal(o[k], w) for o in outs for k, w in zip(("depth", "disp", "flags"), want))
    b.close()


@pytest.mark.parametrize("D", [256, 250])
def test_row_sums_of_four_paths(orc, nat, D):  # noqa: F811
    """Two planes, both sums, from a volume large enough that 16 lanes store the rows as
    their sum; and the default shape, whose rows are planes of their own."""
    check(orc, nat, 1411, 771, D, tunings=((16, 3), (0, 3)), num_paths=4)


def test_row_sums_in_a_batch(nat):  # noqa: F811
    """Slots with rows as sums beside slots without, of 8 and 4 paths: equal to single pairs
    whose rows are planes of their own (32 lanes)."""
    import torch
    ps = [dict(width=W, height=H, max_disp=D, census_w=7, census_h=9, census_mode=0, p1=7, p2=86, uniqueness_pct=10,
               lr_max_diff=1, num_paths=paths, median=3, subpixel=1, focal_px=400.0, baseline_m=0.055)
          for W, H, D, paths in ((1411, 771, 256, 8), (200, 90, 256, 8), (1411, 771, 250, 4), (150, 101, 256, 4))]
    g = torch.Generator(device="cuda").manual_seed(6)
    lefts = [torch.randint(0, 256, (p["height"], p["width"]), generator=g, dtype=torch.uint8, device="cuda") for p in ps]
    rights = [torch.roll(a, -7, 1) for a in lefts]
    b = nat.Batch(ps)
    b.set_tuning(16, 2)
    outs = b.outputs()
    for rep in range(2):
        b.compute(lefts, rights, outs)
        torch.cuda.synchronize()
        for i, (p, o) in enumerate(zip(ps, outs)):
            ss = nat.SimSense(p)
            ss.set_tuning(32, 3)
            for k, t in zip(("depth", "disp", "flags"), ss(lefts[i], rights[i])):
                assert torch.equal(o[k], t), (rep, i, k)
            ss.close()
    b.close()
