"""Where there is no buffer for the cost volume: columns and diagonals count census words
(or, with 64-bit words or 256 disparities, the last direction overwrites the costs it
reads).  The no-allocation call at sizes whose path planes fill its array, against a
handle, whose columns read a volume of its own.  Integers until the last steps, which are
the same kernels: every output bit for bit.  And handles and batches whose volume would
not stay in the caches, against the oracle's summed costs.
"""
import pytest

from test_gpu_aggregate import check, nat  # noqa: F401

pytestmark = pytest.mark.gpu


def params(W, H, D, paths, p2, **kw):
    p = dict(width=W, height=H, max_disp=D, census_w=7, census_h=9, census_mode=0, p1=7, p2=p2, uniqueness_pct=10,
             lr_max_diff=1, num_paths=paths, median=3, subpixel=1, focal_px=400.0, baseline_m=0.055)
    p.update(kw)
    return p


def pair(W, H, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    left = torch.randint(0, 256, (H, W), generator=g, device="cuda", dtype=torch.uint8)
    return left, torch.roll(left, -3, 1)


def padded(D):
    return 16 * next(o for o in (1, 2, 4, 6, 8, 12, 16) if 16 * o >= D)


def compare(nat, p):  # noqa: F811
    import torch
    W, H = p["width"], p["height"]
    left, right = pair(W, H, W * 31 + H)
    ss = nat.SimSense(p)
    want = ss(left, right)
    ss.close()
    for rep in range(2):  # the second call finds the first one's values in the array
        got = [torch.full((H, W), -1.0, device="cuda"), torch.full((H, W), -1.0, device="cuda"),
               torch.full((H, W), 255, dtype=torch.uint8, device="cuda")]
        nat.compute_noalloc(p, left, right, *got)
        for k, (g, w) in enumerate(zip(got, want)):
            assert torch.equal(g, w), (W, H, p["max_disp"], rep, k, int((g != w).sum()))


# every count of disparities per lane, whole and padded; line counts that leave a block's
# last lines without a pixel; the longest columns and rows
@pytest.mark.parametrize("W,H,D,paths", [
    (1730, 256, 16, 8), (935, 256, 29, 8), (481, 255, 64, 8), (320, 240, 96, 8), (317, 241, 81, 8), (250, 240, 128, 8),
    (251, 237, 113, 8), (200, 200, 192, 8), (197, 201, 179, 8), (171, 176, 256, 8), (173, 171, 201, 8),
    (7, 8192, 128, 8), (8192, 7, 128, 8), (320, 240, 192, 4), (333, 231, 180, 4)])
def test_no_room_for_a_volume(nat, W, H, D, paths):  # noqa: F811
    p = params(W, H, D, paths, 200)
    need = nat.scratch_bytes(p)
    assert need <= nat.NOALLOC_SCRATCH_BYTES < need + W * H * padded(D)
    compare(nat, p)


# 64-bit words, the second run of the full left-right check
@pytest.mark.parametrize("W,H,D,kw", [(250, 230, 128, dict(census_mode=1)), (208, 200, 180, dict(census_mode=1)),
                                      (1680, 250, 15, dict(census_mode=1)), (240, 240, 120, dict(lr_mode=1))])
def test_wide_words_and_second_run(nat, W, H, D, kw):  # noqa: F811
    p = params(W, H, D, 8, 130, **kw)
    need = nat.scratch_bytes(p)
    assert need <= nat.NOALLOC_SCRATCH_BYTES < need + W * H * padded(D)
    compare(nat, p)


@pytest.mark.parametrize("W,H,D,paths", [(320, 240, 64, 8), (173, 61, 37, 4), (197, 152, 96, 8)])
def test_room_for_a_volume(nat, W, H, D, paths):  # noqa: F811
    p = params(W, H, D, paths, 200)
    assert nat.scratch_bytes(p) + W * H * padded(D) <= nat.NOALLOC_SCRATCH_BYTES
    compare(nat, p)


# volumes about the sizes from which words are counted (96e6 bytes; 4 directions 160e6, 190e6, 228e6)
@pytest.mark.parametrize("W,H,D,kw", [
    (6100, 1000, 16, {}), (3007, 1000, 30, {}), (1600, 950, 64, {}), (1411, 771, 90, {}), (1411, 708, 96, {}),
    (1300, 580, 128, {}), (1250, 420, 192, {}), (1250, 399, 192, {}), (1249, 421, 179, {}), (62, 8192, 192, {}),
    (8192, 62, 192, {}), (1411, 971, 192, dict(num_paths=4)), (1411, 971, 192, dict(num_paths=4, p2=86)),
    (1411, 943, 192, dict(num_paths=4, p2=86)), (1211, 970, 192, dict(num_paths=4)), (1050, 960, 256, dict(num_paths=4)),
    (2003, 1001, 121, dict(num_paths=4, p2=86))])
def test_large_volumes(orc, nat, W, H, D, kw):  # noqa: F811
    check(orc, nat, W, H, D, **dict(dict(p2=200), **kw))


# columns longer than rows, about the sizes from which words are counted there (712 and 1000
# columns, 192e6 bytes), and 4 directions of 256 disparities
@pytest.mark.parametrize("W,H,D,kw", [
    (397, 2051, 192, {}), (711, 1650, 192, {}), (713, 1650, 192, {}), (1003, 1100, 128, {}),
    (700, 1500, 250, dict(num_paths=4)), (1050, 960, 256, dict(num_paths=4, p2=86))])
def test_long_columns(orc, nat, W, H, D, kw):  # noqa: F811
    check(orc, nat, W, H, D, **dict(dict(p2=200), **kw))


def test_batch_of_both_kinds(nat):  # noqa: F811
    """Slots whose columns count words, read a volume, or have none, of one disparity range:
    equal to their single pairs."""
    import torch
    ps = [params(1250, 420, 192, 8, 200), params(200, 120, 192, 8, 200), params(62, 8192, 185, 8, 200),
          params(150, 90, 192, 2, 86), params(201, 100, 192, 4, 86)]
    pairs = [pair(p["width"], p["height"], i) for i, p in enumerate(ps)]
    b = nat.Batch(ps)
    outs = b.outputs()
    for rep in range(2):
        b.compute([a for a, _ in pairs], [c for _, c in pairs], outs)
        torch.cuda.synchronize()
        for i, (p, (a, c), o) in enumerate(zip(ps, pairs, outs)):
            ss = nat.SimSense(p)
            for k, t in zip(("depth", "disp", "flags"), ss(a, c)):
                assert torch.equal(o[k], t), (rep, i, k)
            ss.close()
    b.close()
