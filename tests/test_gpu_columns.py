"""Where there is no buffer for the cost volume: columns and diagonals count census words
(or, with 64-bit words or 256 disparities, the last direction overwrites the costs it
reads).  The no-allocation call at sizes whose path planes fill its array, against a
handle, whose columns read a volume of its own.  Integers until the last steps, which are
the same kernels: every output bit for bit.
"""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nat():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2201_11924_amd.native as n
    return n


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


def compare(nat, p):
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
def test_no_room_for_a_volume(nat, W, H, D, paths):
    p = params(W, H, D, paths, 200)
    need = nat.scratch_bytes(p)
    assert need <= nat.NOALLOC_SCRATCH_BYTES < need + W * H * padded(D)
    compare(nat, p)


# 64-bit words, the second run of the full left-right check
@pytest.mark.parametrize("W,H,D,kw", [(250, 230, 128, dict(census_mode=1)), (208, 200, 180, dict(census_mode=1)),
                                      (1680, 250, 15, dict(census_mode=1)), (240, 240, 120, dict(lr_mode=1))])
def test_wide_words_and_second_run(nat, W, H, D, kw):
    p = params(W, H, D, 8, 130, **kw)
    need = nat.scratch_bytes(p)
    assert need <= nat.NOALLOC_SCRATCH_BYTES < need + W * H * padded(D)
    compare(nat, p)


@pytest.mark.parametrize("W,H,D,paths", [(320, 240, 64, 8), (173, 61, 37, 4), (197, 152, 96, 8)])
def test_room_for_a_volume(nat, W, H, D, paths):
    p = params(W, H, D, paths, 200)
    assert nat.scratch_bytes(p) + W * H * padded(D) <= nat.NOALLOC_SCRATCH_BYTES
    compare(nat, p)
