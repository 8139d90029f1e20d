"""simsense_scratch_bytes as the no-allocation call's precheck (host arithmetic only)."""
import pytest


@pytest.mark.parametrize("D,paths", [(96, 8), (192, 4)])
def test_scratch_bytes_are_what_the_no_allocation_call_holds(D, paths):
    """Every parameter set whose reported scratch fits the array is taken, also where path
    values do not fit byte sums (p2): these planes fit, one more would not."""
    import paper_2201_11924_amd.native as nat
    p = dict(width=320, height=240, max_disp=D, census_w=7, census_h=9, census_mode=0, p1=7, uniqueness_pct=10,
             lr_max_diff=1, num_paths=paths, median=3, subpixel=1, focal_px=400.0, baseline_m=0.055)
    small, large = nat.scratch_bytes(dict(p, p2=86)), nat.scratch_bytes(dict(p, p2=200))
    assert large == small <= nat.NOALLOC_SCRATCH_BYTES < small + 320 * 240 * D
