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
