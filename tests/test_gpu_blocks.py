"""The block-cost row walks at their edges: every number of disparities per lane, both
block sizes and both word sizes, images wide enough for windows wholly inside, with
last walks of every remainder, against the oracle, bit for bit.
"""
import pytest

from test_gpu_aggregate import check, nat  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,H", [(13, 8), (32, 9), (61, 11), (96, 13), (125, 19), (192, 7), (250, 10)])
@pytest.mark.parametrize("kw", [dict(block_w=3, block_h=3), dict(block_w=5, block_h=5),
                                dict(block_w=3, block_h=3, census_mode=1), dict(block_w=5, block_h=5, census_mode=1)])
def test_row_walks(orc, nat, D, H, kw):  # noqa: F811
    check(orc, nat, (D + 15) // 16 * 16 + 21 + H, H, D, num_paths=4, p1=63, p2=774, **kw)


def test_long_walks(orc, nat):  # noqa: F811
    check(orc, nat, 331, 803, 32, num_paths=2, p1=63, p2=774, block_w=3, block_h=3)
