"""The training step's convolutions and weight gradients at the sizes where their
prefetches and row rings can go wrong: single pixels and rows, strips of one column,
row ranges of every remainder of the ring, element by element against the oracle.
"""
import pytest

import test_gpu_net as tn

pytestmark = pytest.mark.gpu

nat = tn.nat


@pytest.mark.parametrize("B,H,W", [(1, 1, 1), (2, 7, 31), (1, 3, 33), (1, 17, 65), (8, 11, 1000), (4, 23, 2600)])
def test_step_at_edges(nat, B, H, W):  # noqa: F811
    tn.test_training_step_layer_by_layer_matches_oracle(nat, B, H, W)
