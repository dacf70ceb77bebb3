"""The cost refresh on frames whose workgroups take several rounds of pixels
(tiles by the frame's size, runs by the lists' lengths), with few, half and all
pixels assigned, against the oracle."""
import pytest

from tests import test_gpu_cost

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,p,assigned", [
    (257, 128, dict(C=5, r=4), 0.5),                              # tiles of two rounds, from 32768 pixels
    (331, 298, dict(C=3, r=3, grad_weight=0.0), 0.02),            # tiles of 16 x 8, from 98304; runs of 72 pixels
    (514, 511, dict(C=5, r=4, fp16=True), 0.97),                  # 33 tiles in a row; runs of one round
    (512, 384, dict(C=3, r=2, grad_weight=0.0), 0.5),             # 32 tiles in a row
    (515, 513, dict(C=3, r=1, grad_weight=0.0, fp16=True), 0.0),  # the longest runs, 168 pixels
    (515, 513, dict(C=5, r=4), 0.0),                              # and 140 pixels
])
def test_cost_refresh_in_rounds(W, H, p, assigned):
    test_gpu_cost.test_cost_refresh(W, H, p, assigned)
