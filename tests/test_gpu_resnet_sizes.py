"""Convolution loads at grids other than 224 px gives: rows that wrap within a step, the stem without its resident window."""
import pytest

from test_gpu_resnet import _run

pytestmark = pytest.mark.gpu


# 160 px: grids 80, 40, 20, 10 and 5 wide, a 32-row step of the weight gradient covers up to seven image rows of 5 and crosses
# tiles; 512 px: the stem's window does not fit its buffer, so forward and weight gradient gather per position
@pytest.mark.timeout(300)
@pytest.mark.parametrize("name,n,tile", [("rn_tiny", 5, 160), ("rn_tiny_bneck", 3, 160), ("rn_tiny", 1, 512)])
def test_grids(name, n, tile):
    _run(name, n=n, tile=tile)
