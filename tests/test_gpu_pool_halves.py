"""Aggregator backward over 256 gate units: both halves of the units in one pass over the rows."""
import pytest

from test_gpu_pool import _pool_case

pytestmark = pytest.mark.gpu


# 512 rows: the fewest the matrix-core kernels take (16 blocks of 32 rows, as many pairs of workgroups); 545: a last block of one
# row; 4095 and 4128: one block less than the 128 pairs of 256 compute units take at once (less its last row), one block more
@pytest.mark.parametrize("rows", [512, 545, 4095, 4128])
def test_backward_of_256_gate_units(rows):
    _pool_case("large", rows, 1)
