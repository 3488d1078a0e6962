"""GPU: gradients in blocks of 64 rows (more than 8192) at the widths 128 and 256, whose one-launch pass then
holds most registers and LDS, with the oracle, inputs and bounds of test_gpu_mlp_split.py: one row in the
last block, and a ragged count of blocks and chunks."""
import pytest

pytestmark = pytest.mark.gpu

import test_gpu_mlp_split as split  # noqa: E402


@pytest.mark.parametrize("n_in,hidden,layers,n", [(4, 128, 2, 8193), (4, 256, 2, 8193), (4, 128, 4, 10007),
                                                  (16, 256, 1, 12350)])
def test_gradients_in_blocks_of_64_rows(n_in, hidden, layers, n):
    split.test_gradients_over_splits(n_in, hidden, layers, n)
