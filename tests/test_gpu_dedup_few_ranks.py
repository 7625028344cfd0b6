"""The de-duplicated layout of few ranks, around the size up to which it is one launch there."""
import pytest

import test_gpu_dedup_once as once

pytestmark = pytest.mark.gpu


# (T, k, R, S, E)
@pytest.mark.parametrize("shape", [(6144, 2, 3, 9, 27), (6147, 2, 3, 9, 27), (8192, 2, 4, 9, 32), (8192, 2, 1, 12, 12),
                                   (16384, 1, 2, 16, 32), (6144, 1, 3, 4, 8)], ids=str)
def test_dedup_layout_few_ranks(oracle, shape):
    once.test_dedup_layout_edges(oracle, shape)
