"""The de-duplicated layout where ranks are counted by ballot: every limit of that rule from both sides, batches that
end inside a wavefront and inside a share, fewer tokens than ranks have lanes."""
import pytest

import test_gpu_dedup_once as once

pytestmark = pytest.mark.gpu


# (T, k, R, S, E)
@pytest.mark.parametrize("shape", [
    (4, 3, 4, 6, 16), (3, 2, 3, 6, 16), (66, 2, 3, 6, 16), (66, 1, 3, 6, 16), (1025, 1, 1, 12, 12), (130, 1, 2, 9, 16),
    (516, 3, 4, 6, 16), (516, 2, 4, 6, 16), (1032, 6, 8, 6, 40), (1024, 6, 8, 6, 40), (1032, 5, 8, 6, 40), (1030, 8, 5, 9, 36),
    (2044, 8, 7, 9, 36), (1035, 8, 9, 9, 36), (16384, 1, 1, 16, 16), (8190, 2, 3, 9, 27), (1638, 10, 2, 30, 40)], ids=str)
def test_dedup_layout_by_ballot(oracle, shape):
    once.test_dedup_layout_edges(oracle, shape)
