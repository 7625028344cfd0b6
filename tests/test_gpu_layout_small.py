"""The one-launch form for small batches: its rule, and its results at the edges of that rule (a pair to a thread,
4096 pairs, 512 tokens), for top-k with and without an instance of its own, and for tables that are larger than
a workgroup or leave no room for the other form."""
import pytest

from paper_2605_10670_amd import binding

import test_gpu_layout_once as once


def test_large_tables_take_the_one_launch():
    """2120 slots: the bitmaps of small batches fit, for one workgroup and for eight."""
    form = binding.load().eep_host_layout_workgroups
    for T in (32, 64):
        assert form(8, 265, 256, 8, T, 0) == 8 and form(8, 265, 256, 8, T, 1) == 1
    assert form(8, 265, 256, 8, 128, 0) == 0


# (T, k, R, S, E)
@pytest.mark.gpu
@pytest.mark.parametrize("policy", [binding.SPREAD, binding.FIRST_LIVE])
@pytest.mark.parametrize("shape", [
    (32, 8, 8, 265, 256), (48, 5, 8, 265, 256), (128, 8, 32, 9, 256), (136, 8, 8, 9, 64), (256, 4, 4, 9, 16),
    (260, 4, 4, 9, 16), (102, 5, 6, 9, 40), (104, 5, 4, 9, 30), (512, 2, 64, 3, 90), (500, 3, 4, 6, 16), (372, 11, 4, 6, 20), (256, 16, 32, 9, 256),
    (128, 32, 4, 20, 64), (128, 8, 128, 9, 1024), (192, 16, 96, 4, 200), (66, 11, 66, 2, 60), (1, 8, 1, 9, 8),
], ids=str)
def test_layout_small(oracle, shape, policy):
    once.test_layout_once(oracle, shape, policy)
