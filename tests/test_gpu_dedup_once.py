"""The de-duplicated layout's one launch at the edges of its rule (64 ranks, top-10, 16384 pairs) and of
its shares of 64 tokens, and the two launches just beyond them, every field equal to the oracle."""
import numpy as np
import pytest

from paper_2605_10670_amd import binding

import gpu_util as gu
from test_gpu_layout_edges import instance

pytestmark = pytest.mark.gpu


# (T, k, R, S, E)
@pytest.mark.parametrize("shape", [
    (1, 1, 1, 3, 3), (63, 8, 3, 9, 20), (64, 7, 2, 4, 8), (65, 5, 1, 40, 32), (130, 8, 65, 2, 100),
    (128, 8, 64, 2, 100), (512, 2, 64, 3, 90), (1024, 10, 8, 36, 256), (1088, 9, 32, 9, 256), (1034, 11, 11, 9, 64),
    (2048, 8, 8, 36, 256), (2056, 8, 8, 36, 256), (16384, 1, 64, 2, 100), (2720, 6, 16, 3, 40), (5460, 3, 4, 6, 16),
], ids=str)
def test_dedup_layout_edges(oracle, shape):
    T, k, R, S, E = shape
    p2l, active, idx = instance(T, k, R, S, E, seed=T + 13 * k)
    ctx = binding.Context(num_ranks=R, slots_per_rank=S, primary_slots=max(1, S - 1), num_logical=E,
                          max_tokens=T, topk=k, hidden=64, strict_coverage=False)
    try:
        ctx.update_placement(p2l)
        ctx.set_membership(active)
        ctx.dispatch_layout(gu.to_dev(idx), T)
        ctx.dedup_layout(T)
        got = ctx.read_dedup(T)
        lay = oracle.step_layout(idx, p2l, active, E, R, S, max(1, S - 1), binding.SPREAD)
        want = oracle.dedup_layout(lay["slot_of"], lay["row_of"], R, S)
        assert got["N_d"] == want["N_d"]
        for name in ("dedup_count", "dedup_offset", "dedup_row", "expand_of"):
            assert np.array_equal(got[name], want[name]), name
        assert np.array_equal(got["dedup_dst"], np.where(want["lead"] == 1, want["dedup_row"], -1))
    finally:
        ctx.destroy()
