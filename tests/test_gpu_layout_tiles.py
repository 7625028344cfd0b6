"""The layout in tiles, which batches of one context take only beyond 16384 pairs, at the sizes and shapes where tiles
are ragged: an instance of two contexts lays out what is more than 384 tokens or 3072 pairs that way.  Every field
equal to the oracle, from the first context and, with another placement, from the second."""
import numpy as np
import pytest

from paper_2605_10670_amd import binding

import gpu_util as gu
from test_gpu_layout_edges import instance

pytestmark = pytest.mark.gpu


# (T, k, R, S, E): ranks of 129, 131, 65, 1 and 400 tokens, one rank, more than 64 ranks and more than 64 tiles, tables
# larger than a workgroup, top-k with and without an instance, pairs of a tile in one, two and four rounds
@pytest.mark.parametrize("policy", [binding.SPREAD, binding.FIRST_LIVE])
@pytest.mark.parametrize("shape", [
    (516, 8, 4, 9, 32), (524, 8, 4, 9, 32), (650, 7, 10, 5, 40), (385, 1, 7, 5, 20), (388, 8, 4, 6, 16), (400, 8, 1, 20, 16),
    (512, 8, 32, 9, 256), (1024, 8, 32, 9, 256), (1024, 2, 32, 9, 256), (1200, 3, 3, 9, 20), (390, 8, 65, 4, 200),
    (1300, 5, 65, 2, 96), (2600, 4, 130, 2, 120), (420, 8, 2, 600, 1030), (1024, 12, 8, 9, 64), (516, 16, 4, 10, 40),
    (128, 32, 4, 20, 64), (1024, 32, 8, 10, 64), (2048, 10, 8, 9, 64), (8192, 1, 8, 3, 20), (8192, 2, 65 - 1, 3, 90),
], ids=str)
def test_layout_in_tiles(oracle, shape, policy):
    T, k, R, S, E = shape
    kw = dict(num_ranks=R, slots_per_rank=S, primary_slots=max(1, S - 1), num_logical=E, max_tokens=T, topk=k,
              hidden=64, policy=policy, strict_coverage=False)
    ctx, other = binding.Context(**kw), None
    try:
        assert binding.load().eep_host_layout_workgroups(R, S, E, k, T, 1) == 0
        other = binding.Context(**kw, parent=ctx)
        p2l, active, idx = instance(T, k, R, S, E, seed=T * 5 + k)
        dev = gu.to_dev(idx)
        ctx.set_membership(active)
        for c, placement in ((ctx, p2l), (other, np.roll(p2l, 1))):
            c.update_placement(placement)
            c.dispatch_layout(dev, T)
            gu.assert_layout_equal(c.read_layout(T), oracle.step_layout(idx, placement, active, E, R, S, max(1, S - 1),
                                                                        policy), T, k)
            assert c.check_layout(T).tolist() == [0, 0, 0, 0]
    finally:
        if other is not None:
            other.destroy()
        ctx.destroy()
