"""The one-launch layout at the edges of its rules: 16384 pairs and the next size, shares of one and of
several source ranks and of a part of one (the last part short or empty), every compile-time top-k, batches that a lane takes
several tokens of, tables larger than a workgroup, experts with none, two, three and more than 32 live
replicas.  Every field bit-equal to the oracle, with dead ranks, masked, repeated and uncovered pairs;
and the same after the instance got a second context: of a launch captured before, whose workgroups
then use one mask, and of one made then, which is one workgroup or tiles."""
import numpy as np
import pytest

from paper_2605_10670_amd import binding

import gpu_util as gu
from test_gpu_layout_edges import instance

pytestmark = pytest.mark.gpu

# (T, k, R, S, E)
SHAPES = [
    (2048, 8, 32, 9, 256), (2080, 8, 32, 9, 256), (1638, 10, 2, 9, 16), (1600, 10, 32, 3, 90),
    (1816, 9, 8, 4, 30), (585, 7, 65, 3, 130), (1024, 5, 4, 6, 16), (512, 4, 1, 9, 8), (516, 4, 1, 9, 8),
    (8192, 2, 16, 6, 40), (5456, 3, 11, 4, 20), (16384, 1, 64, 2, 100), (600, 2, 150, 8, 1100),
    (64, 8, 32, 9, 256), (72, 8, 24, 9, 200), (194, 8, 2, 9, 16), (770, 10, 2, 9, 16), (26, 32, 1, 40, 32), (82, 10, 1, 12, 11), (1360, 12, 16, 4, 32), (720, 6, 48, 4, 12), (700, 4, 20, 40, 9),
    (256, 8, 32, 9, 256), (384, 8, 12, 9, 64), (360, 8, 9, 9, 64), (384, 3, 128, 4, 200),
]


def check(ctx, oracle, idx, p2l, mask, shape, policy):
    T, k, R, S, E = shape
    want = oracle.step_layout(idx, p2l, mask, E, R, S, max(1, S - 1), policy)
    gu.assert_layout_equal(ctx.read_layout(T), want, T, k)
    assert ctx.check_layout(T).tolist() == [0, 0, 0, 0]


@pytest.mark.parametrize("policy", [binding.SPREAD, binding.FIRST_LIVE])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_layout_once(oracle, shape, policy):
    T, k, R, S, E = shape
    p2l, active, idx = instance(T, k, R, S, E, seed=T * 7 + k)
    idx[: T // 8, 0] = np.arange(E)[E // 2]            # one expert that many tokens name
    for j in range(1, k):
        idx[: T // 8, j][idx[: T // 8, j] == E // 2] = -1
    kw = dict(num_ranks=R, slots_per_rank=S, primary_slots=max(1, S - 1), num_logical=E, max_tokens=T,
              topk=k, hidden=64, policy=policy, strict_coverage=False)
    ctx, other, stream = binding.Context(**kw), None, None
    try:
        import torch
        stream = torch.cuda.Stream()
        dev = gu.to_dev(idx)
        torch.cuda.synchronize()
        ctx.update_placement(p2l, stream)
        ctx.set_membership(active, stream)
        ctx.dispatch_layout(dev, T, stream)
        stream.synchronize()
        check(ctx, oracle, idx, p2l, active, shape, policy)
        ctx.graph_begin(stream)
        ctx.dispatch_layout(dev, T, stream)
        graph = ctx.graph_end(stream)
        other = binding.Context(**kw, parent=ctx)
        for mask in (np.ones(R, np.int32), active):
            ctx.set_membership(mask, stream)
            graph.launch(stream)
            stream.synchronize()
            check(ctx, oracle, idx, p2l, mask, shape, policy)
            changed = mask.copy()
            changed[0] ^= R > 1
            ctx.set_membership(changed, stream)
            ctx.dispatch_layout(dev, T, stream)            # launched with two contexts
            stream.synchronize()
            check(ctx, oracle, idx, p2l, changed, shape, policy)
        graph.destroy()
    finally:
        if other is not None:
            other.destroy()
        ctx.destroy()
