"""dispatch_layout at the edges of its launch forms: pairs per thread (1024, 2048, 4096 pairs), the
limits of the one-launch form for small batches (512 tokens, 4096 pairs), top-k with and without a lane form, masks in a
register (up to 64 ranks) and in LDS, experts with more than 32 replicas, slot counts around the
scan's groups of 64 and 320.  Every field bit-equal to the oracle, with dead ranks, masked, repeated
and uncovered pairs."""
import numpy as np
import pytest

from paper_2605_10670_amd import binding

import gpu_util as gu

pytestmark = pytest.mark.gpu

# (T, k, R, S, E)
SHAPES = [
    (1, 1, 1, 1, 1), (32, 8, 32, 9, 256), (128, 8, 32, 9, 256), (160, 8, 32, 9, 256),
    (256, 8, 32, 9, 256), (288, 8, 32, 9, 256), (512, 8, 32, 9, 256), (544, 8, 32, 9, 256),
    (127, 8, 1, 20, 16), (129, 8, 3, 7, 16), (513, 8, 1, 12, 12), (512, 4, 4, 6, 16),
    (512, 1, 8, 3, 8), (514, 2, 2, 9, 12), (500, 2, 4, 6, 16), (510, 6, 6, 5, 24), (128, 32, 4, 20, 64),
    (132, 32, 4, 20, 64), (96, 3, 32, 2, 40), (400, 16, 16, 5, 40), (260, 8, 65, 2, 96),
    (1300, 8, 65, 2, 96), (200, 4, 100, 3, 250), (160, 2, 8, 10, 2), (1600, 2, 8, 10, 2),
    (64, 8, 32, 10, 300), (64, 8, 1, 321, 300), (640, 8, 64, 10, 600), (64, 5, 64, 10, 600),
    (4096, 10, 32, 9, 256), (3000, 1, 24, 5, 96), (4160, 8, 65, 4, 200), (5976, 6, 24, 5, 96),
    (8192, 8, 64, 3, 150),
]


def instance(T, k, R, S, E, seed):
    rng = np.random.default_rng(seed)
    P = R * S
    p2l = rng.integers(0, E, P).astype(np.int32)
    first = rng.permutation(P)[:min(P, E)]
    p2l[first] = np.arange(first.size)             # most experts have at least one replica
    p2l[rng.random(P) < 0.05] = -1
    active = (rng.random(R) < 0.85).astype(np.int32)
    active[rng.integers(R)] = 1
    idx = np.argsort(rng.random((T, max(E, k))), axis=1)[:, :k].astype(np.int32)
    idx[idx >= E] = -1
    idx[rng.random(idx.shape) < 0.02] = E
    if k > 1:
        again = rng.random(T) < 0.1
        idx[again, k - 1] = idx[again, 0]
    return p2l, active, idx


@pytest.mark.parametrize("policy", [binding.SPREAD, binding.FIRST_LIVE])
@pytest.mark.parametrize("T,k,R,S,E", SHAPES)
def test_layout_forms(oracle, T, k, R, S, E, policy):
    S_prim = max(1, S - 1)
    p2l, active, idx = instance(T, k, R, S, E, seed=T * 31 + R)
    ctx = binding.Context(num_ranks=R, slots_per_rank=S, primary_slots=S_prim, num_logical=E,
                          max_tokens=T, topk=k, hidden=64, policy=policy, strict_coverage=False)
    try:
        ctx.update_placement(p2l)
        ctx.set_membership(active)
        ctx.dispatch_layout(gu.to_dev(idx), T)
        got = ctx.read_layout(T)
        want = oracle.step_layout(idx, p2l, active, E, R, S, S_prim, policy)
        gu.assert_layout_equal(got, want, T, k)
        assert ctx.check_layout(T).tolist() == [0, 0, 0, 0]
    finally:
        ctx.destroy()


# P + (E + 1) + P values: 96 and 97 (one short launch or one long), 960 and 961 (one long launch or
# two), 1921 (three)
@pytest.mark.parametrize("P,E", [(40, 15), (40, 16), (320, 319), (320, 320), (640, 640)])
def test_placement_update_spans_launches(P, E):
    ctx = binding.Context(num_ranks=P, slots_per_rank=1, primary_slots=1, num_logical=E,
                          max_tokens=0, topk=1, hidden=64, strict_coverage=False)
    try:
        rng = np.random.default_rng(P + E)
        version = 0
        for _ in range(2):
            p2l = rng.integers(-1, E, P).astype(np.int32)
            ctx.update_placement(p2l)
            version += 1
            off, lst = binding.host_replica_lists(p2l, E, 1, 1)
            assert np.array_equal(ctx.read("phys_to_logical", P), p2l)
            assert np.array_equal(ctx.read("l2p_off", E + 1), off)
            assert np.array_equal(ctx.read("l2p_list", P), lst)
            active = (rng.random(P) < 0.5).astype(np.int32)
            ctx.set_membership(active)
            version += 1
            assert np.array_equal(ctx.read("active", P), active)
            ctx.dispatch_layout(None, 0)
            assert ctx.read("status", 4)[3] == version
    finally:
        ctx.destroy()


@pytest.mark.parametrize("T,k", [(64, 8), (512, 8), (320, 3), (1024, 8)])
def test_layout_over_its_router_indices(oracle, T, k):
    """slot_of given the router indices' own memory: the caller needs them no longer."""
    import torch
    R, S, E = 32, 9, 256
    p2l, active, idx = instance(T, k, R, S, E, seed=T + k)
    off, lst = binding.host_replica_lists(p2l, E, S, S - 1)
    sizes = dict(slot_of=T * k, row_of=T * k, src_of=T * k, count=R * S, offset=R * S + 1,
                 rank_count=R, rank_offset=R + 1, cnt_src=R * R * S, status=4)
    out = {n: torch.zeros(m, dtype=torch.int32, device="cuda") for n, m in sizes.items()}
    out["slot_of"].copy_(torch.from_numpy(idx.reshape(-1)))
    binding.dispatch_layout_noalloc(R=R, S=S, E=E, k=k, policy=binding.SPREAD,
                                    topk_idx=out["slot_of"], active=gu.to_dev(active),
                                    l2p_off=gu.to_dev(off), l2p_list=gu.to_dev(lst), out=out, T=T)
    want = oracle.step_layout(idx, p2l, active, E, R, S, S - 1, binding.SPREAD)
    for n in ("slot_of", "row_of", "src_of", "count", "offset", "cnt_src"):
        assert np.array_equal(out[n].cpu().numpy(), want[n].reshape(-1)), n


@pytest.mark.parametrize("T,R", [(130, 65), (1300, 65), (128, 32)])
def test_what_lies_behind_the_replica_lists_is_not_used(oracle, T, R):
    """Lists shorter than the slot count (empty slots), with arbitrary values behind them."""
    import torch
    k, S, E = 4, 3, 90
    p2l, active, idx = instance(T, k, R, S, E, seed=T + R)
    p2l[R * S // 2:] = -1
    off, lst = binding.host_replica_lists(p2l, E, S, S - 1)
    n = int(off[E])
    assert n < R * S
    lst[n:] = np.resize(np.array([2**31 - 1, -2**31, R * S, 10**6, -7], np.int32), R * S - n)
    sizes = dict(slot_of=T * k, row_of=T * k, src_of=T * k, count=R * S, offset=R * S + 1,
                 rank_count=R, rank_offset=R + 1, cnt_src=R * R * S, status=4)
    out = {name: torch.zeros(m, dtype=torch.int32, device="cuda") for name, m in sizes.items()}
    binding.dispatch_layout_noalloc(R=R, S=S, E=E, k=k, policy=binding.SPREAD, topk_idx=gu.to_dev(idx),
                                    active=gu.to_dev(active), l2p_off=gu.to_dev(off),
                                    l2p_list=gu.to_dev(lst), out=out, T=T)
    want = oracle.step_layout(idx, p2l, active, E, R, S, S - 1, binding.SPREAD)
    for name in ("slot_of", "row_of", "src_of", "count", "offset", "cnt_src"):
        assert np.array_equal(out[name].cpu().numpy(), want[name].reshape(-1)), name
