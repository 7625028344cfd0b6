"""Layouts captured while their instance had one context and replayed when it has two: the workgroups of a
launch use one mask also where it changes meanwhile, and every launch leaves the words they agree
through as it found them.  Shares of whole ranks and of a part of one, few and many ranks, tables larger
than a workgroup."""
import numpy as np
import pytest
import torch

from paper_2605_10670_amd import binding

import gpu_util as gu
from test_gpu_layout_edges import instance

pytestmark = pytest.mark.gpu


# (R, S, E, k, batch sizes)
@pytest.mark.parametrize("R,S,E,k,sizes", [
    (32, 9, 256, 8, (256, 2048)), (8, 36, 256, 8, (2048, 512)), (2, 9, 16, 8, (1024, 256)), (1, 16, 16, 3, (5001,)),
    (48, 4, 96, 5, (480, 2496)), (65, 3, 130, 7, (585, 2340)), (200, 6, 1100, 4, (600, 4000)),
    (1000, 2, 500, 2, (1000, 8000)), (64, 9, 512, 10, (1024,)), (8, 140, 500, 4, (1024, 520)),
], ids=str)
def test_one_mask_for_all_workgroups(oracle, R, S, E, k, sizes):
    T_max = max(sizes)
    shape = dict(num_ranks=R, slots_per_rank=S, primary_slots=max(1, S - 1), num_logical=E, max_tokens=T_max, topk=k,
                 hidden=64, strict_coverage=False)
    p2l, active, idx = instance(T_max, k, R, S, E, seed=R + k)
    ctx, other = binding.Context(**shape), None
    stream, updates = torch.cuda.Stream(), torch.cuda.Stream()
    dev = gu.to_dev(idx)
    torch.cuda.synchronize()
    graphs = {}
    try:
        ctx.update_placement(p2l, stream)
        ctx.set_membership(active, stream)
        for T in sizes:
            ctx.dispatch_layout(dev, T, stream)
            stream.synchronize()
            ctx.graph_begin(stream)
            ctx.dispatch_layout(dev, T, stream)
            graphs[T] = ctx.graph_end(stream)
        other = binding.Context(**shape, parent=ctx)
        # ranks in turn, one at a time, so that a layout that runs meanwhile has one of two masks
        mask = active.copy()
        for step in range(12):
            before, mask = mask, mask.copy()
            mask[(step * 7) % R] ^= 1
            T = sizes[step % len(sizes)]
            graphs[T].launch(stream)
            other.set_membership(mask, updates)
            torch.cuda.synchronize()
            if T == sizes[-1]:                           # (the last one that was laid out in a call)
                assert ctx.check_layout(T).tolist() == [0, 0, 0, 0]
            got = ctx.read_layout(T)
            want = [oracle.step_layout(idx[:T], p2l, m, E, R, S, max(1, S - 1), binding.SPREAD) for m in (before, mask)]
            fits = [all(np.array_equal(got[key], w[key]) for key in gu.LAYOUT_KEYS) for w in want]
            assert any(fits), step
            graphs[T].launch(stream)                     # the mask is still now
            stream.synchronize()
            gu.assert_layout_equal(ctx.read_layout(T), want[1], T, k)
    finally:
        for graph in graphs.values():
            graph.destroy()
        if other is not None:
            other.destroy()
        ctx.destroy()


# (R, S, E, k, batch sizes): beyond one workgroup (384 tokens, 3072 pairs), at the limits of the one-launch form, and past them
@pytest.mark.parametrize("R,S,E,k,sizes", [
    (32, 9, 256, 8, (416, 512, 2048, 2080)), (2, 9, 16, 8, (1024, 386)), (1, 16, 16, 3, (385, 5461, 5462)),
    (48, 4, 96, 5, (3264, 480)), (65, 3, 130, 7, (455, 2340)), (1000, 2, 500, 2, (8000, 1000)), (64, 9, 512, 10, (384, 1600)),
    (8, 140, 500, 4, (1024, 776))], ids=str)
def test_launched_with_two_contexts(oracle, R, S, E, k, sizes):
    T_max = max(sizes)
    shape = dict(num_ranks=R, slots_per_rank=S, primary_slots=max(1, S - 1), num_logical=E, max_tokens=T_max, topk=k,
                 hidden=64, strict_coverage=False)
    p2l, active, idx = instance(T_max, k, R, S, E, seed=R + k + 1)
    ctx = binding.Context(**shape)
    other = binding.Context(**shape, parent=ctx)
    stream, updates = torch.cuda.Stream(), torch.cuda.Stream()
    dev = gu.to_dev(idx)
    torch.cuda.synchronize()
    try:
        ctx.update_placement(p2l, stream)
        ctx.set_membership(active, stream)
        stream.synchronize()
        mask = active.copy()
        for step in range(3 * len(sizes)):
            before, mask = mask, mask.copy()
            mask[(step * 7) % R] ^= 1
            T = sizes[step % len(sizes)]
            ctx.dispatch_layout(dev, T, stream)
            other.set_membership(mask, updates)
            torch.cuda.synchronize()
            assert ctx.check_layout(T).tolist() == [0, 0, 0, 0]
            got = ctx.read_layout(T)
            want = [oracle.step_layout(idx[:T], p2l, m, E, R, S, max(1, S - 1), binding.SPREAD) for m in (before, mask)]
            one_launch = T * k <= 16384 and R < 1000     # (tiles may send some pairs by one mask and some by the other)
            assert not one_launch or any(all(np.array_equal(got[key], w[key]) for key in gu.LAYOUT_KEYS) for w in want)
            ctx.dispatch_layout(dev, T, stream)          # the mask is still now
            stream.synchronize()
            gu.assert_layout_equal(ctx.read_layout(T), want[1], T, k)
    finally:
        other.destroy()
        ctx.destroy()
