"""A rank that leaves the mask while a repair copies from it: a slot's outcome names where its first bytes came from, whenever
in the copy that was."""
import numpy as np
import pytest
import torch

from oracle import planner as ref
from paper_2605_10670_amd import binding, synth

from test_gpu_repair_moves import _context

pytestmark = pytest.mark.gpu


# (slots per rank, moves, bytes): one launch with the tables, 64 workgroups to a slot; and the moves in a launch of their own, 4 to
# a slot.  Either way there are more workgroups than the GPU holds at once, so they look at the mask at different times.
@pytest.mark.parametrize("S,moves,slot_bytes", [(40, 70, 4 << 20), (500, 1470, 4 * 65536)])
def test_outcome_of_sources_that_leave_meanwhile(S, moves, slot_bytes):
    R, E, gone = 4, 30, 1
    P = R * S
    p2l = np.full(P, -1, np.int32)
    held = np.arange(gone * S, gone * S + min(E, S))              # rank 1 holds everything, the others are empty
    p2l[held] = np.arange(held.size)
    plan = dict(p2l=p2l.copy(), kind=np.where(p2l >= 0, binding.SRC_LOCAL, binding.SRC_NONE).astype(np.int32),
                src_slot=np.full(P, -1, np.int32))
    to = np.nonzero(p2l < 0)[0]
    to = to[to // S != gone][:moves]
    source = held[np.arange(to.size) % held.size]
    plan["p2l"][to], plan["kind"][to], plan["src_slot"][to] = p2l[source], binding.SRC_PEER, source
    live, dead = synth.active_mask(R), synth.active_mask(R, (gone,))
    weights = torch.zeros((P, slot_bytes), dtype=torch.uint8, device="cuda")
    backup = torch.full((E, slot_bytes), 2, dtype=torch.uint8, device="cuda")
    ctx = _context(R, S, S, E)
    copying, other = torch.cuda.Stream(), torch.cuda.Stream()
    try:
        for _ in range(6):
            weights.zero_()
            weights[torch.from_numpy(held).cuda()] = 1            # 1: from a slot, 2: from the backup
            ctx.update_placement(p2l)
            ctx.set_membership(live)
            torch.cuda.synchronize()
            ctx.apply_repair(weights, backup, slot_bytes, plan, stream=copying)
            ctx.set_membership(dead, stream=other)
            outcome = ctx.read_repair_outcome()
            first = weights[:, 0].cpu().numpy()
            assert (outcome[to] == np.where(first[to] == 1, ref.FROM_PEER, ref.FROM_DRAM_FALLBACK)).all()
            assert set(first[to]) <= {1, 2} and not outcome[np.setdiff1d(np.arange(P), to)].any()
    finally:
        ctx.destroy()
