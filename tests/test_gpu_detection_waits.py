"""What a combine that waits for signals does with the rows it waited for: every part of a token's
row leaves out the pairs of a dropped rank, and outputs that arrive while the kernel waits are the
ones it sums.  Expected values: the same combine without detection, on the rows that are left."""
import time

import numpy as np
import pytest
import torch

from paper_2605_10670_amd import binding, synth

import gpu_util as gu

pytestmark = pytest.mark.gpu


def _context(T, H, k, R=32, E=256):
    ctx = binding.Context(num_ranks=R, slots_per_rank=E // R, primary_slots=E // R, num_logical=E,
                          max_tokens=T, topk=k, hidden=H, strict_coverage=False)
    ctx.update_placement(synth.preferred_placement(R, E // R, 0))
    g = torch.Generator(device="cuda").manual_seed(T + H + k)
    idx = torch.topk(torch.rand((T, E), generator=g, device="cuda"), k, dim=1)[1].to(torch.int32)
    w = torch.rand((T, k), generator=g, device="cuda")
    x = torch.randn((T, H), generator=g, device="cuda").to(torch.bfloat16)
    return ctx, idx.contiguous(), w, x


# More wavefronts than the chip holds at once, so that many start while others time out; with a
# masked pair in every other token, and with every pair routed.
@pytest.mark.parametrize("k", [8, 4, 3])
@pytest.mark.parametrize("masked", [False, True])
def test_all_parts_of_a_row_leave_out_a_dropped_rank(k, masked):
    T, H, R, silent = 2048, 7168, 32, 6
    ctx, idx, w, x = _context(T, H, k)
    try:
        if masked:
            idx[::2, 0] = -1
        recv = torch.zeros((T * k, H), dtype=torch.bfloat16, device="cuda")
        out, want = (torch.empty((T, H), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        hold = np.zeros(R, np.int32)
        hold[silent] = 1
        ctx.debug_withhold_signal(hold)
        for trial in range(8):
            ctx.set_detection(200_000)
            ctx.dispatch_layout(idx, T)
            ctx.dispatch(x, recv, T)
            ctx.signal_experts_done()
            ctx.combine(recv, w, out, T)
            assert ctx.read_failures().tolist() == hold.tolist()
            got = ctx.read_layout(T)
            gone = got["slot_of"] // (256 // R) == silent
            assert gone.any() and np.array_equal(got["row_of"] < 0, (got["slot_of"] < 0) | gone)
            ctx.set_detection(0)
            ctx.combine(recv, w, want, T)
            differ = (out.view(torch.int16) != want.view(torch.int16)).any(dim=1)
            assert not differ.any(), f"trial {trial}: {int(differ.sum())} tokens"
            ctx.set_membership(np.ones(R, np.int32))
    finally:
        ctx.destroy()


# (rows of two whole parts, and of one part and a single vector: fewer lanes than pairs)
@pytest.mark.parametrize("k", [1, 2, 3, 4, 6, 8, 20])
@pytest.mark.parametrize("masked,H", [(False, 1024), (True, 1024), (True, 520)])
def test_outputs_that_arrive_while_combine_waits(k, masked, H):
    T, R = 64, 32
    ctx, idx, w, x = _context(T, H, k)
    try:
        if masked:
            idx[::2, 0] = -1
        recv = torch.zeros((T * k, H), dtype=torch.bfloat16, device="cuda")
        y = torch.zeros_like(recv)
        out, want = (torch.empty((T, H), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        y.copy_(recv)                       # (the copy kernel is loaded before anything waits)
        ctx.signal_experts_done()
        torch.cuda.synchronize()
        # Streams share a few hardware queues; two on one queue do not overlap, the wait then
        # runs into its time-out, and the next pair of streams is tried.
        for _ in range(16):
            main, side = torch.cuda.Stream(), torch.cuda.Stream()
            ctx.dispatch_layout(idx, T, main)
            ctx.dispatch(x, recv, T, stream=main)
            y.zero_()
            torch.cuda.synchronize()
            ctx.set_detection(100_000_000)
            ctx.combine(y, w, out, T, main)     # waits: no rank has signalled this step
            time.sleep(0.005)
            with torch.cuda.stream(side):
                y.copy_(recv)                   # the experts' outputs of the step ...
            ctx.signal_experts_done(side)       # ... and their signals
            torch.cuda.synchronize()
            if ctx.read_failures(main).sum() == 0:
                break
            ctx.set_membership(np.ones(R, np.int32))
            torch.cuda.synchronize()
        else:
            raise AssertionError("no two streams overlapped")
        ctx.set_detection(0)
        ctx.combine(y, w, want, T, main)
        torch.cuda.synchronize()
        assert torch.equal(out.view(torch.int16), want.view(torch.int16)), "sums of stale rows"
    finally:
        ctx.destroy()
