"""Dispatch and combine of batches of 512 tokens and more whose rows go in narrow pieces because they are few bytes, and
just beyond the limits of that: rows of less than a piece, of whole ones and with a remainder, tokens with dropped pairs.
Moved bytes equal, combine bit-equal to the fp32 chain."""
import numpy as np
import pytest
import torch

from paper_2605_10670_amd import binding

import gpu_util as gu
from test_gpu_layout_edges import instance

pytestmark = pytest.mark.gpu


# (T, k, H, x dtype): 6 MiB of tokens, 14 MiB of receive rows for k >= 4, and sizes around them
@pytest.mark.parametrize("T,k,H,dtype", [
    (512, 2, 1024, "bf16"), (512, 8, 1792, "bf16"), (513, 8, 1792, "bf16"), (700, 4, 2600, "bf16"), (1023, 7, 1000, "bf16"),
    (1024, 8, 896, "bf16"), (1025, 8, 904, "bf16"), (1024, 3, 3072, "bf16"), (1024, 3, 3080, "bf16"), (1500, 2, 2056, "bf16"),
    (3072, 2, 1024, "bf16"), (2000, 6, 24, "bf16"), (768, 4, 1032, "f32"), (1536, 2, 1024, "f32"), (600, 9, 1024, "bf16"),
    (2100, 1, 1024, "bf16")])
def test_dispatch_and_combine(oracle, T, k, H, dtype):
    R, S, E = 1, 24, 20
    p2l, _, idx = instance(T, k, R, S, E, seed=T + k + H)
    p2l[p2l == 3] = 4                                  # expert 3 has no replica: some pairs are dropped
    ctx = binding.Context(num_ranks=R, slots_per_rank=S, primary_slots=S - 1, num_logical=E, max_tokens=T, topk=k,
                          hidden=H, x_dtype=dtype, y_dtype=dtype, out_dtype="f32", strict_coverage=False)
    try:
        ctx.update_placement(p2l)
        ctx.dispatch_layout(gu.to_dev(idx), T)
        tdt = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
        x = torch.randn((T, H), device="cuda").to(tdt)
        recv = torch.full((T * k, H), 7.0, device="cuda", dtype=tdt)
        w = np.random.default_rng(T).random((T, k), dtype=np.float32)
        out = torch.full((T, H), 7.0, device="cuda")
        ctx.dispatch(x, recv, T)
        ctx.combine(recv, gu.to_dev(w), out, T)
        row_of, src, N = ctx.read("row_of", T * k), ctx.read("src_of", T * k), int(ctx.read("status", 4)[0])
        token = torch.from_numpy(src[:N] // k).cuda().long()
        assert torch.equal(recv[:N], x[token]) and bool((recv[N:] == 7.0).all())
        rows = recv.view(torch.int16).cpu().numpy().view(np.uint16) if dtype == "bf16" else recv.cpu().numpy()
        want = oracle.combine_chain32(rows, oracle.BF16 if dtype == "bf16" else oracle.F32, w, row_of.reshape(T, k))
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32))
    finally:
        ctx.destroy()
