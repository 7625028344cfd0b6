"""Combine at every compile-time top-k and at larger ones, which go in batches of 8, 4 and 1 rows: all pairs
routed, some dropped, tokens with no row at all, with failure detection and without, each data type of
rows and results, a row of less than and of more than one part.  Bit-equal to the oracle's fp32 chain."""
import numpy as np
import pytest
import torch

from paper_2605_10670_amd import binding

import gpu_util as gu
from test_gpu_layout_edges import instance

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("detect", [False, True])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 16, 23, 32])
def test_combine_topk(oracle, k, detect):
    R, S, E, T = 4, 12, 40, 24
    for (y, out, H), dropped in zip([("bf16", "bf16", 520), ("bf16", "f32", 64), ("f32", "f32", 516),
                                     ("f32", "bf16", 1032)], [True, False, False, True]):
        p2l, active, idx = instance(T, k, R, S, E, seed=k + H)
        if not dropped:
            p2l, active = np.arange(R * S, dtype=np.int32) % E, np.ones(R, np.int32)
            idx = np.argsort(np.random.default_rng(k).random((T, E)), axis=1)[:, :k].astype(np.int32)
        else:
            idx[5] = -1                                    # a token without any row
        ctx = binding.Context(num_ranks=R, slots_per_rank=S, primary_slots=S - 1, num_logical=E,
                              max_tokens=T, topk=k, hidden=H, x_dtype=y, y_dtype=y, out_dtype=out,
                              strict_coverage=False)
        try:
            ctx.update_placement(p2l)
            ctx.set_membership(active)
            if detect:
                ctx.set_detection(1_000_000_000)
            rng = np.random.default_rng(k * 100 + H)
            rows32 = rng.standard_normal((T * k, H), dtype=np.float32)
            rows = rows32 if y == "f32" else oracle.f32_to_bf16(rows32)
            w = rng.random((T, k), dtype=np.float32)
            ctx.dispatch_layout(gu.to_dev(idx), T)
            row_of = ctx.read("row_of", T * k).reshape(T, k)
            assert (row_of < 0).any() == dropped
            if detect:
                ctx.signal_experts_done()
            got = gu.dev_empty(T, H, out, fill=0)
            ctx.combine(gu.to_dev(rows), gu.to_dev(w), got, T)
            torch.cuda.synchronize()
            want = oracle.combine_chain32(rows, oracle.F32 if y == "f32" else oracle.BF16, w, row_of)
            if out == "bf16":
                want = oracle.f32_to_bf16(want)
            got = gu.to_host(got, gu.NP_OF[out])
            assert np.array_equal(got.view(np.uint8), want.view(np.uint8)), (y, out, H)
        finally:
            ctx.destroy()
