"""Combine of more than ten rows a token where some pairs have none: what stands in a row that is not the token's own, a
NaN among them, does not reach its result.  With failure detection and without."""
import numpy as np
import pytest
import torch

from paper_2605_10670_amd import binding

import gpu_util as gu
from test_gpu_layout_edges import instance

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("detect", [False, True])
@pytest.mark.parametrize("k,y", [(11, "bf16"), (12, "f32"), (16, "bf16"), (23, "f32"), (32, "bf16")])
def test_foreign_rows_stay_out(oracle, k, y, detect):
    R, S, E, T, H = 4, 12, 40, 96, 1032
    p2l, active, idx = instance(T, k, R, S, E, seed=k)
    idx[3] = -1                                        # no row at all
    idx[4, 1:] = -1                                    # one, the first
    idx[5, : k - 1] = -1                               # one, the last
    ctx = binding.Context(num_ranks=R, slots_per_rank=S, primary_slots=S - 1, num_logical=E, max_tokens=T, topk=k,
                          hidden=H, x_dtype=y, y_dtype=y, out_dtype="f32", strict_coverage=False)
    try:
        ctx.update_placement(p2l)
        ctx.set_membership(active)
        if detect:
            ctx.set_detection(1_000_000_000)
        ctx.dispatch_layout(gu.to_dev(idx), T)
        row_of = ctx.read("row_of", T * k).reshape(T, k)
        rng = np.random.default_rng(k)
        rows = rng.standard_normal((T * k, H), dtype=np.float32)
        hit = [0, *row_of[row_of >= 0][::37]]
        rows[hit] = np.nan
        bits = rows if y == "f32" else oracle.f32_to_bf16(rows)
        w = rng.random((T, k), dtype=np.float32)
        if detect:
            ctx.signal_experts_done()
        out = gu.dev_empty(T, H, "f32", fill=0)
        ctx.combine(gu.to_dev(bits), gu.to_dev(w), out, T)
        torch.cuda.synchronize()
        got = out.cpu().numpy()
        of_token = np.isin(row_of, hit).any(axis=1)
        assert of_token.any() and not of_token.all() and (row_of < 0).any(axis=1)[~of_token].any()
        assert np.array_equal(np.isnan(got).all(axis=1), of_token) and np.array_equal(np.isnan(got).any(axis=1), of_token)
        want = oracle.combine_chain32(bits, oracle.F32 if y == "f32" else oracle.BF16, w, row_of)
        assert np.array_equal(got[~of_token].view(np.uint32), want[~of_token].view(np.uint32))
    finally:
        ctx.destroy()
