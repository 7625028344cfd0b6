"""Dispatch of rows of just under, exactly and more than 4 GiB: byte offsets inside a row and from row to
row that take more than 32 bits.  Every moved row equals its token's."""
import numpy as np
import pytest
import torch

from paper_2605_10670_amd import binding

import gpu_util as gu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k,H", [(2, 1, 2**30 - 4), (2, 1, 2**30), (1, 2, 2**30 + 520)], ids=str)
def test_huge_rows(T, k, H):
    if torch.cuda.mem_get_info()[0] < 40 << 30:
        pytest.skip("needs 40 GiB of device memory")
    ctx = binding.Context(num_ranks=1, slots_per_rank=4, primary_slots=4, num_logical=4, max_tokens=T, topk=k,
                          hidden=H, x_dtype="f32", y_dtype="f32", out_dtype="f32")
    x = recv = None
    try:
        ctx.update_placement(np.arange(4, dtype=np.int32))
        ctx.dispatch_layout(gu.to_dev(np.array([[3, 1]] if k == 2 else [[3], [1]], np.int32)), T)
        x = torch.empty((T, H), dtype=torch.int32, device="cuda")
        for t in range(T):
            torch.arange(H, dtype=torch.int32, device="cuda", out=x[t]).mul_(2 * t + 3)
        recv = torch.full((T * k, H), -1, dtype=torch.int32, device="cuda")
        ctx.dispatch(x, recv, T)
        src = ctx.read("src_of", T * k)
        assert sorted(src) == list(range(T * k))
        for row in range(T * k):
            assert torch.equal(recv[row], x[src[row] // k]), row
    finally:
        ctx.destroy()
        del x, recv
        torch.cuda.empty_cache()
