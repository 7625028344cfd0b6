"""Dispatch of small batches, where a row is spread over wavefronts: every compile-time top-k and the
general one, rows of less than a piece, of whole pieces and with a remainder, batch sizes at which the
pieces change, and fp8 scale rows of one to more than 64 vectors in the payload's launch and just
beyond it.  Moved bytes equal, rows past the last routed pair untouched."""
import numpy as np
import pytest
import torch

from paper_2605_10670_amd import binding

import gpu_util as gu
from test_gpu_layout_edges import instance

pytestmark = pytest.mark.gpu

# (T, k, H, x dtype)
CASES = ([(64, k, 1536, "bf16") for k in range(1, 11)] + [(32, k, 1024, "fp8") for k in range(1, 11)] +
         [(31, 4, 8, "bf16"), (511, 2, 520, "bf16"), (512, 8, 512, "bf16"), (512, 3, 1544, "bf16"),
          (1023, 2, 1032, "bf16"), (1024, 2, 2880, "bf16"), (40, 5, 1032, "f32"), (16, 8, 33280, "fp8"),
          (511, 6, 512, "fp8"), (512, 8, 1536, "fp8"), (1023, 2, 2560, "fp8"), (1024, 3, 2560, "fp8"),
          (1025, 8, 512, "fp8"), (24, 12, 4608, "fp8")])


@pytest.mark.parametrize("T,k,H,dtype", CASES)
def test_small_batch_dispatch(T, k, H, dtype):
    R, S, E = 1, 24, 20
    p2l, _, idx = instance(T, k, R, S, E, seed=T + k + H)
    p2l[p2l == 3] = 4                                  # expert 3 has no replica: some pairs are dropped
    size = {"f32": 4, "bf16": 2, "fp8": 1}[dtype]
    ctx = binding.Context(num_ranks=R, slots_per_rank=S, primary_slots=S - 1, num_logical=E, max_tokens=T,
                          topk=k, hidden=H, x_dtype=dtype, y_dtype="f32" if dtype == "f32" else "bf16",
                          strict_coverage=False)
    try:
        ctx.update_placement(p2l)
        ctx.dispatch_layout(gu.to_dev(idx), T)
        rng = np.random.default_rng(T)
        x = rng.integers(0, 256, (T, H * size), dtype=np.uint8)
        recv = torch.full((T * k, H * size), 0x5A, dtype=torch.uint8, device="cuda")
        scales = {}
        if dtype == "fp8":
            sc = rng.random((T, H // 128), dtype=np.float32)
            recv_sc = torch.full((T * k, H // 128), -1.0, device="cuda")
            scales = dict(x_scale=gu.to_dev(sc), recv_scale=recv_sc)
        ctx.dispatch(gu.to_dev(x), recv, T, **scales)
        src, N = ctx.read("src_of", T * k), ctx.read("status", 4)[0]
        assert N < T * k or k == 1
        got = recv.cpu().numpy()
        assert np.array_equal(got[:N], x[src[:N] // k]) and (got[N:] == 0x5A).all()
        if dtype == "fp8":
            got = recv_sc.cpu().numpy()
            assert np.array_equal(got[:N], sc[src[:N] // k]) and (got[N:] == -1.0).all()
    finally:
        ctx.destroy()
