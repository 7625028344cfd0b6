"""The one-launch layout of batches whose tokens are no ordinary router's: copies of one token, padding that names no
expert at the end, scattered or in every pair, an expert that all tokens name first or last, repeats.  Fields equal to
the oracle's, among them the numbers of dropped pairs."""
import numpy as np
import pytest

from paper_2605_10670_amd import binding

import gpu_util as gu
from test_gpu_layout_edges import instance

pytestmark = pytest.mark.gpu


def batch(kind, idx, E, rng):
    T, k = idx.shape
    out = idx.copy()
    if kind == "same":
        out[:] = out[T // 2]
    elif kind == "half the same":
        out[T // 3:] = out[T // 3]
    elif kind == "first the same":
        out[:, 0] = E - 1
    elif kind == "last the same":
        out[:, -1] = E // 2
    elif kind == "most the same":
        out[:, : k // 2 + 1] = np.arange(k // 2 + 1)
    elif kind == "end padded":
        out[T // 5 + 1:] = -1
    elif kind == "all padded":
        out[:] = E
    elif kind == "tokens padded":
        out[rng.random(T) < 0.5] = -1
    elif kind == "pairs padded":
        out[rng.random((T, k)) < 0.5] = -1
    elif kind == "repeats":
        out[:, k // 2:] = out[:, : k - k // 2]
    return out


# (T, k, R, S, E): shares of several ranks, of one, of a part of one; a pair to a token; tables larger than a workgroup
@pytest.mark.parametrize("kind", ["same", "half the same", "first the same", "last the same", "most the same",
                                  "end padded", "all padded", "tokens padded", "pairs padded", "repeats"])
@pytest.mark.parametrize("shape", [(1984, 8, 32, 9, 256), (1610, 10, 2, 9, 16), (1024, 5, 4, 6, 16), (8000, 2, 16, 6, 40),
                                   (16384, 1, 64, 2, 100), (600, 2, 150, 8, 1100)], ids=str)
def test_skewed_layouts(oracle, shape, kind):
    T, k, R, S, E = shape
    p2l, active, idx = instance(T, k, R, S, E, seed=T + k)
    idx = batch(kind, idx, E, np.random.default_rng(T))
    ctx = binding.Context(num_ranks=R, slots_per_rank=S, primary_slots=max(1, S - 1), num_logical=E, max_tokens=T,
                          topk=k, hidden=64, strict_coverage=False)
    try:
        ctx.update_placement(p2l)
        ctx.set_membership(active)
        ctx.dispatch_layout(gu.to_dev(idx), T)
        got = ctx.read_layout(T)
        want = oracle.step_layout(idx, p2l, active, E, R, S, max(1, S - 1), binding.SPREAD)
        gu.assert_layout_equal(got, want, T, k)
        assert (got["n_uncovered"], got["n_masked"]) == (want["n_uncovered"], want["n_masked"])
    finally:
        ctx.destroy()
