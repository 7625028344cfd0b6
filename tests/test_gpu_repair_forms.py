"""Weight movement in each of its forms: the whole repair in one launch (shorter and longer move lists and tables) and as
three, reloads from host memory by few workgroups and from device memory by many, slots of less than a workgroup's
vectors, of whole chunks and with a ragged tail, sources that dropped out, nothing to move.  Byte-exact, the tables, their
version, and the layout that follows from them."""
import numpy as np
import pytest
import torch

from paper_2605_10670_amd import binding

import gpu_util as gu
from test_gpu_repair_moves import _context, _expect, _run, _store

pytestmark = pytest.mark.gpu


# (R, S, E): 3 * moves + 2 * R * S + E + 1 words; 320 and 960 are the limits
@pytest.mark.parametrize("pinned", [False, True])
@pytest.mark.parametrize("R,S,E,peers,reloads,slot_bytes", [
    (4, 3, 8, 0, 0, 64), (4, 3, 8, 0, 1, 16), (4, 3, 8, 2, 0, 4112), (4, 3, 8, 0, 7, 65536), (8, 10, 120, 3, 10, 4096),
    (8, 10, 120, 4, 9, 4096 * 63), (8, 10, 120, 4, 10, 4096 * 64 + 16), (8, 10, 120, 5, 11, 4096 * 65 - 16),
    (16, 20, 301, 2, 4, 65552), (16, 20, 301, 3, 4, 65552), (16, 20, 301, 0, 9, 1 << 18), (16, 20, 301, 9, 0, 1 << 18),
    (16, 40, 400, 20, 70, 4112)])
def test_forms(oracle, R, S, E, peers, reloads, slot_bytes, pinned):
    rng = np.random.default_rng(R + E + peers + reloads)
    P = R * S
    cur = rng.permutation(np.concatenate([np.arange(min(E, P // 2)), np.full(P - min(E, P // 2), -1)])).astype(np.int32)
    full, empty = rng.permutation(np.nonzero(cur >= 0)[0]), rng.permutation(np.nonzero(cur < 0)[0])
    kind = np.where(cur >= 0, binding.SRC_LOCAL, binding.SRC_NONE).astype(np.int32)
    p2l, src = cur.copy(), np.full(P, -1, np.int32)
    for i, slot in enumerate(empty[:peers]):
        p2l[slot], kind[slot], src[slot] = cur[full[i % full.size]], binding.SRC_PEER, full[i % full.size]
    for slot in np.concatenate([empty[peers:], full[peers:]])[:reloads]:
        p2l[slot], kind[slot] = rng.integers(E), binding.SRC_DRAM
    active = np.ones(R, np.int32)
    if peers > 2:
        active[full[0] // S] = 0                       # that copy comes from the backup instead
    weights, backup = _store(rng, cur, E, slot_bytes)
    ctx = _context(R, S, S, E)
    try:
        ctx.update_placement(cur)
        ctx.set_membership(active)
        idx = torch.from_numpy(rng.integers(0, E, size=(4 * R, min(2, E)), dtype=np.int32)).cuda()
        ctx.dispatch_layout(idx, 4 * R)
        version = int(ctx.read("status", 4)[3])
        plan = dict(p2l=p2l, kind=kind, src_slot=src)
        got_w, got_o = _run(ctx, weights, backup, plan, slot_bytes, pinned)
        want_w, want_o = _expect(weights, backup, plan, active, S)
        assert np.array_equal(got_o, want_o)
        assert np.array_equal(got_w, want_w)
        tables = {f: ctx.read(f, n) for f, n in (("phys_to_logical", P), ("l2p_off", E + 1), ("l2p_list", P))}
        other = _context(R, S, S, E)
        try:
            other.update_placement(p2l)
            for field, got in tables.items():
                assert np.array_equal(got, other.read(field, got.size)), field
        finally:
            other.destroy()
        ctx.dispatch_layout(idx, 4 * R)
        gu.assert_layout_equal(ctx.read_layout(4 * R), oracle.step_layout(idx.cpu().numpy(), p2l, active, E, R, S, S,
                                                                          oracle.SPREAD), 4 * R, min(2, E))
        assert int(ctx.read("status", 4)[3]) == version + 1
    finally:
        ctx.destroy()
