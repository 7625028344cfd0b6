"""The expert stand-ins on their own: every code of the fp8 format, group sizes that are and are
not powers of two, streams that end inside a block, rows past N."""
import numpy as np
import pytest
import torch

from paper_2605_10670_amd import binding, synth

import gpu_util as gu

pytestmark = pytest.mark.gpu


def routed_context(T, H, k=2, masked=0, **kw):
    """Context with a layout of T tokens on 4 ranks x 2 slots, the last `masked` pairs dropped."""
    E, R = 8, 4
    ctx = binding.Context(num_ranks=R, slots_per_rank=2, primary_slots=2, num_logical=E, max_tokens=T,
                          topk=k, hidden=H, **kw)
    p2l = synth.preferred_placement(R, 2, 0)
    ctx.update_placement(p2l)
    idx = np.stack([np.random.default_rng(T + H + t).permutation(E)[:k] for t in range(T)])
    idx = idx.astype(np.int32)
    if masked:
        idx.reshape(-1)[-masked:] = -1
    ctx.dispatch_layout(gu.to_dev(idx), T)
    return ctx, p2l, idx


# 512 vectors of 8 codes per block: streams of less than one block, of exactly one and of
# several, with 0, 1 and many vectors left over
@pytest.mark.parametrize("T,H,group,masked", [(4, 64, 16, 1), (4, 512, 128, 0), (32, 512, 128, 5),
                                              (12, 192, 48, 0), (44, 1152, 96, 3), (36, 192, 48, 1),
                                              (64, 7168, 128, 7), (20, 6400, 1600, 2)])
def test_dequant_stand_in(oracle, T, H, group, masked):
    k = 2
    ctx, _, _ = routed_context(T, H, k, masked, x_dtype="fp8", scale_group=group)
    try:
        rng = np.random.default_rng(H)
        q = rng.permutation(np.resize(np.arange(256, dtype=np.uint8), T * k * H)).reshape(T * k, H)
        sc = np.exp(rng.uniform(-20, 5, (T * k, H // group))).astype(np.float32)
        sc[0, 0] = 1e-41                       # a subnormal scale
        y = gu.dev_empty(T * k, H, "bf16", fill=0x1234)
        ctx.expert_stub("dequant", gu.to_dev(q), y, T, recv_scale=gu.to_dev(sc))
        N = T * k - masked
        got = gu.to_host(y, np.uint16)
        want = oracle.stub_dequant(q, sc, N, group)
        nan = (q & 0x7f) == 0x7f               # both NaN codes, quiet, with the code's sign
        assert ((want[:N] & 0x7fff) > 0x7f80)[nan[:N]].all()
        want[nan] = 0x7fc0 | ((q[nan].astype(np.uint16) & 0x80) << 8)
        assert np.array_equal(got[:N], want[:N])
        assert (got[N:] == 0x1234).all(), "rows past N were written"
    finally:
        ctx.destroy()


# row sizes around whole passes: 1 vector, one short of / exactly / one past 64 and 128 vectors, a
# prime number of 64-vector sets above 14, an odd remainder; small batches split rows over
# wavefronts, 1024 tokens and more do not; 8192 rows change the expansion's width, and so do more
# than 1024 vectors (16 KiB)
@pytest.mark.parametrize("vecs", [1, 63, 64, 65, 128, 129, 360, 15 * 64, 1024, 17 * 64, 17 * 64 - 3,
                                  24 * 64])
@pytest.mark.parametrize("T", [4, 1020, 1024])
def test_pack_and_expand_row_shapes(T, vecs):
    H, k = vecs * 4, 8                      # fp32 rows: 4 channels per 16-byte vector
    ctx, _, _ = routed_context(T, H, k, 5, x_dtype="f32", y_dtype="f32", out_dtype="f32")
    try:
        x = torch.randint(-2**31, 2**31 - 1, (T, H), dtype=torch.int32, device="cuda")
        recv, recv_d, recv_e = (torch.full((T * k, H), 77, dtype=torch.int32, device="cuda")
                                for _ in range(3))
        ctx.dispatch(x, recv, T)
        lay = ctx.read_layout(T)
        N = lay["N"]
        tok = torch.from_numpy(lay["src_of"][:N] // k).long().cuda()
        assert torch.equal(recv[:N], x[tok]) and (recv[N:] == 77).all()
        ctx.dedup_layout(T)
        ctx.dispatch_dedup(x, recv_d, T)
        ctx.expand(recv_d, recv_e, T)
        assert torch.equal(recv_e[:N], x[tok]) and (recv_e[N:] == 77).all()
        assert (recv_d[ctx.read_dedup(T)["N_d"]:] == 77).all()
    finally:
        ctx.destroy()


# rows of 1, 64, 65 and several passes of 64 x 16 channels; 1 to 64 lanes per group; the form with
# a wavefront per 64 vectors (below 1024 tokens) and the one with a wavefront per token
@pytest.mark.parametrize("T,H,group", [(4, 64, 16), (8, 1024, 16), (4, 7168, 128), (8, 1280, 64),
                                       (12, 2048, 512), (4, 8192, 1024), (1028, 512, 64),
                                       (1024, 7168, 128), (1024, 8192, 256)])
def test_dispatch_quant_forms(oracle, T, H, group):
    k = 2
    ctx, _, _ = routed_context(T, H, k, 3, x_dtype="fp8", scale_group=group)
    try:
        rng = np.random.default_rng(T + H)
        x = rng.standard_normal((T, H)).astype(np.float32)
        x *= np.exp2(rng.integers(-130, 120, (T, H // group))).repeat(group, axis=1).astype(np.float32)
        x[0] = np.exp2(rng.integers(-20, 4, H)).astype(np.float32)     # ties and tiny quotients
        x[1, :group] = 0.0
        bits = synth.f32_to_bf16_bits(x)
        bits[2] = rng.integers(0, 0x7f80, H) | (rng.integers(0, 2, H) << 15)   # any finite bf16
        bits[3, ::7] = 0x8000                                          # negative zeros
        recv = gu.dev_empty(T * k, H, "fp8", fill=0x5a)
        sc = torch.full((T * k, H // group), -7.0, device="cuda")
        ctx.dispatch_quant(gu.to_dev(bits), recv, sc, T)
        lay = ctx.read_layout(T)
        q, want_sc = oracle.quantize_e4m3(bits, group)
        N = lay["N"]
        assert N == T * k - 3
        tok = lay["src_of"][:N] // k
        assert np.array_equal(recv.cpu().numpy()[:N], q[tok])
        assert np.array_equal(sc.cpu().numpy()[:N].view(np.uint32), want_sc[tok].view(np.uint32))
        assert (recv.cpu().numpy()[N:] == 0x5a).all() and (sc.cpu().numpy()[N:] == -7.0).all()
    finally:
        ctx.destroy()


@pytest.mark.parametrize("T", [4, 1024])
def test_dispatch_quant_with_infinities_and_nan(T):
    """A group with an infinity has an infinite scale: finite channels become zeros, infinities the
    NaN code; NaN channels become the NaN code and do not raise the scale."""
    H, group, k = 512, 128, 2
    ctx, _, _ = routed_context(T, H, k, 0, x_dtype="fp8", scale_group=group)
    try:
        x = np.ones((T, H), np.float32)
        x[:, 5] = -np.inf
        x[:, group + 3] = np.nan
        x[:, 2 * group:3 * group] = 3e38
        bits = synth.f32_to_bf16_bits(x)
        bits[:, group + 3] = 0x7fc0
        recv = gu.dev_empty(T * k, H, "fp8", fill=0)
        sc = torch.zeros((T * k, H // group), device="cuda")
        ctx.dispatch_quant(gu.to_dev(bits), recv, sc, T)
        got, s = recv.cpu().numpy(), sc.cpu().numpy()
        assert np.isinf(s[:, 0]).all() and (got[:, 5] & 0x7f == 0x7f).all()
        assert (np.delete(got[:, :group], 5, axis=1) == 0).all()
        assert (s[:, 1] == np.float32(1) / np.float32(448)).all() and (got[:, group + 3] == 0x7f).all()
        assert (np.delete(got[:, group:2 * group], 3, axis=1) == 0x7e).all()
        assert (got[:, 2 * group:3 * group] == 0x7e).all() and (got[:, 3 * group:] == 0x7e).all()
    finally:
        ctx.destroy()


# more pairs than the eight row indices that a split wavefront fetches at once: one and two past
# them, two and four sets; pieces of one vector per lane (below 512 tokens), of two (below 1024)
# and whole rows, with and without a remainder; pairs without a row in every set
@pytest.mark.parametrize("k", [8, 9, 10, 16, 17, 32])
@pytest.mark.parametrize("T,vecs", [(4, 128), (508, 192), (508, 360), (512, 256), (1020, 200), (1020, 449),
                                    (1024, 200)])
def test_pack_of_many_pairs(T, vecs, k):
    R, S, H = 4, 10, vecs * 4
    ctx = binding.Context(num_ranks=R, slots_per_rank=S, primary_slots=S, num_logical=R * S,
                          max_tokens=T, topk=k, hidden=H, x_dtype="f32", y_dtype="f32", out_dtype="f32")
    try:
        ctx.update_placement(synth.preferred_placement(R, S, 0))
        rng = np.random.default_rng(T + vecs + k)
        idx = np.argsort(rng.random((T, R * S)), axis=1)[:, :k].astype(np.int32)
        idx[::2, 5] = -1
        idx[1::3, k - 1] = -1
        idx[::4, min(8, k - 1)] = -1
        idx[T - 1] = -1
        ctx.dispatch_layout(gu.to_dev(idx), T)
        x = torch.randint(-2**31, 2**31 - 1, (T, H), dtype=torch.int32, device="cuda")
        recv = torch.full((T * k, H), 77, dtype=torch.int32, device="cuda")
        ctx.dispatch(x, recv, T)
        lay = ctx.read_layout(T)
        N = lay["N"]
        assert N == (idx >= 0).sum()
        tok = torch.from_numpy(lay["src_of"][:N] // k).long().cuda()
        assert torch.equal(recv[:N], x[tok]) and (recv[N:] == 77).all()
    finally:
        ctx.destroy()


# row sizes of one part, of two, of an odd number and ending inside one, on both sides of the token
# counts between which combine takes parts in pairs; small whole numbers, so every order is exact
@pytest.mark.parametrize("vecs", [64, 65, 128, 129, 192, 360])
@pytest.mark.parametrize("T", [508, 512, 516, 1020, 1024])
@pytest.mark.parametrize("k,detect", [(2, False), (2, True), (3, False), (8, True)])
def test_combine_row_shapes(T, vecs, k, detect):
    H = vecs * 4
    ctx, _, _ = routed_context(T, H, k, 5, x_dtype="f32", y_dtype="f32", out_dtype="f32")
    try:
        y = torch.randint(-99, 100, (T * k, H), device="cuda").float()
        w = torch.randint(1, 9, (T, k), device="cuda").float()
        out = torch.full((T + 1, H), 0.5, device="cuda")
        if detect:
            ctx.set_detection(200_000_000)
            ctx.signal_experts_done()
        ctx.combine(y, w, out, T)
        row = torch.from_numpy(ctx.read_layout(T)["row_of"].reshape(T, k)).long().cuda()
        want = ((w * (row >= 0)).unsqueeze(2) * y[row.clamp(min=0)]).sum(1)
        assert torch.equal(out[:T], want) and (out[T] == 0.5).all()
    finally:
        ctx.destroy()


def test_combine_of_more_wavefronts_than_one_launch_takes():
    """2^25 + 1 tokens whose rows end one vector past a part: 2^26 + 2 wavefronts of 64 lanes, more
    than the 2^32 lanes that a grid dimension may have."""
    T, H = 2**25 + 1, 520
    ctx = binding.Context(num_ranks=1, slots_per_rank=1, primary_slots=1, num_logical=1,
                          max_tokens=T, topk=1, hidden=H)
    try:
        ctx.update_placement(np.zeros(1, np.int32))
        y = torch.randint(0, 0x7f00, (T, H), dtype=torch.int16, device="cuda")   # finite bf16
        out = torch.empty_like(y)
        ctx.dispatch_layout(torch.zeros((T, 1), dtype=torch.int32, device="cuda"), T)
        ctx.combine(y, torch.ones((T, 1), device="cuda"), out, T)
        assert torch.equal(out, y)
    finally:
        ctx.destroy()
        y = out = None
        torch.cuda.empty_cache()            # (70 GB)


def test_stand_ins_of_more_rows_than_one_launch_takes():
    """2^24 + 3 rows at 256 lanes each; masked tokens at the end."""
    T, H, masked = 2**24 + 3, 8, 2
    ctx = binding.Context(num_ranks=1, slots_per_rank=1, primary_slots=1, num_logical=1,
                          max_tokens=T, topk=1, hidden=H)
    try:
        ctx.update_placement(np.zeros(1, np.int32))
        idx = torch.zeros((T, 1), dtype=torch.int32, device="cuda")
        idx[-masked:] = -1
        x = torch.randint(0, 0x7f00, (T, H), dtype=torch.int16, device="cuda")
        recv, y = (torch.full((T, H), 77, dtype=torch.int16, device="cuda") for _ in range(2))
        N = T - masked
        ctx.dispatch_layout(idx, T)
        ctx.dispatch(x, recv, T)
        assert torch.equal(recv[:N], x[:N]) and (recv[N:] == 77).all()
        for kind in ("identity", "scale"):
            y.fill_(77)
            ctx.expert_stub(kind, recv, y, T, expert_scale=torch.ones(1, device="cuda"))
            assert torch.equal(y[:N], x[:N]) and (y[N:] == 77).all(), kind
    finally:
        ctx.destroy()
