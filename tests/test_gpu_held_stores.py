"""Stores that are held in the L2s: a dispatch in one node with its layout, by who reads its rows; expansion and the scaling stand-in at the limits
of the sizes at which they hold theirs (in captured steps only), and one step to either side.  Beside them a dispatch of its own and quantisation, which
never do, at the same sizes, in every form (whole rows, pieces of one and two kilobytes, rows with a remainder, scale rows, a
group that needs the division).  Moved bytes equal, rows past the last routed pair untouched."""
import re
import subprocess

import numpy as np
import pytest
import torch

from paper_2605_10670_amd import binding, build

import gpu_util as gu
from test_gpu_layout_edges import instance
from test_gpu_layout_pack import Step, kernel_of, last_node

gpu = pytest.mark.gpu


def context(T, k, H, R=1, **kw):
    S, E = 24 // R, 20
    p2l, _, idx = instance(T, k, R, S, E, seed=T + k + H)
    p2l[p2l == 3] = 4                                  # expert 3 has no replica: some pairs are dropped
    ctx = binding.Context(num_ranks=R, slots_per_rank=S, primary_slots=S - 1, num_logical=E, max_tokens=T, topk=k,
                          hidden=H, strict_coverage=False, **kw)
    ctx.update_placement(p2l)
    ctx.dispatch_layout(gu.to_dev(idx), T)
    src = torch.from_numpy(ctx.read("src_of", T * k)).cuda().long()
    return ctx, src, int(ctx.read("status", 4)[0])


def random_rows(T, H, dtype):
    size = {"f32": 4, "bf16": 2, "fp8": 1}[dtype]
    return torch.randint(0, 256, (T, H * size), dtype=torch.uint8, device="cuda")


def launch(ctx, captured, call):
    """The call by itself, or captured and replayed."""
    if not captured:
        return call(None)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    ctx.graph_begin(stream)
    call(stream)
    graph = ctx.graph_end(stream)
    graph.launch(stream)
    stream.synchronize()
    graph.destroy()


# (T, k, H, x dtype): receive rows of 13.9 to 26.1 MiB (fp8 3.9 to 13.1), around 512 and 1024 tokens
@gpu
@pytest.mark.parametrize("T,k,H,dtype", [
    (224, 4, 8128, "bf16"), (226, 4, 8136, "bf16"), (160, 8, 7168, "bf16"), (500, 6, 2880, "bf16"),
    (511, 8, 3328, "bf16"), (600, 5, 3080, "bf16"), (1000, 8, 1024, "bf16"), (1024, 8, 1024, "bf16"),
    (1100, 9, 1288, "bf16"), (3000, 4, 520, "f32"), (1660, 8, 1024, "bf16"), (1670, 8, 1024, "bf16"),
    (300, 12, 3584, "bf16"), (73, 8, 7168, "fp8"), (74, 8, 7168, "fp8"), (600, 8, 2048, "fp8"), (1024, 8, 1536, "fp8"),
    (1070, 8, 1536, "fp8"), (1150, 8, 1536, "fp8")])
def test_dispatch(T, k, H, dtype):
    ctx, src, N = context(T, k, H, x_dtype=dtype, y_dtype="f32" if dtype == "f32" else "bf16")
    try:
        x = random_rows(T, H, dtype)
        recv = torch.full((T * k, x.shape[1]), 0x5A, dtype=torch.uint8, device="cuda")
        scales = {}
        if dtype == "fp8":
            scales = dict(x_scale=torch.rand((T, H // 128), device="cuda"),
                          recv_scale=torch.full((T * k, H // 128), -1.0, device="cuda"))
        ctx.dispatch(x, recv, T, **scales)
        assert N < T * k
        assert torch.equal(recv[:N], x[src[:N] // k]) and bool((recv[N:] == 0x5A).all())
        if scales:
            got = scales["recv_scale"]
            assert torch.equal(got[:N], scales["x_scale"][src[:N] // k]) and bool((got[N:] == -1.0).all())
    finally:
        ctx.destroy()


# who reads the receive rows: combine, of 12 to 28 MiB; a stand-in, of 12 to 16, fp8 4 to 8 (both limits and the next size);
# and calls that do not, or not directly behind the dispatch
@gpu
@pytest.mark.parametrize("T,H,dtype,reader,want", [
    (384, 2048, "bf16", "combine", True), (383, 2048, "bf16", "combine", False), (896, 2048, "bf16", "combine", True),
    (897, 2048, "bf16", "combine", False), (256, 7168, "bf16", "combine", True), (500, 2888, "bf16", "combine", True),
    (600, 3080, "bf16", "combine", False), (192, 2048, "f32", "combine", True),
    (384, 2048, "bf16", "stand-in", True), (383, 2048, "bf16", "stand-in", False), (512, 2048, "bf16", "stand-in", True),
    (513, 2048, "bf16", "stand-in", False), (256, 2048, "fp8", "stand-in", True), (255, 2048, "fp8", "stand-in", False),
    (512, 2048, "fp8", "stand-in", True), (513, 2048, "fp8", "stand-in", False),
    (256, 7168, "bf16", "nobody", False), (256, 2048, "fp8", "nobody", False), (256, 7168, "bf16", "other rows", False),
    (256, 7168, "bf16", "after a kernel", False), (256, 7168, "bf16", "after the signals", True),
    (256, 7168, "bf16", "after a dispatch", False)])
def test_dispatch_with_its_layout(oracle, T, H, dtype, reader, want):
    k = 8
    step = Step(T, k, H, 1, 24, 20, dtype)
    ctx, st = step.ctx, step.stream
    y_type = torch.float32 if dtype == "f32" else torch.bfloat16
    rows = step.recv if dtype == "fp8" else step.recv.view(y_type)
    y, w = torch.zeros((T * k, H), device="cuda", dtype=y_type), torch.rand((T, k), device="cuda")
    out, scale = torch.zeros((T, H), device="cuda", dtype=torch.bfloat16), torch.ones(20, device="cuda")
    torch.cuda.synchronize()
    graph, fused = None, {}

    def read():
        if reader == "nobody":
            return
        if reader == "stand-in":
            ctx.expert_stub("dequant" if dtype == "fp8" else "scale", rows, y, T,
                            recv_scale=step.scales.get("recv_scale"), expert_scale=scale, stream=st)
        elif reader == "after a kernel":
            with torch.cuda.stream(st):
                w.mul_(1.0)
        elif reader == "after the signals":
            ctx.signal_experts_done(st)
        elif reader == "after a dispatch":
            step.dispatch()
        ctx.combine(y if reader in ("stand-in", "other rows") else rows, w, out, T, st)

    try:
        if reader == "after the signals":
            ctx.set_detection(1_000_000_000)
        graph, n = step.capture(step.layout, step.dispatch, lambda: fused.update(node=last_node(st)), read,
                                lambda: fused.update(flags=kernel_of(fused["node"]).word(8)))
        assert n == {"nobody": 1, "stand-in": 3, "after a kernel": 3, "after the signals": 3, "after a dispatch": 3}.get(reader, 2)
        assert fused["flags"] >> 31 == want
        for _ in range(2):
            step.renew()
            graph.launch(st)
            step.check(oracle)
    finally:
        if graph is not None:
            graph.destroy()
        ctx.destroy()


@gpu
@pytest.mark.parametrize("T,H", [(96, 7680), (112, 7176), (300, 3584), (512, 2048), (1400, 1504), (520, 4032), (524, 4032)])
def test_expansion(T, H):
    k = 8
    ctx, src, N = context(T, k, H, R=2, x_dtype="bf16", y_dtype="bf16")
    try:
        x = random_rows(T, H, "bf16")
        recv_d, recv = torch.zeros((T * k, 2 * H), dtype=torch.uint8, device="cuda"), torch.full(
            (T * k, 2 * H), 0x5A, dtype=torch.uint8, device="cuda")
        ctx.dedup_layout(T)
        ctx.dispatch_dedup(x, recv_d, T)
        w, out = torch.rand((T, k), device="cuda"), torch.zeros((T, H), dtype=torch.bfloat16, device="cuda")

        def run(st, combined):
            ctx.expand(recv_d, recv, T, stream=st)
            if combined:
                ctx.combine(recv.view(torch.bfloat16), w, out, T, st)

        for captured, combined in ((False, False), (True, False), (True, True)):
            recv.fill_(0x5A)
            launch(ctx, captured, lambda st: run(st, combined))
            assert torch.equal(recv[:N], x[src[:N] // k]) and bool((recv[N:] == 0x5A).all())
    finally:
        ctx.destroy()


@gpu
@pytest.mark.parametrize("T,H", [(127, 7168), (128, 7168), (1024, 1024), (1100, 1024), (219, 7168), (220, 7168)])
def test_quantisation(oracle, T, H):
    k = 8
    ctx, src, N = context(T, k, H, x_dtype="fp8", y_dtype="bf16")
    try:
        x = (torch.randn((T, H), device="cuda") * torch.exp(3 * torch.randn((T, 1), device="cuda"))).to(torch.bfloat16)
        x[3, 5] = 3e38
        x[3, :128] *= 1e-38                            # a scale that no product may stand in for the quotient of
        x[5, 200] = float("inf")
        recv = torch.full((T * k, H), 0x5A, dtype=torch.uint8, device="cuda")
        scale = torch.full((T * k, H // 128), -1.0, device="cuda")
        ctx.dispatch_quant(x, recv, scale, T)
        q, sc = oracle.quantize_e4m3(x.view(torch.int16).cpu().numpy().view(np.uint16))
        token = (src[:N] // k).cpu().numpy()
        assert np.array_equal(recv[:N].cpu().numpy(), q[token]) and bool((recv[N:] == 0x5A).all())
        assert np.array_equal(scale[:N].cpu().numpy().view(np.uint32), sc[token].view(np.uint32))
    finally:
        ctx.destroy()


@gpu
@pytest.mark.parametrize("T,H,dtype", [(80, 8184, "bf16"), (81, 8192, "bf16"), (256, 2048, "f32"), (700, 3080, "bf16"),
                                       (576, 4096, "bf16"), (580, 4096, "bf16"),
                                       (128, 8192, "bf16"), (130, 8192, "bf16"), (416, 4096, "bf16"), (418, 4096, "bf16")])
def test_scaling_stand_in(T, H, dtype):
    k, E = 8, 20
    ctx, src, N = context(T, k, H, x_dtype=dtype, y_dtype=dtype, out_dtype=dtype)
    try:
        tdt = {"f32": torch.float32, "bf16": torch.bfloat16}[dtype]
        recv = torch.randn((T * k, H), device="cuda").to(tdt)
        y = torch.empty((T * k, H), device="cuda", dtype=tdt)
        s = torch.rand(E, device="cuda") + 0.5
        p2l = torch.from_numpy(ctx.read("phys_to_logical", 24)).cuda().long()
        slot = torch.from_numpy(ctx.read("slot_of", T * k)).cuda().long()
        want = (recv[:N].float() * s[p2l[slot[src[:N]]]][:, None]).to(tdt)
        for captured in (False, True):
            y.fill_(7.0)
            launch(ctx, captured, lambda st: ctx.expert_stub("scale", recv, y, T, expert_scale=s, stream=st))
            assert torch.equal(y[:N], want) and bool((y[N:] == 7.0).all())
    finally:
        ctx.destroy()


@gpu
@pytest.mark.parametrize("call,T,want", [("stand-in", 256, True), ("expansion", 256, True), ("expansion", 191, False),
                                         ("expansion", 192, True), ("expansion", 512, True), ("expansion", 513, False),
                                         ("expansion, other rows", 256, False), ("expansion, after a kernel", 256, False)])
def test_held_only_in_a_captured_step(call, T, want):
    """Call by call the next buffers may be other ones, and held stores lose there; an expansion's do so too where another
    kernel reads its rows."""
    k, H = 8, 4096                                     # 16 MiB of receive rows for 256 tokens
    ctx, _, _ = context(T, k, H)
    try:
        recv, y = (torch.zeros((T * k, H), device="cuda", dtype=torch.bfloat16) for _ in range(2))
        scale, w = torch.ones(20, device="cuda"), torch.rand((T, k), device="cuda")
        out = torch.zeros((T, H), device="cuda", dtype=torch.bfloat16)
        ctx.dedup_layout(T)

        def run(st):
            if call == "stand-in":
                ctx.expert_stub("scale", recv, y, T, expert_scale=scale, stream=st)
                return
            ctx.expand(recv, y, T, stream=st)
            if call.endswith("kernel"):
                with torch.cuda.stream(st):
                    scale.mul_(1.0)
            ctx.combine(recv if call.endswith("rows") else y, w, out, T, st)

        launch(ctx, True, run)
        for captured in (False, True):
            with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as prof:
                launch(ctx, captured, run)
                torch.cuda.synchronize()
            names = [e.key for e in prof.key_averages() if "k_stub_scale" in e.key or "k_expand" in e.key]
            assert len(names) == 1 and re.search(r"(true|false)>\(", names[0])[1] == str(captured and want).lower(), names
    finally:
        ctx.destroy()


def test_held_stores_make_their_scalar_address(tmp_path):
    """As the write-through ones (test_scalar_addresses.py): the address of a store from scalar registers is added up
    by the two scalar instructions right ahead of it."""
    src, out = tmp_path / "store.hip", tmp_path / "store.s"
    src.write_text('#include "rows.hpp"\n'
                   "__global__ void k(char* p, const eep::u32x4* v, const int* rows) {\n"
                   "  for (int j = 0; j < 4; ++j)\n"
                   "    eep::store_row_at<true>(p, (int64_t)rows[j] * 7168, threadIdx.x * 16, v[threadIdx.x]);\n}\n")
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([build.HIPCC, *flags, "-w", "-I", build.HERE + "/csrc", "-S", "--cuda-device-only", "-o", str(out),
                    str(src)], check=True)
    lines = [s for s in (line.split(";")[0].strip() for line in out.read_text().splitlines()) if s]
    stores = 0
    for i, line in enumerate(lines):
        m = re.match(r"global_store_dwordx4 v\d+, v\[\d+:\d+\], s\[(98):(99)\] nt$", line)
        if m:
            stores += 1
            low, high = lines[i - 2], lines[i - 1]
            assert low.startswith(f"s_add_u32 s{m[1]},") and high.startswith(f"s_addc_u32 s{m[2]},"), lines[i - 4:i + 1]
    assert stores > 0
