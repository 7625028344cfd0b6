"""Layout and dispatch as one node of a captured graph: which captures become one, every form of the kernels against the
oracle's layout and a gather of the rows, several replays with tables and inputs that change between them, and replays
after the instance has got a second context whose membership changes meanwhile."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2605_10670_amd import binding

import gpu_util as gu
from test_gpu_layout_edges import instance

pytestmark = pytest.mark.gpu


def hip():
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    return ctypes.CDLL(path)


def nodes_captured(stream):
    """Nodes that the running capture of `stream` holds so far."""
    lib, status, graph = hip(), ctypes.c_int(), ctypes.c_void_p()
    assert lib.hipStreamGetCaptureInfo_v2(ctypes.c_void_p(stream.cuda_stream), ctypes.byref(status), None,
                                          ctypes.byref(graph), None, None) == 0
    n = ctypes.c_size_t()
    assert lib.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
    return n.value


class Step:
    """A context with its tables, and the buffers of one step."""

    def __init__(self, T, k, H, R, S, E, dtype="bf16", policy=binding.SPREAD, seed=0, **kw):
        self.T, self.k, self.H, self.R, self.S, self.E, self.policy = T, k, H, R, S, E, policy
        self.p2l, self.active, self.idx = instance(T, k, R, S, E, seed=seed + T + k + H)
        self.size = {"f32": 4, "bf16": 2, "fp8": 1}[dtype]
        self.shape = dict(num_ranks=R, slots_per_rank=S, primary_slots=max(1, S - 1), num_logical=E, max_tokens=T, topk=k,
                          hidden=H, x_dtype=dtype, y_dtype="f32" if dtype == "f32" else "bf16", policy=policy,
                          strict_coverage=False)
        self.ctx = binding.Context(**self.shape, **kw)
        self.stream = torch.cuda.Stream()
        self.idx_dev = gu.to_dev(self.idx)
        self.x = torch.randint(0, 256, (T, H * self.size), dtype=torch.uint8, device="cuda")
        self.recv = torch.full((T * k, H * self.size), 0x5A, dtype=torch.uint8, device="cuda")
        self.scales = {}
        if dtype == "fp8":
            self.scales = dict(x_scale=torch.rand((T, H // 128), device="cuda"),
                               recv_scale=torch.full((T * k, H // 128), -1.0, device="cuda"))
        torch.cuda.synchronize()
        self.tables(self.p2l, self.active)
        self.layout()                                  # (the library is loaded before the first capture)
        self.dispatch()
        self.stream.synchronize()

    def tables(self, p2l, active):
        self.p2l, self.active = p2l, active
        self.ctx.update_placement(p2l, self.stream)
        self.ctx.set_membership(active, self.stream)
        self.stream.synchronize()

    def layout(self, stream=None):
        self.ctx.dispatch_layout(self.idx_dev, self.T, stream or self.stream)

    def dispatch(self, stream=None):
        self.ctx.dispatch(self.x, self.recv, self.T, stream=stream or self.stream, **self.scales)

    def capture(self, *calls):
        """Captures the calls -> (graph, nodes)."""
        self.ctx.graph_begin(self.stream)
        for call in calls or (self.layout, self.dispatch):
            call()
        n = nodes_captured(self.stream)
        return self.ctx.graph_end(self.stream), n

    def renew(self):
        torch.cuda.synchronize()
        self.x.random_(0, 256)
        self.recv.fill_(0x5A)
        if self.scales:
            self.scales["x_scale"].uniform_()
            self.scales["recv_scale"].fill_(-1.0)
        torch.cuda.synchronize()

    def check(self, oracle, active=None):
        self.stream.synchronize()
        want = oracle.step_layout(self.idx, self.p2l, self.active if active is None else active, self.E, self.R, self.S,
                                  max(1, self.S - 1), self.policy)
        gu.assert_layout_equal(self.ctx.read_layout(self.T), want, self.T, self.k)
        self.check_rows()

    def check_rows(self):
        assert self.ctx.check_layout(self.T).tolist() == [0, 0, 0, 0]
        N = int(self.ctx.read("status", 4)[0])
        token = torch.from_numpy(self.ctx.read("src_of", self.T * self.k)[:N] // self.k).cuda().long()
        assert torch.equal(self.recv[:N], self.x[token]) and bool((self.recv[N:] == 0x5A).all())
        if self.scales:
            got = self.scales["recv_scale"]
            assert torch.equal(got[:N], self.scales["x_scale"][token]) and bool((got[N:] == -1.0).all())


# (T, k, H, R, S, E, x dtype), nodes expected: 1 = together
CASES = ([((40, k, 1032, 4, 6, 20, "bf16"), 1) for k in range(1, 11)] +                  # every compile-time top-k
         [((T, 8, 1024, 1, 24, 20, "bf16"), 1) for T in (1, 31, 127, 128, 129, 511, 512, 1023, 1024, 1025, 2047, 2048)] +
         [((T, 4, 7168, 2, 12, 20, "bf16"), 1) for T in (2, 254, 256, 258, 512, 768)] +  # few pairs, many pieces, rounds
         [((32, 8, 24, 32, 9, 256, "bf16"), 1), ((64, 8, 520, 64, 9, 512, "bf16"), 1), ((600, 6, 2880, 24, 5, 96, "bf16"), 1),
          ((1152, 2, 4608, 48, 2, 48, "bf16"), 1), ((400, 4, 2560, 8, 100, 700, "bf16"), 1), ((96, 8, 1024, 2, 500, 900, "f32"), 1),
          ((1300, 1, 3584, 4, 8, 30, "bf16"), 1), ((2048, 7, 1536, 16, 3, 40, "bf16"), 1), ((1280, 10, 640, 5, 8, 30, "f32"), 1),
          ((160, 8, 7168, 32, 9, 256, "fp8"), 1), ((32, 4, 512, 8, 3, 20, "fp8"), 1), ((700, 3, 1536, 4, 9, 30, "fp8"), 1),
          ((1023, 8, 1024, 1, 24, 20, "fp8"), 1), ((184, 2, 8192, 8, 3, 20, "f32"), 1),
          ((63, 8, 1024, 1, 24, 20, "bf16"), 1), ((64, 8, 7168, 2, 12, 20, "bf16"), 1),      # a pair to each of 512 threads or 1024
          ((65, 8, 7168, 1, 24, 20, "bf16"), 1), ((128, 4, 8192, 2, 12, 20, "f32"), 1), ((128, 4, 1024, 4, 128, 500, "bf16"), 1),
          ((128, 4, 1024, 4, 129, 500, "bf16"), 1), ((128, 4, 1024, 4, 128, 513, "bf16"), 1),
          # rounds of workgroups that fit a CU together, and not: pairs, top-10's registers, threads for many slots
          ((1536, 4, 1088, 32, 9, 256, "bf16"), 1), ((1568, 4, 1088, 32, 9, 256, "bf16"), 2), ((512, 10, 3584, 8, 9, 64, "bf16"), 1),
          ((608, 10, 3080, 8, 9, 64, "bf16"), 2), ((640, 4, 2560, 64, 9, 512, "bf16"), 1), ((1344, 4, 1088, 64, 9, 512, "bf16"), 1),
          ((1408, 4, 1088, 64, 9, 512, "bf16"), 2), ((640, 10, 1088, 64, 9, 512, "bf16"), 1), ((704, 10, 1088, 64, 9, 512, "bf16"), 2),
          # in two or more: tokens, pairs, top-k, ranks, pieces, scale rows
          ((2050, 7, 64, 2, 12, 20, "bf16"), 2), ((2048, 9, 64, 2, 12, 20, "bf16"), 3), ((64, 11, 64, 2, 12, 20, "bf16"), 2),
          ((130, 8, 64, 65, 2, 80, "bf16"), 2), ((440, 8, 8192, 2, 12, 20, "f32"), 2), ((1024, 8, 512, 2, 12, 20, "fp8"), 3),
          ((16, 2, 33280, 2, 12, 20, "fp8"), 2)])


@pytest.mark.parametrize("shape,nodes", CASES, ids=str)
def test_layout_and_dispatch(oracle, shape, nodes):
    step = Step(*shape)
    graph = None
    try:
        graph, n = step.capture()
        assert n == nodes
        for replay in range(3):
            step.renew()
            if replay == 1:                            # a rank fails, an expert loses its replicas
                active, p2l = step.active.copy(), step.p2l.copy()
                active[-1] = 1 - active[-1]
                p2l[p2l == 3] = 4
                step.tables(p2l, active)
            graph.launch(step.stream)
            step.check(oracle)
        step.renew()
        step.layout()                                  # and eagerly, with the same result
        step.dispatch()
        step.check(oracle)
    finally:
        if graph is not None:
            graph.destroy()
        step.ctx.destroy()


# pieces of 1 and 2 KiB, and whole rows in passes of four and seven vectors
@pytest.mark.parametrize("T,k,H", [(256, 8, 7168), (1028, 8, 1024), (1536, 2, 2048), (640, 8, 5120), (600, 3, 5768),
                                   (1600, 2, 2048), (1024, 6, 3096), (1100, 5, 7168), (1300, 1, 3584)])
def test_combine_behind_one_node(T, k, H):
    """A step whose layout and dispatch are one node: the sums of the receive rows, and of other rows of the same size, as
    the calls one by one give them."""
    step = Step(T, k, H, 4, 6, 20)
    graph = None
    try:
        w = torch.rand((T, k), device="cuda")
        y = torch.randn((T * k, H), device="cuda").to(torch.bfloat16)
        out = [torch.zeros((T, H), dtype=torch.bfloat16, device="cuda") for _ in range(2)]

        def combine():
            step.ctx.combine(step.recv.view(torch.bfloat16), w, out[0], T, step.stream)
            step.ctx.combine(y, w, out[1], T, step.stream)

        def renew():
            step.renew()
            step.x.copy_(torch.randn((T, H), device="cuda").to(torch.bfloat16).view(torch.uint8))
            torch.cuda.synchronize()

        graph, n = step.capture(step.layout, step.dispatch, combine)
        assert n == 3
        for _ in range(2):
            renew()
            graph.launch(step.stream)
            step.stream.synchronize()
            got = [o.clone() for o in out]
            for o in out:
                o.zero_()
            step.recv.fill_(0x5A)
            torch.cuda.synchronize()
            for call in (step.layout, step.dispatch, combine):
                call()
            step.stream.synchronize()
            assert all(torch.equal(a, b) and bool(a.any()) for a, b in zip(got, out))
    finally:
        if graph is not None:
            graph.destroy()
        step.ctx.destroy()


class KernelNodeParams(ctypes.Structure):
    _fields_ = [("block", ctypes.c_uint32 * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                ("grid", ctypes.c_uint32 * 3), ("args", ctypes.POINTER(ctypes.POINTER(ctypes.c_uint32))),
                ("lds", ctypes.c_uint32)]

    def word(self, i):
        """Argument i, a 32-bit word."""
        return self.args[i][0]


def last_node(stream):
    """The node that the running capture of `stream` holds last."""
    lib, status, node, n = hip(), ctypes.c_int(), ctypes.POINTER(ctypes.c_void_p)(), ctypes.c_size_t()
    assert lib.hipStreamGetCaptureInfo_v2(ctypes.c_void_p(stream.cuda_stream), ctypes.byref(status), None, None,
                                          ctypes.byref(node), ctypes.byref(n)) == 0 and n.value == 1
    return node[0]


def kernel_of(node):
    params = KernelNodeParams()
    assert hip().hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(params)) == 0
    return params


def last_kernel(stream):
    """The kernel that the running capture of `stream` holds last."""
    return kernel_of(last_node(stream))


def test_combine_takes_the_rows_as_the_last_dispatch_cut_them():
    """A dispatch in one node with its layout may cut the rows in another way than one of its own does, and combine
    goes by the last one that wrote them."""
    T, k, H = 1028, 8, 1024                            # pieces of 1 KiB in the one, whole rows in the other
    step = Step(T, k, H, 4, 6, 20)
    w, out = torch.rand((T, k), device="cuda"), torch.zeros((T, H), dtype=torch.bfloat16, device="cuda")
    recv_d = torch.zeros_like(step.recv)
    dedup = lambda: step.ctx.dedup_layout(T, step.stream)
    packed = lambda: step.ctx.dispatch_dedup(step.x, recv_d, T, step.stream)
    expand = lambda: step.ctx.expand(recv_d, step.recv, T, step.stream)
    grids = []

    def combine():
        step.ctx.combine(step.recv.view(torch.bfloat16), w, out, T, step.stream)
        grids.append(last_kernel(step.stream).grid[0])

    try:
        for calls in ((step.layout, step.dispatch), (step.layout, step.dispatch, step.dispatch),
                      (step.layout, step.dispatch, dedup, packed, expand), (step.layout, step.dispatch, dedup, packed)):
            step.capture(*calls, combine)[0].destroy()
        step.layout()
        step.capture(step.dispatch, combine)[0].destroy()
        assert grids == [T * 2, T // 8 * 16 + 16, T // 8 * 16 + 16, T * 2, T // 8 * 16 + 16]
    finally:
        step.ctx.destroy()


@pytest.mark.parametrize("router", ["repeats", "padding", "copies", "outside", "first live"])
@pytest.mark.parametrize("T,k", [(96, 8), (640, 8), (320, 3), (64, 4)])
def test_routers(oracle, router, T, k):
    step = Step(T, k, 1024, 4, 9, 30, policy=binding.FIRST_LIVE if router == "first live" else binding.SPREAD)
    graph = None
    try:
        idx = step.idx
        if router == "repeats":
            idx[::3, k - 1] = idx[::3, 0]
        elif router == "padding":
            idx[T // 3:] = -1
        elif router == "copies":
            idx[:] = idx[0]
        elif router == "outside":
            idx[::2, 0], idx[1::5, 1] = 30, 2**31 - 1
        graph, n = step.capture()
        assert n == 1
        step.idx_dev.copy_(gu.to_dev(idx))
        for _ in range(2):
            step.renew()
            graph.launch(step.stream)
            step.check(oracle)
    finally:
        if graph is not None:
            graph.destroy()
        step.ctx.destroy()


def test_what_becomes_one_node(oracle):
    """One node only where the dispatch is captured right behind its layout, on its stream, with nothing else waiting
    for the layout, and no buffer that the two could share."""
    step = Step(64, 8, 1024, 4, 9, 30)
    other, side = Step(64, 8, 1024, 4, 9, 30, seed=1), torch.cuda.Stream()
    graphs = []

    def captured(*calls):
        graph, n = step.capture(*calls)
        graphs.append(graph)
        step.renew()
        graph.launch(step.stream)
        return n

    def on_side(call):                                 # forked behind what was captured so far, and joined
        def run():
            side.wait_stream(step.stream)
            call(side)
            step.stream.wait_stream(side)
        return run

    try:
        assert captured() == 1
        step.check(oracle)
        assert captured(step.layout, step.dispatch, step.dispatch) == 2
        step.check(oracle)
        assert captured(step.layout, lambda: step.ctx.set_membership(step.active, step.stream), step.dispatch) == 3
        step.check(oracle)
        assert captured(step.layout, on_side(step.dispatch)) == 2                  # on another stream
        step.check(oracle)
        assert captured(step.layout, lambda: other.layout(step.stream), step.dispatch) == 3
        step.check(oracle)

        def follower():                                # something else waits for the layout
            side.wait_stream(step.stream)
            other.layout(side)
            step.dispatch()
            step.stream.wait_stream(side)
        assert captured(step.layout, follower) == 3
        step.check(oracle)
        assert captured(step.layout, step.dispatch, step.layout, step.dispatch) == 2
        step.check(oracle)
        # the router indices lie in the receive buffer (the layout is done with them when rows are written)
        hidden = step.recv.view(torch.int32).reshape(-1)[:step.T * step.k].view(step.T, step.k)
        mine = step.idx_dev
        step.idx_dev = hidden
        graph, n = step.capture()
        graphs.append(graph)
        assert n == 2
        step.renew()
        hidden.copy_(mine)
        torch.cuda.synchronize()
        graph.launch(step.stream)
        step.stream.synchronize()
        N = int(step.ctx.read("status", 4)[0])
        token = torch.from_numpy(step.ctx.read("src_of", step.T * step.k)[:N] // step.k).cuda().long()
        assert torch.equal(step.recv[:N], step.x[token])
    finally:
        for graph in graphs:
            graph.destroy()
        other.ctx.destroy()
        step.ctx.destroy()


@pytest.mark.parametrize("mode", ["global", "thread_local", "relaxed"])
def test_captured_by_torch(oracle, mode):
    """torch's own capture, in each of its modes, with its kernels around the two calls."""
    step = Step(96, 8, 1024, 4, 9, 30)
    try:
        pairs = torch.zeros_like(step.idx_dev)
        seen = torch.zeros_like(step.recv[:1])
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=step.stream, capture_error_mode=mode):
            mine, step.idx_dev = step.idx_dev, pairs
            pairs.copy_(mine)
            step.layout()
            step.dispatch()
            n = nodes_captured(step.stream)
            seen.copy_(step.recv[:1])
        assert n == 2
        for _ in range(3):
            step.renew()
            pairs.zero_()
            torch.cuda.synchronize()
            with torch.cuda.stream(step.stream):
                graph.replay()
            step.check(oracle)
            assert torch.equal(seen, step.recv[:1])
        del graph
    finally:
        step.ctx.destroy()


def test_wrong_calls_are_refused_while_captured():
    """As eagerly, and the capture goes on."""
    step = Step(64, 8, 1024, 4, 9, 30)
    try:
        step.ctx.graph_begin(step.stream)
        step.layout()
        for args in ((step.x, step.recv, 32), (step.x.view(-1)[1:], step.recv, 64)):
            with pytest.raises(binding.EepError):
                step.ctx.dispatch(*args, stream=step.stream)
        step.dispatch()
        step.ctx.graph_end(step.stream).destroy()
    finally:
        step.ctx.destroy()


@pytest.mark.parametrize("T,k,R,S,E", [(64, 8, 32, 9, 256), (128, 4, 4, 9, 30), (512, 8, 32, 9, 256), (1536, 8, 2, 12, 20),
                                       (480, 5, 48, 4, 96), (64, 10, 64, 9, 512)])
def test_one_mask_for_all_workgroups(oracle, T, k, R, S, E):
    """Captured while the instance had one context, and with two, and replayed when it has two and the mask changes
    meanwhile: a layout of either mask, and the rows that belong to it."""
    step, other, graphs = Step(T, k, 512, R, S, E), None, []
    updates = torch.cuda.Stream()
    try:
        for i in range(2):
            graph, n = step.capture()
            graphs.append(graph)
            assert n == 1
            if i == 0:
                other = binding.Context(**step.shape, parent=step.ctx)
        mask = step.active.copy()
        for i in range(12):
            before, mask = mask, mask.copy()
            mask[(i * 7) % R] ^= 1
            step.renew()
            graphs[i % 2].launch(step.stream)
            other.set_membership(mask, updates)
            torch.cuda.synchronize()
            step.check_rows()
            got = step.ctx.read_layout(T)
            want = [oracle.step_layout(step.idx, step.p2l, m, E, R, S, max(1, S - 1), binding.SPREAD) for m in (before, mask)]
            assert any(all(np.array_equal(got[key], w[key]) for key in gu.LAYOUT_KEYS) for w in want), i
            step.renew()
            graphs[i // 2 % 2].launch(step.stream)     # the mask is still now
            step.check(oracle, mask)
        other.destroy()
        other = None
        step.renew()
        graphs[1].launch(step.stream)                  # and with one context again
        step.check(oracle, mask)
    finally:
        for graph in graphs:
            graph.destroy()
        if other is not None:
            other.destroy()
        step.ctx.destroy()
