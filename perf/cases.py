"""The calls that a program makes of this library, as timed cases.

A case is one pass through the public entry points of `paper_2605_10670_amd.binding`:

  kind "step"    dispatch_layout, dispatch, [expert_stub], combine
  kind "quant"   dispatch_layout, dispatch_quant, expert_stub (dequantise), combine
  kind "dedup"   dispatch_layout, dedup_layout, dispatch_dedup, expand, combine
  kind "churn"   a rank fails and rejoins: both table updates, then graph replays, twice
  kind "repair"  a rank fails and rejoins with its weights: the planners, both weight
                 movements, both membership updates

`steps` > 0: that many steps (the MoE layers of one forward pass, each with its own
router choices, token rows and outputs, one receive buffer for all) are captured once
and a pass replays the graph, as serving does; 0: the calls are made one by one.

Every result has one correct value: layouts and moved rows are copies, the stand-ins
round one product, and the combine's order and rounding are part of its contract (fp32,
one fused multiply-add per routed pair, ascending).  So the tolerance is "exact".
"""
import math

import numpy as np
import torch

from paper_2605_10670_amd import binding, synth

TORCH_OF = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.uint8}
BYTES_OF = {"f32": 4, "bf16": 2, "fp8": 1}
GROUP = 128                 # channels per fp8 scale
DETECT_NS = 1_000_000_000   # the paper's time-out of one second

DEFAULTS = dict(kind="step", steps=0, tokens=4096, hidden=7168, experts=256, topk=8, ranks=32,
                primary=8, redundant=1, x="bf16", y="bf16", out="bf16", stub="identity", failed=0,
                repaired=True, zipf=False, first_live=False, detect=False)


def _case(name, **kw):
    return dict(DEFAULTS, name=name, **kw)


def listed():
    return [
        # the smallest whole step, one call after the other: 128 fp32 tokens, top-2 of 16
        # experts, 4 ranks, one of them failed and its experts remapped
        _case("tiny-f32-top2", tokens=128, hidden=1024, experts=16, topk=2, ranks=4, primary=4,
              redundant=2, x="f32", y="f32", out="f32", stub="scale", failed=1),
        # decode at the lowest concurrency: one token per rank, captured forward pass
        _case("decode-32", steps=8, tokens=32),
        # decode at the concurrency of the paper's serving runs, eight tokens per rank
        _case("decode-256", steps=8, tokens=256),
        # decode at full batch, the benchmark's shape: 128 tokens per rank
        _case("decode-4096", steps=4),
        # full-batch decode after a failure: hot experts live only in redundant slots
        _case("decode-4096-zipf", failed=1, zipf=True),
        # decode between a failure and its repair: failure detection on, the dead rank's
        # experts are not placed anywhere yet, so some pairs of many tokens are dropped
        _case("decode-1024-degraded", tokens=1024, failed=1, repaired=False, detect=True),
        # a ragged prefill batch of a smaller model: top-6, rows that are no whole number of
        # wavefronts, token count that is no power of two, fp32 results, 24 ranks
        _case("prefill-5976-top6", tokens=5976, hidden=2880, experts=96, topk=6, ranks=24,
              primary=4, redundant=1, out="f32", stub="scale"),
        # prefill with fp8 rows and their scales, two ranks failed and remapped
        _case("prefill-16384-fp8", tokens=16384, x="fp8", stub="dequant", failed=2),
        # full-batch decode with the quantisation fused into dispatch
        _case("decode-4096-quant", kind="quant", x="fp8", stub="dequant"),
        # few ranks with many experts each: a row crosses once per rank and is expanded there
        _case("decode-2048-dedup", kind="dedup", tokens=2048, ranks=8, primary=32, redundant=4),
        # membership churn under captured graphs, 4 steps per phase, per-expert scalar experts
        _case("churn-2048", kind="churn", steps=4, tokens=2048, hidden=4096, experts=128, ranks=16,
              stub="scale", failed=1),
        # failure and rejoin with weights: 4.7 MB per expert, backup in pinned host memory
        _case("repair-64", kind="repair", tokens=16, hidden=2048, experts=64, ranks=8, primary=8,
              redundant=2, failed=1),
    ]


# The largest pass that draw() may give, in bytes a pass cannot do without.
MOST_BYTES = 5.5e9


def draw(rng):
    while True:
        kind = rng.choices(["step", "quant", "dedup", "churn", "repair"], [70, 9, 9, 8, 4])[0]
        ranks = rng.choice([2, 4, 6, 8, 8, 12, 16, 16, 24, 32, 32, 48, 64])
        primary = rng.choice([1, 2, 3, 4, 4, 6, 8, 8, 12, 16])
        redundant = rng.choice([0, 1, 1, 2, 4])
        if not 4 <= ranks * primary <= 512:
            continue
        topk = min(rng.choice([1, 2, 3, 4, 6, 8, 8, 8, 8, 10]), ranks * primary)
        per_rank = max(1, round(math.exp(rng.uniform(0.0, math.log(600.0)))))
        tokens = ranks * per_rank
        wide = math.exp(rng.uniform(math.log(512.0), math.log(8192.0)))
        hidden = 512 * max(1, round(wide / 512)) if rng.random() < 0.6 else 32 * round(wide / 32)
        dtypes = rng.choices([("bf16", "bf16", "bf16"), ("bf16", "bf16", "f32"),
                              ("f32", "f32", "f32"), ("f32", "f32", "bf16"),
                              ("fp8", "bf16", "bf16"), ("fp8", "bf16", "f32")],
                             [50, 10, 10, 5, 20, 5])[0]
        c = dict(DEFAULTS, kind=kind, tokens=tokens, hidden=hidden, ranks=ranks, primary=primary,
                 redundant=redundant, experts=ranks * primary, topk=topk, x=dtypes[0], y=dtypes[1],
                 out=dtypes[2], zipf=rng.random() < 0.25, first_live=rng.random() < 0.1)
        if kind == "step":
            c["steps"] = rng.choice([0, 0, 2, 4, 8])
            c["detect"] = rng.random() < 0.15
            c["failed"] = rng.choice([0, 0, 1, 2])
            c["repaired"] = rng.random() < 0.8
            c["stub"] = "dequant" if c["x"] == "fp8" else rng.choice(["identity", "scale"])
        elif kind == "quant":
            c.update(x="fp8", y="bf16", stub="dequant", failed=rng.choice([0, 1]),
                     repaired=rng.random() < 0.8)
        elif kind == "dedup":
            if c["x"] == "fp8":
                c.update(x="bf16", y="bf16")
            c.update(failed=rng.choice([0, 1]), repaired=rng.random() < 0.8)
        else:
            if c["x"] == "fp8":
                c.update(x="bf16", y="bf16")
            c.update(failed=1, steps=rng.choice([1, 2, 4]) if kind == "churn" else 0,
                     stub="scale" if kind == "churn" else "identity")
            if kind == "repair":
                c["hidden"] = 256 * rng.randint(2, 12)
        if c["x"] == "fp8":                        # scale rows are whole 16-byte vectors
            c["hidden"] = 512 * max(1, round(hidden / 512))
        if c["failed"] >= ranks:
            continue
        if c["repaired"] and c["failed"] * primary > (ranks - c["failed"]) * redundant:
            continue                               # no room for the lost experts
        if kind == "repair" and (c["hidden"] ** 2 * c["experts"] > 3.2e8 or ranks < 3):
            continue                               # keeps the pinned backup small
        if work(c)["bytes"] > MOST_BYTES or per_rank * ranks > 16384:
            continue
        return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _tables(case):
    """(placement in force, mask, preferred placement, failed ranks)"""
    R, sp, sr = case["ranks"], case["primary"], case["redundant"]
    pref = synth.preferred_placement(R, sp, sr)
    failed = tuple((R // 2 + 1 + 5 * i) % R for i in range(case["failed"]))
    p2l = synth.repaired_placement(pref, failed, R, sp, sr) if failed and case["repaired"] else pref
    return p2l, synth.active_mask(R, failed), pref, failed


def _inputs(case, seed):
    """One list entry per step: router choices and weights, token rows (and scales)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    T, H, E, k = case["tokens"], case["hidden"], case["experts"], case["topk"]
    bias = torch.zeros(E, device="cuda")
    if case["zipf"]:        # a skewed router; the failed rank's experts are the hottest
        lost = [f * case["primary"] + i for f in _tables(case)[3] for i in range(case["primary"])]
        order = lost + [e for e in range(E) if e not in set(lost)]
        bias[torch.tensor(order, device="cuda")] = -1.2 * torch.log(
            torch.arange(1, E + 1, device="cuda").float())
    n = max(1, case["steps"]) * (2 if case["kind"] == "churn" else 1)
    sets = []
    for _ in range(n):
        logits = torch.randn((T, E), generator=g, device="cuda") + bias
        top, idx = torch.topk(logits, k, dim=1)
        x = torch.randn((T, H), generator=g, device="cuda")
        s = dict(idx=idx.to(torch.int32), w=torch.softmax(top.double(), 1).float())
        if case["kind"] == "quant":
            s["x"] = x.to(torch.bfloat16)
        elif case["x"] == "fp8":
            s["x"], s["scale"] = _quantise(x)
        else:
            s["x"] = x.to(TORCH_OF[case["x"]])
        sets.append(s)
    return sets


def _quantise(x):
    xg = x.float().view(x.shape[0], -1, GROUP)
    scale = xg.abs().amax(2) / 448.0
    scale[scale == 0] = 1.0
    codes = (xg / scale[:, :, None]).view(x.shape).to(torch.float8_e4m3fn).view(torch.uint8)
    return codes.contiguous(), scale


def _expert_scale(case):
    return (0.5 + torch.arange(case["experts"], device="cuda") / case["experts"]).float()


class State:
    """Context, buffers and graphs of one program."""

    def __init__(self):
        self.graphs = []
        self.ctx = None

    def __del__(self):
        if self.ctx is not None:
            torch.cuda.synchronize()
            for g in self.graphs:
                g.destroy()
            self.ctx.destroy()


def _context(case, st):
    """A context in caller-owned memory, so that its arrays can be returned as tensors."""
    shape = dict(num_ranks=case["ranks"], slots_per_rank=case["primary"] + case["redundant"],
                 primary_slots=case["primary"], num_logical=case["experts"],
                 max_tokens=case["tokens"], topk=case["topk"], hidden=case["hidden"],
                 x_dtype=case["x"], y_dtype=case["y"], out_dtype=case["out"],
                 policy=binding.FIRST_LIVE if case["first_live"] else binding.SPREAD,
                 strict_coverage=bool(case["repaired"]))
    ws = torch.zeros(binding.workspace_bytes(**shape), dtype=torch.uint8, device="cuda")
    st.ctx = ctx = binding.Context(workspace=ws, **shape)
    T, k, R, P = case["tokens"], case["topk"], case["ranks"], ctx.P
    ptr = ctx.view_pointers()
    sizes = dict(slot_of=T * k, row_of=T * k, src_of=T * k, count=P, offset=P + 1, rank_count=R,
                 rank_offset=R + 1, cnt_src=R * P)
    ints = ws.view(torch.int32)
    st.layout = {}
    for name, n in sizes.items():
        at = (ptr[name] - ws.data_ptr()) // 4
        st.layout[name] = ints[at:at + n]
    at = (ptr["status"] - ws.data_ptr()) // 4
    st.layout["status"] = ints[at:at + 3]   # the fourth word counts table updates


def prepare(case, seed):
    st = State()
    st.case, T, k, H = case, case["tokens"], case["topk"], case["hidden"]
    p2l, active, pref, failed = _tables(case)
    _context(case, st)
    st.tables = (p2l, active, pref, np.ones_like(active), failed)
    if case["kind"] == "repair":
        return _prepare_repair(case, seed, st)
    st.ctx.update_placement(pref if case["kind"] == "churn" else p2l)
    if case["kind"] != "churn":
        st.ctx.set_membership(active)
    st.sets = _inputs(case, seed)
    for s in st.sets:
        s["out"] = torch.zeros((T, H), dtype=TORCH_OF[case["out"]], device="cuda")
    st.recv = torch.zeros((T * k, H), dtype=TORCH_OF[case["x"]], device="cuda")
    st.recv_scale = (torch.zeros((T * k, H // GROUP), device="cuda") if case["x"] == "fp8" else None)
    st.y = (st.recv if case["stub"] == "identity" else
            torch.zeros((T * k, H), dtype=TORCH_OF[case["y"]], device="cuda"))
    st.expert_scale = _expert_scale(case) if case["stub"] == "scale" else None
    if case["kind"] == "dedup":
        st.recv_dedup = torch.zeros_like(st.recv)
    if case["detect"]:
        st.ctx.set_detection(DETECT_NS)
    if case["steps"]:
        _step(st, st.sets[0])       # every kernel is loaded before the first capture
        torch.cuda.synchronize()
        side = torch.cuda.Stream()
        per = case["steps"]
        for at in range(0, len(st.sets), per):
            st.ctx.graph_begin(side)
            for s in st.sets[at:at + per]:
                _step(st, s, side)
            st.graphs.append(st.ctx.graph_end(side))
    return st


def _slot_bytes(case):
    """Three one-byte matrices of hidden x 3/8 hidden."""
    return 3 * case["hidden"] * (3 * case["hidden"] // 8) // 16 * 16


def _prepare_repair(case, seed, st):
    E, P = case["experts"], st.ctx.P
    st.slot_bytes = _slot_bytes(case)
    g = torch.Generator(device="cuda").manual_seed(seed)
    store = torch.randint(-2**31, 2**31 - 1, (E, st.slot_bytes // 4), generator=g, device="cuda",
                          dtype=torch.int32).view(torch.uint8)
    st.backup = torch.empty((E, st.slot_bytes), dtype=torch.uint8, pin_memory=True)
    st.backup.copy_(store)
    pref = st.tables[2]
    st.weights = store[torch.from_numpy(np.maximum(pref, 0)).long().cuda()]
    st.ctx.update_placement(pref)
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _step(st, s, stream=None):
    ctx, case = st.ctx, st.case
    T, kind = case["tokens"], case["kind"]
    ctx.dispatch_layout(s["idx"], T, stream)
    if kind == "quant":
        ctx.dispatch_quant(s["x"], st.recv, st.recv_scale, T, stream)
    elif kind == "dedup":
        ctx.dedup_layout(T, stream)
        ctx.dispatch_dedup(s["x"], st.recv_dedup, T, stream)
        ctx.expand(st.recv_dedup, st.recv, T, stream)
    else:
        ctx.dispatch(s["x"], st.recv, T, s.get("scale"), st.recv_scale, stream)
    if case["stub"] != "identity":
        ctx.expert_stub(case["stub"], st.recv, st.y, T, st.recv_scale, st.expert_scale, stream)
    elif case["detect"]:
        ctx.signal_experts_done(stream)
    ctx.combine(st.y, s["w"], s["out"], T, stream)


def run(st):
    kind = st.case["kind"]
    if kind == "repair":
        return _run_repair(st)
    if kind == "churn":
        p2l, dead, pref, live, _ = st.tables
        st.ctx.update_placement(p2l)
        st.ctx.set_membership(dead)
        st.graphs[0].launch(None)
        st.ctx.set_membership(live)
        st.ctx.update_placement(pref)
        st.graphs[1].launch(None)
    elif st.graphs:
        st.graphs[0].launch(None)
    else:
        _step(st, st.sets[0])
    got = dict(st.layout, out=[s["out"] for s in st.sets], recv=st.recv)
    if st.recv_scale is not None:
        got["recv_scale"] = st.recv_scale
    if st.y is not st.recv:
        got["y"] = st.y
    if kind == "dedup":
        got["recv_dedup"] = st.recv_dedup
    return got


def _plans(case, pref, dead, live, failed):
    """Repair after the loss, the returning ranks' empty slots, their reload, the return."""
    R, sp, E = case["ranks"], case["primary"], case["experts"]
    S = sp + case["redundant"]
    plan = binding.plan_repair(pref, dead, R, S, sp, E)
    lost, target = plan["p2l"].copy(), plan["p2l"].copy()
    for f in failed:
        lost[f * S:(f + 1) * S] = -1
        target[f * S:(f + 1) * S] = pref[f * S:(f + 1) * S]
    back = binding.plan_transition(lost, target, dead, live, R, S, sp, E)
    return plan, lost, back, binding.plan_transition(target, pref, live, live, R, S, sp, E)


def _run_repair(st):
    ctx = st.ctx
    _, dead, pref, live, failed = st.tables
    plan, lost, back, resume = _plans(st.case, pref, dead, live, failed)
    # the rank is lost: cover its experts on the others, then take it out of the mask
    ctx.apply_repair(st.weights, st.backup, st.slot_bytes, plan)
    ctx.set_membership(dead)
    # it comes back empty: load its experts, let it join, return to the preferred placement
    ctx.update_placement(lost)
    ctx.apply_repair(st.weights, st.backup, st.slot_bytes, back)
    ctx.set_membership(live)
    ctx.apply_repair(st.weights, st.backup, st.slot_bytes, resume)
    return st.weights


# ---------------------------------------------------------------------------
# what a pass cannot do without, and its results in 64 bits
# ---------------------------------------------------------------------------
def _routed_share(case):
    """Share of the pairs that have a live replica."""
    p2l, active, _, _ = _tables(case)
    S = case["primary"] + case["redundant"]
    live = {int(e) for p, e in enumerate(p2l) if e >= 0 and active[p // S]}
    return len(live) / case["experts"]


def work(case):
    T, k, H = case["tokens"], case["topk"], case["hidden"]
    if case["kind"] == "repair":
        _, dead, pref, failed = _tables(case)
        plan, _, back, resume = _plans(case, pref, dead, np.ones_like(dead), failed)
        moves = sum(p["peer"] + p["dram"] for p in (plan, back, resume))
        return {"bytes": 2.0 * moves * _slot_bytes(case), "flops": 0}
    pairs = T * k * _routed_share(case)
    xb, yb, ob = (BYTES_OF[case[n]] for n in ("x", "y", "out"))
    sb = 4 / GROUP if case["x"] == "fp8" else 0
    b = T * H * ((2 if case["kind"] == "quant" else xb + sb) + ob) + pairs * H * (xb + sb + yb)
    if case["stub"] != "identity":
        b += pairs * H * (xb + sb + yb)            # the expert stage reads its rows and writes its own
    if case["kind"] == "dedup":                    # rows are written, read and written again
        R = case["ranks"]
        per_rank = 1 - (1 - 1 / R) ** k
        b += 2 * T * R * per_rank * H * xb
    b += T * k * 4 * 7                             # router choices, weights and the row tables
    flops = 2.0 * pairs * H
    n = max(1, case["steps"]) * (2 if case["kind"] == "churn" else 1)
    return {"bytes": float(n * b), "flops": float(n * flops)}


def tolerance(case):
    return "exact"


def _routes(case, idx, p2l, active):
    """Row of every pair (-1: dropped) from the rules: the first live replica or replica
    (t mod n) of the live ones, primary slots first; rows by slot, then by token."""
    S = case["primary"] + case["redundant"]
    T, k = idx.shape
    lists = [[] for _ in range(case["experts"])]
    order = sorted(range(len(p2l)), key=lambda p: (p % S >= case["primary"], p))
    for p in order:
        if p2l[p] >= 0 and active[p // S]:
            lists[p2l[p]].append(p)
    most = max(1, max(len(v) for v in lists))
    table = torch.tensor([v + [-1] * (most - len(v)) for v in lists], device=idx.device)
    n = torch.tensor([max(1, len(v)) for v in lists], device=idx.device)
    e = idx.long()
    t = torch.arange(T, device=idx.device)[:, None]
    pick = torch.zeros_like(e) if case["first_live"] else t % n[e]
    slot = table[e, pick].reshape(-1)
    key = torch.where(slot < 0, torch.full_like(slot, len(p2l)), slot)
    by_slot = torch.sort(key, stable=True).indices
    row = torch.empty_like(slot)
    row[by_slot] = torch.arange(T * k, device=idx.device)
    return torch.where(slot < 0, torch.full_like(slot, -1), row).view(T, k)


def exact(case, seed):
    if case["kind"] == "repair":
        return None
    T, k, H = case["tokens"], case["topk"], case["hidden"]
    p2l, active, pref, _ = _tables(case)
    sets = _inputs(case, seed)
    scale_of = _expert_scale(case).double()
    fp8 = case["x"] == "fp8"
    zeros = lambda n: torch.zeros((T * k, n), dtype=torch.float64, device="cuda")
    got = dict.fromkeys(("slot_of", "row_of", "src_of", "count", "offset", "rank_count",
                         "rank_offset", "cnt_src", "status", "recv", "recv_dedup"))
    got["out"] = []
    if fp8:
        got["recv_scale"] = zeros(H // GROUP)
    else:
        got["recv"] = zeros(H)
    if case["stub"] != "identity":
        got["y"] = zeros(H)
    for i, s in enumerate(sets):
        second = case["kind"] == "churn" and i >= case["steps"]
        row = _routes(case, s["idx"], pref if second else p2l,
                      np.ones_like(active) if second else active)
        routed = row >= 0
        codes, sc = (_quantise(s["x"]) if case["kind"] == "quant" else (s["x"], s.get("scale")))
        if fp8:
            x = (codes.view(torch.float8_e4m3fn).double().view(T, -1, GROUP)
                 * sc.double()[:, :, None]).view(T, H)
        else:
            x = s["x"].double()
        factor = (scale_of[s["idx"].long()] if case["stub"] == "scale" else
                  torch.ones((T, k), dtype=torch.float64, device="cuda"))
        got["out"].append((s["w"].double() * factor * routed).sum(1)[:, None] * x)
        # the receive rows are the last step's; where pairs are dropped, rows past its last
        # one still hold those of earlier steps
        if i + 1 < len(sets) and case["repaired"]:
            continue
        rows, token = row[routed], torch.nonzero(routed)[:, 0]
        if fp8:
            got["recv_scale"][rows] = sc.double()[token]
        else:
            got["recv"][rows] = x[token]
        if "y" in got:
            got["y"][rows] = x[token] * factor[routed][:, None]
    return got
