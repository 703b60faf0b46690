"""The work that a program using this library has it do on one GPU: whole
balancing steps of the paper's MoE layers, the planner, the row dispatch, the
combine gather, the gradient reduction and the relay packing, at the sizes of
the five workloads in gen/ and at ragged and small ones.

A case's "kind" says which entry points one pass calls:
  step      count, plan_replicate, reroute_and_pack, dispatch_layout and
            dispatch_scatter: one layer's forward balancing step
  route     count, plan, dispatch and combine: routing and its way back for a
            layer whose replicas are in place already
  plan      count and plan (both halves)
  dispatch  dispatch of a layer that is planned already
  combine   combine of the experts' output rows (forward; the same gather
            serves the backward of the dispatch)
  grad      grad_reduce of the replicas' fp32 gradients (backward)
  relay     relay_plan and pack_relay of a layer that is planned already

Sizes: R ranks, E experts, n_slot redundant slots per rank, top-k k, T tokens
of this rank, hidden size H, expert width F (a blob is 3 * H * F elements),
u_min.  Routing: logits N(0, 1) plus a bias per expert that the "layer"
number fixes (a trained router's preferences), "zipf" (-scale * log of a
random rank), "normal" (scale * N(0, 1)) or "burst" (8 hot experts at +scale);
"groups" / "top_groups" restrict a token to its best expert groups; "pad" is
the share of trailing tokens that are padding (ids -1).  The rank under test is
the one whose main experts draw the most tokens.  "blobs" and "copies" are the
weight blobs which that rank replicates, and the replicas of them, under the
plan of the listed routing (they vary little with the seed); they enter only
the bytes of work().
"""
import math

import torch

import paper_2606_04101_amd as uep

DEV = "cuda"
MAX_STAGING = 64  # staging entries a program holds at most


def _case(name, kind, R, E, n_slot, k, T, H, F, u_min, bias, scale, layer=0,
          groups=0, top_groups=0, pad=0.0, blobs=1, copies=1):
    return dict(name=name, kind=kind, R=R, E=E, n_slot=n_slot, k=k, T=T, H=H, F=F,
                u_min=u_min, bias=bias, scale=scale, layer=layer, groups=groups,
                top_groups=top_groups, pad=pad, blobs=blobs, copies=copies)


def listed():
    return [
        # the tiny workload's whole step: launches and latency are everything
        _case("tiny_step", "step", 4, 16, 2, 2, 512, 256, 512, 32, "normal", 1.5),
        # a serving microbatch of 128 tokens: routing there and back, weights in place
        _case("small_route", "route", 32, 128, 2, 8, 128, 4096, 1408, 32, "zipf", 0.35),
        # one layer's forward step, GLM-4.5-Air-shaped
        _case("glm45air_step", "step", 32, 128, 2, 8, 4096, 4096, 1408, 1024, "zipf", 0.352,
              layer=9, copies=2),
        # one layer's forward step in training, DeepSeek-V3-shaped (the headline workload)
        _case("dsv3_train_step", "step", 64, 256, 1, 8, 4096, 7168, 2048, 1024, "zipf", 0.348,
              layer=9, groups=8, top_groups=4, copies=2),
        # one layer's prefill step with hot-expert bursts, DeepSeek-V3-shaped: the largest
        _case("dsv3_prefill_step", "step", 32, 256, 2, 8, 16384, 7168, 2048, 1024, "burst", 3.0,
              groups=8, top_groups=4, copies=3),
        # load counting and both planner halves at the largest group, Qwen3-235B-shaped
        _case("qwen3_plan", "plan", 64, 128, 2, 8, 8192, 4096, 1536, 1024, "normal", 1.0,
              layer=8),
        # the dispatch alone, when the weights' distribution is overlapped elsewhere
        _case("qwen3_dispatch", "dispatch", 64, 128, 2, 8, 8192, 4096, 1536, 1024, "normal", 1.0,
              layer=8),
        # a ragged batch: odd token count, padding, top-6, rows of 2.8 K
        _case("ragged_dispatch", "dispatch", 12, 72, 3, 6, 2999, 2880, 1536, 64, "zipf", 0.5,
              pad=0.11),
        # expert outputs back to token order, DeepSeek-V3-shaped training layer
        _case("dsv3_combine", "combine", 64, 256, 1, 8, 4096, 7168, 2048, 1024, "zipf", 0.348,
              layer=9, groups=8, top_groups=4, copies=2),
        # the same with more experts a token than 8, a ragged batch and row
        _case("ragged_combine", "combine", 16, 192, 2, 12, 3001, 4104, 1024, 256, "zipf", 0.35,
              pad=0.07),
        # the replicas' gradients into the main gradients, DeepSeek-V3-shaped training layer
        _case("dsv3_grad", "grad", 64, 256, 1, 8, 4096, 7168, 2048, 1024, "zipf", 0.348,
              layer=9, groups=8, top_groups=4, copies=2),
        # relay trees of the hot experts and the packing under them, Qwen3-235B-shaped
        _case("qwen3_relay", "relay", 64, 128, 2, 8, 8192, 4096, 1536, 1024, "normal", 1.0,
              layer=8, copies=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed kinds: any supported group up to R = 64 and
    512 experts, up to 12 experts a token, 32 to 16384 tokens, rows of 256 to
    12288 elements."""
    kind = rng.choice(["step", "step", "route", "plan", "dispatch", "dispatch", "combine",
                       "combine", "grad", "relay"])
    R = rng.choice([4, 8, 12, 16, 24, 32, 48, 64])
    n_main = rng.randint(2, max(2, min(16, 512 // R)))
    E = R * n_main
    n_slot = rng.randint(1, min(4, 256 // R))
    k = rng.choice([v for v in (1, 2, 4, 6, 8, 8, 8, 10, 12) if v <= E])
    T = _log_int(rng, 32, 16384)
    H = 8 * _log_int(rng, 32, 1536)
    F = 64 * _log_int(rng, 2, 32)
    while T * k * H > (1 << 29):  # at most 1 GiB of dispatched rows
        T //= 2
    while H * F > (1 << 23):
        F = max(64, F // 128 * 64)
    mean = max(1, R * T * k // E)  # u_min about 1/32 to 1/2 of an expert's mean load
    u_min = max(1, int(mean * 2.0 ** rng.uniform(-5, -1)))
    bias, scale = rng.choice([("zipf", rng.uniform(0.2, 0.6)), ("normal", rng.uniform(0.5, 1.5)),
                              ("burst", rng.uniform(1.5, 3.0))])
    grouped = E % 8 == 0 and k <= 4 * (E // 8) and E // 8 >= 2 and rng.random() < 0.3
    c = _case("", kind, R, E, n_slot, k, T, H, F, u_min, bias, scale, rng.randrange(1, 1 << 20),
              8 if grouped else 0, 4 if grouped else 0,
              rng.choice([0.0, 0.0, rng.uniform(0.01, 0.3)]))
    del c["name"]
    return c


def _routing(c, gen, bias):
    """[T, k] int32 expert ids of one rank's tokens."""
    T, E, k = c["T"], c["E"], c["k"]
    z = torch.randn(T, E, device=DEV, generator=gen) + bias
    if c["groups"]:
        zg = z.view(T, c["groups"], E // c["groups"])
        score = zg.topk(2, dim=2).values.sum(2)
        keep = torch.zeros_like(score, dtype=torch.bool)
        keep.scatter_(1, score.topk(c["top_groups"], dim=1).indices, True)
        z = zg.masked_fill(~keep[:, :, None], float("-inf")).view(T, E)
    ids = z.topk(k, dim=1).indices.to(torch.int32)
    if c["pad"] > 0:
        ids[T - int(T * c["pad"]):] = -1
    return ids.contiguous()


def _count(c, ids):
    ids = ids.reshape(-1).to(torch.int64)
    n = torch.zeros(c["E"] + 1, dtype=torch.int32, device=DEV)  # the last bin takes the padding
    n.scatter_add_(0, torch.where(ids < 0, c["E"], ids),
                   torch.ones_like(ids, dtype=torch.int32))
    return n[:-1]


def prepare(case, seed):
    c = case
    R, E, T, k, H = c["R"], c["E"], c["T"], c["k"], c["H"]
    gen = torch.Generator(device=DEV).manual_seed(seed)
    lg = torch.Generator(device=DEV).manual_seed(7919 * c["layer"] + 13)
    if c["bias"] == "zipf":
        order = torch.rand(E, device=DEV, generator=lg).argsort().to(torch.float32)
        bias = -c["scale"] * torch.log(order + 1.0)
    elif c["bias"] == "normal":
        bias = c["scale"] * torch.randn(E, device=DEV, generator=lg)
    else:
        bias = torch.zeros(E, device=DEV)
        bias[torch.rand(E, device=DEV, generator=lg).argsort()[:8]] = c["scale"]
    ids = [_routing(c, gen, bias) for _ in range(R)]
    load = torch.stack([_count(c, t) for t in ids])
    rank = int(load.sum(0).view(R, E // R).sum(1).argmax())
    g = uep.Group(R, E, c["n_slot"], c["u_min"], 101, 100)
    W, kind = 3 * H * c["F"], c["kind"]
    n_main, cap = E // R, min(R * c["n_slot"], MAX_STAGING)
    s = dict(c=c, g=g, rank=rank, load=load.contiguous(), topk=ids[rank], W=W, cap=cap,
             plan=uep.Plan(g), status=torch.zeros(1, dtype=torch.int32, device=DEV))
    del ids

    def bf16(*shape):  # normal values, made in place: no fp32 copy of a large blob
        return torch.empty(*shape, dtype=torch.bfloat16, device=DEV).normal_(generator=gen)

    def zeros(dtype, *shape):
        return torch.zeros(*shape, dtype=dtype, device=DEV)

    if kind in ("dispatch", "combine", "grad", "relay"):  # the layer is planned already
        uep.ultraep_plan(s["load"], g, s["plan"])
    if kind in ("step", "route", "dispatch"):
        s["x"] = bf16(T, H)
        s["send"] = zeros(torch.bfloat16, T * k, H)
    if kind in ("step", "route", "dispatch", "combine"):
        s["row_of_slot"] = zeros(torch.int32, T * k)
        s["block_off"] = zeros(torch.int64, R * g.S + 1)
        s["ws"] = zeros(torch.uint8, uep.ultraep_dispatch_ws_bytes(T, k, g))
    if kind in ("route", "combine"):
        s["y"] = bf16(T * k, H)
        s["gate"] = torch.softmax(torch.randn(T, k, device=DEV, generator=gen), 1).contiguous()
        s["out"] = zeros(torch.bfloat16, T, H)
    if kind == "combine":
        uep.ultraep_dispatch_layout(s["topk"], T, k, rank, g, s["plan"], s["row_of_slot"],
                                    s["block_off"], s["ws"], s["status"])
    if kind in ("step", "relay"):
        s["w_main"] = bf16(n_main, W)
        s["staging"] = zeros(torch.bfloat16, cap, W)
        s["dest_off"] = zeros(torch.int64, R + 1)
    if kind == "relay":
        s["relay_src"] = bf16(c["n_slot"], W)
        s["slot_src"] = zeros(torch.int32, R * c["n_slot"])
        s["send_vol"] = zeros(torch.int32, R)
        s["relay_stats"] = zeros(torch.int64, 4)
    if kind == "grad":
        s["main_grad"] = torch.randn(n_main, W, device=DEV, generator=gen)
        s["rgrad"] = torch.randn(cap, W, device=DEV, generator=gen)
    return s


def _raw(t):
    return t.view(torch.int16)  # copied bytes: compared as whole numbers


def _plan_out(s):
    return {f: getattr(s["plan"], f) for f in uep.PLAN_FIELDS}


def run(s):
    c, g, plan, st, rank = s["c"], s["g"], s["plan"], s["status"], s["rank"]
    T, k, H, W, kind = c["T"], c["k"], c["H"], s["W"], c["kind"]
    if kind == "step":
        uep.ultraep_count(s["topk"], T, k, c["E"], 1, s["load"][rank], st)
        uep.ultraep_plan_replicate(s["load"], g, plan)
        uep.ultraep_reroute_and_pack(s["load"], g, plan, s["w_main"], W, rank, s["staging"],
                                     s["cap"], s["dest_off"], st)
        uep.ultraep_dispatch_layout(s["topk"], T, k, rank, g, plan, s["row_of_slot"],
                                    s["block_off"], s["ws"], st)
        uep.ultraep_dispatch_scatter(s["x"], T, k, H, s["row_of_slot"], s["block_off"][-1:],
                                     s["send"])
        return dict(_plan_out(s), load=s["load"], staging=_raw(s["staging"]),
                    dest_off=s["dest_off"], row_of_slot=s["row_of_slot"],
                    block_off=s["block_off"], send=_raw(s["send"]), status=st)
    if kind == "route":
        uep.ultraep_count(s["topk"], T, k, c["E"], 1, s["load"][rank], st)
        uep.ultraep_plan(s["load"], g, plan)
        uep.ultraep_dispatch(s["x"], s["topk"], T, k, H, rank, g, plan, s["send"],
                             s["row_of_slot"], s["block_off"], s["ws"], st)
        uep.ultraep_combine(s["y"], T * k, s["gate"], s["row_of_slot"], T, k, H, s["out"], st)
        return dict(_plan_out(s), load=s["load"], row_of_slot=s["row_of_slot"],
                    block_off=s["block_off"], send=_raw(s["send"]), out=s["out"], status=st)
    if kind == "plan":
        uep.ultraep_count(s["topk"], T, k, c["E"], 1, s["load"][rank], st)
        uep.ultraep_plan(s["load"], g, plan)
        return dict(_plan_out(s), load=s["load"], status=st)
    if kind == "dispatch":
        uep.ultraep_dispatch(s["x"], s["topk"], T, k, H, rank, g, plan, s["send"],
                             s["row_of_slot"], s["block_off"], s["ws"], st)
        return dict(row_of_slot=s["row_of_slot"], block_off=s["block_off"],
                    send=_raw(s["send"]), status=st)
    if kind == "combine":
        uep.ultraep_combine(s["y"], T * k, s["gate"], s["row_of_slot"], T, k, H, s["out"], st)
        return dict(out=s["out"], status=st)
    if kind == "grad":
        uep.ultraep_grad_reduce(s["main_grad"], s["rgrad"], W, rank, g, plan, s["cap"], st)
        return dict(main_grad=s["main_grad"], rgrad=s["rgrad"], status=st)
    uep.ultraep_relay_plan(g, plan, 4, s["slot_src"], s["send_vol"], s["relay_stats"], st)
    uep.ultraep_pack_relay(s["w_main"], s["relay_src"], W, rank, g, plan, s["slot_src"],
                           s["staging"], s["cap"], s["dest_off"], st)
    return dict(slot_src=s["slot_src"], send_vol=s["send_vol"], relay_stats=s["relay_stats"],
                staging=_raw(s["staging"]), dest_off=s["dest_off"], status=st)


def work(case):
    """Bytes read once and written once.  send and y count T * k rows (the
    padding's rows are zero-filled, or not read); the plan is its load matrix,
    quotas, host lists and reroute split."""
    c = case
    R, E, T, k, H = c["R"], c["E"], c["T"], c["k"], c["H"]
    W = 3 * H * c["F"]
    routed = (T - int(T * c["pad"])) * k
    ncol = E + R * c["n_slot"]
    ids = 4 * T * k
    plan = 4 * R * E + 4 * (R * c["n_slot"] + E * R + E + 2 * ncol + R * ncol)
    rows = 2 * T * H + 2 * T * k * H + ids          # x, send, row_of_slot
    gather = 2 * routed * H + 2 * T * H + 2 * ids   # y, out, gate and row_of_slot
    pack = 2 * W * (c["blobs"] + c["copies"])
    flops = 2 * routed * H
    kind = c["kind"]
    if kind == "step":
        return {"bytes": ids + plan + rows + pack, "flops": 0}
    if kind == "route":
        return {"bytes": ids + plan + rows + gather, "flops": flops}
    if kind == "plan":
        return {"bytes": ids + plan, "flops": 0}
    if kind == "dispatch":
        return {"bytes": ids + rows, "flops": 0}
    if kind == "combine":
        return {"bytes": gather, "flops": flops}
    if kind == "grad":
        return {"bytes": 4 * W * (2 * c["blobs"] + 2 * c["copies"]), "flops": W * c["copies"]}
    return {"bytes": pack, "flops": 0}


def tolerance(case):
    """Integers and copied bytes are exact; the fp32 sums of the combine and
    of the gradient reduction have one stated order and one rounding each, so
    they are exact too."""
    return "exact"


def exact(case, seed):
    """combine and grad in 64 bits, from the same inputs.  The other outputs
    are whole numbers and copied bytes, which have no such value."""
    c = case
    if c["kind"] not in ("combine", "grad"):
        return None
    s = prepare(case, seed)
    if c["kind"] == "combine":
        rows = s["row_of_slot"].view(c["T"], c["k"]).to(torch.int64)
        out = torch.zeros(c["T"], c["H"], dtype=torch.float64, device=DEV)
        for j in range(c["k"]):
            r = rows[:, j]
            w = torch.where(r < 0, 0.0, s["gate"][:, j].to(torch.float64))
            out += w[:, None] * s["y"][r.clamp(min=0)].to(torch.float64)
        return dict(out=out, status=None)
    n_main, rank = c["E"] // c["R"], s["rank"]
    mg = s["main_grad"].to(torch.float64)
    rg = s["rgrad"].to(torch.float64)
    entry = 0
    for e in s["plan"].slot_expert.tolist():  # destination rank, then slot
        if e >= 0 and e // n_main == rank:
            mg[e - rank * n_main] += rg[entry]
            rg[entry] = 0.0
            entry += 1
    return dict(main_grad=mg, rgrad=rg, status=None)
