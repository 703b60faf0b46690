"""The native half of the Python binding against the ctypes half: calls that
it takes and calls that it leaves to the ctypes code give the same results
and the same errors, over the argument forms the binding accepts (positional
and keyword, bf16 and int16 tensors, streams as None, torch streams and
addresses, other integer types).  Needs an MI355X."""
import ctypes
import gc
import sys
import weakref

import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import gpu_path as gp
    import paper_2606_04101_amd as uep

R, E, NS, T, k, H, W = 4, 16, 2, 65, 3, 136, 64


# the native functions: arguments in order; a tensor as its size in elements and
# its type, ws a workspace (its size is the library's to check)
I32, I64, U16, F32 = (getattr(torch, t) for t in ("int32", "int64", "int16", "float32"))
S, CAP, V = E // R + NS, 5, T * k
TOPK, ROWS, STATUS, LOAD = (V, I32), (V, I32), (1, I32), (R * E, I32)
PACKED = [(CAP * W, U16), CAP, (R + 1, I64), STATUS]
ENTRIES = {
    "count": [TOPK, T, k, E, 1, (E, I32), STATUS],
    "plan": [LOAD, "g", "plan", "ws"],
    "plan_noalloc": [LOAD, "g", "plan"],
    "plan_replicate": [LOAD, "g", "plan", "ws"],
    "plan_reroute": [LOAD, "g", "plan"],
    "dispatch": [(T * H, U16), TOPK, T, k, H, 1, "g", "plan", (V * H, U16), ROWS, (R * S + 1, I64),
                 "ws", STATUS],
    "dispatch_layout": [TOPK, T, k, 1, "g", "plan", ROWS, (R * S + 1, I64), "ws", STATUS],
    "dispatch_scatter": [(T * H, U16), T, k, H, ROWS, (1, I64), (V * H, U16)],
    "pack_replicas": [(E // R * W, U16), W, 1, "g", "plan"] + PACKED,
    "reroute_and_pack": [LOAD, "g", "plan", (E // R * W, U16), W, 1] + PACKED,
    "relay_plan": ["g", "plan", 1, (R * NS, I32), (R, I32), (4, I64), STATUS],
    "pack_relay": [(E // R * W, U16), (NS * W, U16), W, 1, "g", "plan", (R * NS, I32)] + PACKED,
    "combine": [(V * H, U16), V, (V, F32), ROWS, T, k, H, (T * H, U16), STATUS],
    "grad_reduce": [(E // R * W, F32), (CAP * W, F32), W, 1, "g", "plan", CAP, STATUS],
}


@pytest.fixture
def ctypes_only(monkeypatch):
    """The ctypes half alone: every native function declines."""
    class Declines:
        def __getattr__(self, name):
            return lambda *a: None
    def use():
        monkeypatch.setattr(uep, "_native", Declines())
    return use


def whole_step(stream):
    g = uep.Group(R, E, NS, 1)
    og = oracle.Group(R, E, NS, 1)
    rng = np.random.default_rng(5)
    tk = np.minimum(rng.geometric(0.2, (R, T, k)) - 1, E - 1).astype(np.int32)
    load, _ = oracle.count(tk, E, R)
    i32 = dict(dtype=torch.int32, device=gp.DEV)
    i64 = dict(dtype=torch.int64, device=gp.DEV)
    st = torch.zeros(1, **i32)
    rank = int(np.argmax(load.sum(0).reshape(R, -1).sum(1)))
    ld = gp.dev_i32(load)
    topk = gp.dev_i32(tk[rank])
    plan = uep.Plan(g, gp.DEV)
    for f in uep.PLAN_FIELDS:
        getattr(plan, f).fill_(-9)
    x = gp.dev_u16(rng.integers(0, 1 << 15, (T, H)).astype(np.uint16)).view(torch.bfloat16)
    w = gp.dev_u16(rng.integers(0, 1 << 15, (E // R, W)).astype(np.uint16))
    o = {n: torch.full(s, -7, **d) for n, s, d in [
        ("row_of_slot", (T * k,), i32), ("block_off", (R * g.S + 1,), i64),
        ("dest_off", (R + 1,), i64), ("slot_src", (R * NS,), i32), ("send_vol", (R,), i32),
        ("relay_stats", (4,), i64), ("load", (R, E), i32)]}
    for n, s in [("send", (T * k, H)), ("staging", (8, W)), ("relayed", (8, W)), ("out", (T, H))]:
        o[n] = torch.full(s, 77, dtype=torch.int16, device=gp.DEV)
    gate = torch.rand(T, k, device=gp.DEV, generator=torch.Generator(gp.DEV).manual_seed(1))
    o["main_grad"] = torch.ones(E // R, W, device=gp.DEV)
    o["rgrad"] = torch.full((8, W), 0.5, device=gp.DEV)
    rsrc = torch.zeros(NS, W, dtype=torch.int16, device=gp.DEV)
    ws = torch.empty(uep.ultraep_dispatch_ws_bytes(T, k, g), dtype=torch.uint8, device=gp.DEV)
    torch.cuda.synchronize()
    kw = dict(stream=stream)
    uep.ultraep_count(topk, T, k, E, 1, o["load"][rank], st, **kw)
    uep.ultraep_plan(ld, g, plan, ws=plan.ws, **kw)
    uep.ultraep_plan_noalloc(ld, g, plan, **kw)
    uep.ultraep_plan_replicate(load=ld, g=g, plan=plan, **kw)
    uep.ultraep_plan_reroute(ld, g, plan, **kw)
    uep.ultraep_reroute_and_pack(ld, g, plan, w, W, rank, o["staging"], 8, o["dest_off"], st, **kw)
    uep.ultraep_pack_replicas(w, W, rank, g, plan, o["staging"], 8, o["dest_off"], st, **kw)
    uep.ultraep_dispatch(x, topk, T, k, H, rank, g, plan, o["send"], o["row_of_slot"],
                         o["block_off"], ws, st, **kw)
    uep.ultraep_dispatch_layout(topk, T, k, rank, g, plan, o["row_of_slot"], o["block_off"], ws,
                                st, **kw)
    uep.ultraep_dispatch_scatter(x, T, k, H, o["row_of_slot"], o["block_off"][-1:], o["send"], **kw)
    uep.ultraep_combine(o["send"], T * k, gate, o["row_of_slot"], T, k, H, o["out"], st, **kw)
    uep.ultraep_grad_reduce(o["main_grad"], o["rgrad"], W, rank, g, plan, 8, st, **kw)
    uep.ultraep_relay_plan(g, plan, 1, o["slot_src"], o["send_vol"], o["relay_stats"], st, **kw)
    uep.ultraep_pack_relay(w, rsrc, W, rank, g, plan, o["slot_src"], o["relayed"], 8,
                           o["dest_off"], st, **kw)
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    o.update({f: getattr(plan, f) for f in uep.PLAN_FIELDS})
    return {n: v.cpu() for n, v in o.items()}


@pytest.mark.parametrize("how", ["none", "torch", "address"])
def test_both_halves_agree(ctypes_only, how):
    s = torch.cuda.Stream()
    stream = {"none": None, "torch": s, "address": s.cuda_stream}[how]
    a = whole_step(stream)
    ctypes_only()
    b = whole_step(stream)
    for n in a:
        assert torch.equal(a[n], b[n]), n


def test_native_half_takes_the_ordinary_call(monkeypatch):
    """No call of a step reaches the ctypes code: the native half takes every
    one of the entry points, and a refusal of the library comes through it."""
    native, seen = uep._load_native(), set()

    class Takes:
        def __getattr__(self, name):
            def call(*a):
                rc = getattr(native, name)(*a)
                assert rc is not None, name
                seen.add(name)
                return rc
            return call
    monkeypatch.setattr(uep, "_native", Takes())
    whole_step(None)
    assert seen == set(ENTRIES)
    monkeypatch.setattr(uep, "_native", native)
    monkeypatch.setattr(uep, "_need", None)
    monkeypatch.setattr(uep, "_ptr", None)
    st, c = gp.zero_status(), torch.zeros(E, dtype=torch.int32, device=gp.DEV)
    assert uep.ultraep_count(torch.zeros(6, dtype=torch.int32, device=gp.DEV), 2, 3, E, 1, c, st) == 0
    assert c[0].item() == 6
    big = torch.zeros(2000, dtype=torch.int32, device=gp.DEV)
    with pytest.raises(uep.UltraEPError):  # a refusal of the library itself (E > 1024)
        uep.ultraep_count(None, 0, 3, 2000, 1, big, st)


@pytest.mark.parametrize("name", list(ENTRIES))
def test_every_buffer_is_checked(name):
    """Each buffer of each entry point on the host, strided, one element short,
    of another element size or missing: the native half leaves the call to
    the ctypes half (nothing is enqueued), which refuses it."""
    g = uep.Group(R, E, NS, 1)
    plan = uep.Plan(g, gp.DEV)
    args = [torch.zeros(a[0], dtype=a[1], device=gp.DEV) if isinstance(a, tuple)
            else {"g": g, "plan": plan, "ws": plan.ws}.get(a, a) for a in ENTRIES[name]]
    native, python = getattr(uep._load_native(), name), getattr(uep, "ultraep_" + name)
    for i, a in enumerate(ENTRIES[name]):
        if not isinstance(args[i], torch.Tensor):
            continue
        t = args[i]
        n = t.numel()
        bad = {"host": t.cpu()}
        if n > 1:
            bad["strided"] = torch.zeros(2 * n, dtype=t.dtype, device=gp.DEV)[::2]
        if a != "ws":
            bad.update(short=t[:-1], missing=None,
                       width=torch.zeros(n, dtype=I32 if t.dtype != I32 and t.dtype != F32 else I64,
                                         device=gp.DEV))
        for how, b in bad.items():
            call = args[:i] + [b] + args[i + 1:]
            assert native(*call, None) is None, (name, i, how)
            with pytest.raises(ValueError):
                python(*call)
    for i in range(len(args)):  # and none is left out of the arguments
        assert native(*args[:i], *args[i + 1:], None) is None


@pytest.mark.parametrize("bad", ["host", "strided", "short", "width", "missing"])
def test_refusals_stay(bad):
    V = 40
    topk = torch.zeros(V, dtype=torch.int32, device=gp.DEV)
    counts = torch.zeros(E, dtype=torch.int32, device=gp.DEV)
    t = {"host": topk.cpu(), "strided": torch.zeros(2 * V, dtype=torch.int32, device=gp.DEV)[::2],
         "short": topk[:-1], "width": topk.to(torch.int64), "missing": None}[bad]
    with pytest.raises(ValueError):
        uep.ultraep_count(t, V, 1, E, 1, counts, gp.zero_status())


def test_other_argument_types():
    """Integers that are not plain ints, a subclass of Group and a plan's own
    workspace passed by hand go the way they went before."""
    counts = torch.zeros(E, dtype=torch.int32, device=gp.DEV)
    topk = torch.ones(8, dtype=torch.int32, device=gp.DEV)
    assert uep.ultraep_count(topk, 8, True, E, 1, counts, gp.zero_status()) == 0
    with pytest.raises(ctypes.ArgumentError):
        uep.ultraep_count(topk, 8, 1.0, E, 1, counts, gp.zero_status())

    class Mine(uep.Group):
        pass
    g = Mine(R, E, NS, 1)
    plan = uep.Plan(g, gp.DEV)
    load = torch.full((R, E), 3, dtype=torch.int32, device=gp.DEV)
    assert uep.ultraep_plan(load, g, plan) == 0
    with pytest.raises(uep.UltraEPError):
        uep.ultraep_plan(load, uep.Group(R, E, NS, 1), plan, ws=plan.ws[:16])
    torch.cuda.synchronize()
    assert counts[1].item() == 8


@pytest.fixture
def bound_to():
    """Binds the native half to a Python function in place of one entry point
    (nothing is enqueued), and back to the library afterwards."""
    n = uep._load_native()
    def bind(name, fn):
        n.bind({name: ctypes.cast(fn, ctypes.c_void_p).value}, uep.Group, uep.Plan, uep.PlanBuf)
        return n
    yield bind
    uep._load_native()


def test_native_half_holds_what_a_call_uses(bound_to):
    """A Plan that is given another descriptor and workspace during a call (by
    another thread, the interpreter lock being released) keeps those the call
    was made with until it returns, and not longer."""
    g = uep.Group(R, E, NS, 1)
    plan = uep.Plan(g, gp.DEV)
    refs = weakref.ref(plan.c), weakref.ref(plan.ws)
    seen = []

    @ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p, ctypes.c_void_p, ctypes.c_void_p,
                      ctypes.c_void_p, ctypes.c_size_t, ctypes.c_void_p)
    def entry(load, group, buf, ws, ws_bytes, stream):
        plan.c = plan.ws = None
        gc.collect()
        seen.append([r() is not None for r in refs])
        return 0

    n = bound_to("ultraep_plan", entry)
    load = torch.zeros(R, E, dtype=torch.int32, device=gp.DEV)
    assert n.plan(load, g, plan, None, None) == 0
    assert seen == [[True, True]]
    gc.collect()
    assert [r() for r in refs] == [None, None]


def test_native_half_keeps_no_reference_of_a_call_it_declines():
    """Among them a workspace whose memory may not be written."""
    g = uep.Group(R, E, NS, 1)
    plan = uep.Plan(g, gp.DEV)
    load = torch.zeros(R, E, dtype=torch.int32, device=gp.DEV)
    torch._C._set_throw_on_mutable_data_ptr(plan.ws)
    n, ws, c = uep._load_native(), plan.ws, plan.c
    before = sys.getrefcount(ws), sys.getrefcount(c)
    for _ in range(5):
        assert n.plan(load, g, plan, None, None) is None
        assert n.plan(load, g, plan, ws, None) is None
        assert n.plan(load[:-1], g, plan, None, None) is None
    assert (sys.getrefcount(ws), sys.getrefcount(c)) == before
