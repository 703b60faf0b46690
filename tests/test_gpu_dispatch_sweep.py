"""A wide randomized sweep of the whole path on small rows: 1000 seeded
groups (1 to 64 ranks, up to 1024 experts, 0 to 4 redundant slots per rank)
and routings (distinct top-k per token from uniform, Zipf-skewed or hot-rank
expert popularity, a quarter of the slots masked, or ids with repeats), from
0 to 2500 tokens per rank and top-1 to top-8.  The counts, every plan buffer,
and for two ranks the dispatch (send, row_of_slot, block_off, through both
the one-call and the split entry points) and the packing (staging, dest_off)
are compared with the oracle byte for byte; a second sweep covers the
relay trees, the relay packing, the combine gather and the gradient
reduction.  Needs an MI355X."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    import gpu_path as gp
    import paper_2606_04101_amd as uep


def sweep_routing(seed):
    rng = np.random.default_rng(70_000 + seed)
    R = int(rng.choice([1, 2, 3, 4, 7, 8, 16, 24, 32, 64]))
    nm = int(rng.choice([1, 2, 3, 4, 8, 16]))
    nm = min(nm, 1024 // R)
    E = R * nm
    NS = min(int(rng.integers(0, 5)), 256 // R)
    k = int(min(rng.choice([1, 2, 4, 6, 8]), E))
    T = int(rng.choice([0, 1, 37, 500, 1024, 2500]))
    u_min = int(rng.choice([1, 4, 16, 64]))
    kind = int(rng.integers(0, 5))
    if kind == 0:
        p = np.full(E, 1.0 / E)
    elif kind == 1:  # Zipf-skewed expert popularity
        p = 1.0 / np.arange(1, E + 1) ** rng.uniform(0.5, 1.5)
        rng.shuffle(p)
        p /= p.sum()
    else:  # the experts of a few ranks are hot
        p = np.ones(E)
        for h in rng.choice(R, max(1, R // 4), replace=False):
            p[h * nm:(h + 1) * nm] *= rng.uniform(5, 40)
        p /= p.sum()
    tk = rng.choice(E, (R, T, k), p=p).astype(np.int32)
    if kind != 4:  # distinct experts per token: redraw repeats (kind 4 keeps them)
        for j in range(1, k):
            for _ in range(64):
                dup = (tk[:, :, j:j + 1] == tk[:, :, :j]).any(axis=2)
                if not dup.any():
                    break
                tk[:, :, j][dup] = rng.choice(E, int(dup.sum()), p=p)
    if kind == 3:
        tk[rng.random(tk.shape) < 0.25] = -1
    H = 8 * int(rng.integers(1, 25))
    W = 8 * int(rng.integers(1, 65))
    return rng, tk, R, E, NS, k, T, u_min, H, W


@pytest.mark.parametrize("block", range(4))
def test_dispatch_sweep(block):
    checked = 0
    for seed in range(block * 250, (block + 1) * 250):
        rng, tk, R, E, NS, k, T, u_min, H, W = sweep_routing(seed)
        where = f"seed {seed} (R={R} E={E} n_slot={NS} k={k} T={T} u_min={u_min} H={H} W={W})"
        g, og = gp.groups(R, E, NS, u_min)
        try:
            load, ost = oracle.count(tk, E, R)
            assert ost == 0
            if T > 0:
                counts, st = gp.gpu_count(tk, E)
                assert st == 0
                gp.assert_same("counts", counts, load)
            op = oracle.plan(load, og)
            if op.status != oracle.OK:
                continue
            plan = gp.gpu_plan(load, g)
            gp.assert_plan_equal(plan, op)
            X = op.slot_expert.reshape(R, max(NS, 0))
            outb = [int(((X >= 0) & (X // (E // R) == r)).sum()) for r in range(R)]
            for i, r in enumerate(sorted({int(np.argmax(outb)), int(rng.integers(0, R))})):
                x = rng.integers(0, 1 << 16, (T, H)).astype(np.uint16)
                w = rng.integers(0, 1 << 16, (E // R, W)).astype(np.uint16)
                gp.check_rank(x, tk[r], w, r, g, og, plan, op, split=bool((seed + i) % 2))
        except AssertionError as ex:
            raise AssertionError(f"{where}: {ex}") from None
        checked += 1
    assert checked > 200


@pytest.mark.parametrize("block", range(2))
def test_extension_sweep(block):
    """The adjacent steps on the same routings: relay trees at thresholds 0
    and 2 and the relay packing of two ranks, the combine gather of one
    rank's dispatched rows with softmax gates, and the gradient reduction of
    two ranks, against the oracle."""
    from test_gpu_combine_reduce import bf16_normals, check_combine, check_reduce, softmax_gates
    from test_gpu_relay import check as check_relay
    from test_gpu_relay import check_pack_relay
    checked = 0
    for seed in range(1000 + block * 150, 1000 + (block + 1) * 150):
        rng, tk, R, E, NS, k, T, u_min, H, W = sweep_routing(seed)
        where = f"seed {seed} (R={R} E={E} n_slot={NS} k={k} T={T} u_min={u_min} H={H} W={W})"
        g, og = gp.groups(R, E, NS, u_min)
        try:
            load, _ = oracle.count(tk, E, R)
            op = oracle.plan(load, og)
            if op.status != oracle.OK:
                continue
            plan = gp.gpu_plan(load, g)
            gp.assert_plan_equal(plan, op)
            X = op.slot_expert.reshape(R, max(NS, 0))
            outb = [int(((X >= 0) & (X // (E // R) == r)).sum()) for r in range(R)]
            ranks = sorted({int(np.argmax(outb)), int(rng.integers(0, R))})
            for threshold in (0, 2):
                rel = check_relay(g, og, plan, op, threshold)
                check_pack_relay(g, og, plan, op.slot_expert, rel, W, seed, ranks=ranks)
            r = ranks[-1]
            if T > 0:
                send, ros, _, st = gp.gpu_dispatch(bf16_normals(rng, (T, H)), tk[r], r, g, plan)
                assert st == 0
                check_combine(send, softmax_gates(rng, T, k), ros)
            for r in ranks:
                check_reduce(g, og, plan, op.slot_expert, r, 4 * int(rng.integers(1, 200)), rng)
        except AssertionError as ex:
            raise AssertionError(f"{where}: {ex}") from None
        checked += 1
    assert checked > 120


# rows in one unit and cut into units of 1, 2, 4 and 8 chunks per lane (few
# tokens, wide rows), widths around the units' edges, tokens around the rule
@pytest.mark.parametrize("T,k", [(1, 1), (5, 3), (300, 2), (767, 2), (768, 2), (1030, 1)])
@pytest.mark.parametrize("H", [8, 512, 520, 1032, 4096, 4104, 7168, 8192, 8200, 12296])
def test_scatter_units(T, k, H):
    rng = np.random.default_rng(T * 10 + H)
    V = T * k
    x = rng.integers(0, 1 << 16, (T, H)).astype(np.uint16)
    routed = rng.random(V) >= 0.2
    ros = np.full(V, -1, np.int32)
    nr = int(routed.sum())
    ros[routed] = rng.permutation(nr)
    send = torch.full((V, H), 0x5A5A, dtype=torch.int16, device=gp.DEV)
    uep.ultraep_dispatch_scatter(gp.dev_u16(x), T, k, H, gp.dev_i32(ros),
                                 torch.tensor([nr], dtype=torch.int64, device=gp.DEV), send)
    torch.cuda.synchronize()
    ref = np.zeros((V, H), np.uint16)
    ref[ros[routed]] = x[np.arange(V)[routed] // k]
    assert np.array_equal(gp.host_u16(send), ref)


# the lines between whole rows and cut ones, the units over and under the resident
# waves, and wide rows in equal pieces with ordinary stores (whole lines or not,
# one and several units per wave, a last piece of one chunk)
@pytest.mark.parametrize("T,k,H", [
    (511, 16, 1032), (639, 8, 4608), (640, 8, 4608), (767, 8, 4096), (683, 3, 6144),
    (682, 3, 4104), (511, 16, 2048), (512, 16, 2048), (511, 12, 4608), (512, 12, 4608), (399, 2, 8200), (400, 2, 8200), (682, 1, 8704),
    (683, 1, 8704), (911, 2, 8704), (911, 2, 8736), (1100, 1, 8200),
    (267, 3, 16392), (266, 3, 16392), (1367, 1, 24576), (499, 9, 8200), (500, 8, 8200), (503, 9, 24584),
    (400, 16, 8200), (399, 16, 8264), (4099, 1, 8200)])
def test_scatter_lines(T, k, H):
    rng = np.random.default_rng(T + k + H)
    V = T * k
    x = rng.integers(0, 1 << 16, (T, H), dtype=np.uint16)
    routed = rng.random(V) >= 0.1
    ros = np.full(V, -1, np.int32)
    nr = int(routed.sum())
    ros[routed] = rng.permutation(nr)
    room = torch.full((V + 2, H), 0x5A5A, dtype=torch.int16, device=gp.DEV)
    uep.ultraep_dispatch_scatter(gp.dev_u16(x), T, k, H, gp.dev_i32(ros),
                                 torch.tensor([nr], dtype=torch.int64, device=gp.DEV), room[1:-1])
    torch.cuda.synchronize()
    ref = np.zeros((V, H), np.uint16)
    ref[ros[routed]] = x[np.arange(V)[routed] // k]
    assert np.array_equal(gp.host_u16(room[1:-1].contiguous()), ref)
    assert (room[0] == 0x5A5A).all() and (room[-1] == 0x5A5A).all()


# the sums over chunk histograms: threads per expert from 1 to many, chunk
# counts around the first batch of loads and over several batches
@pytest.mark.parametrize("R,E", [(1, 1), (3, 6), (8, 128), (4, 300), (8, 1000), (16, 1024)])
@pytest.mark.parametrize("T", [1, 2049, 4 * 2048, 4 * 2048 + 1, 18 * 2048 + 77, 70 * 2048])
def test_layout_chunk_sums(R, E, T):
    rng = np.random.default_rng(T + E)
    tk = np.minimum(rng.geometric(min(1.0, 8 / E), (R, T, 1)) - 1, E - 1).astype(np.int32)
    tk[rng.random(tk.shape) < 0.1] = -1
    g, og = gp.groups(R, E, 1, max(1, T // 64))
    load, _ = oracle.count(tk, E, R)
    op = oracle.plan(load, og)
    plan = gp.gpu_plan(load, g)
    x = (np.arange(T * 8) & 0xFFFF).astype(np.uint16).reshape(T, 8)
    rank = R - 1
    send, ros, off, st = gp.gpu_dispatch(x, tk[rank], rank, g, plan)
    assert st == 0
    osend, oros, ooff, ost = oracle.dispatch(x, tk[rank], rank, og, op)
    assert np.array_equal(ros, oros) and np.array_equal(off, ooff)
    assert np.array_equal(send, osend)


# one launch up to 10 chunks of 2048 slots (fewer with less than 10 experts, two
# launches when the tables do not fit LDS), around each edge
@pytest.mark.parametrize("R,E,NS", [(1, 2, 0), (2, 6, 1), (64, 64, 4), (64, 128, 2), (32, 512, 8), (16, 1024, 2)])
@pytest.mark.parametrize("V", [1, 2047, 2048, 2049, 3 * 2048, 10 * 2048 - 1, 10 * 2048, 10 * 2048 + 1])
def test_layout_one_launch(R, E, NS, V):
    rng = np.random.default_rng(V + E)
    tk = np.minimum(rng.geometric(min(1.0, 6 / E), (R, V, 1)) - 1, E - 1).astype(np.int32)
    tk[rng.random(tk.shape) < 0.1] = -1
    g, og = gp.groups(R, E, NS, 1)
    load, _ = oracle.count(tk, E, R)
    op = oracle.plan(load, og)
    plan = gp.gpu_plan(load, g)
    x = (np.arange(V * 8) & 0xFFFF).astype(np.uint16).reshape(V, 8)
    for rank in {0, R - 1}:
        send, ros, off, st = gp.gpu_dispatch(x, tk[rank], rank, g, plan)
        assert st == 0
        osend, oros, ooff, ost = oracle.dispatch(x, tk[rank], rank, og, op)
        assert np.array_equal(ros, oros) and np.array_equal(off, ooff)
        assert np.array_equal(send, osend)
    # ids out of range, ids that the shares do not match, host lists of no group
    bad = tk[0].copy()
    bad[V // 2, 0] = E
    assert gp.gpu_dispatch(x, bad, 0, g, plan)[3] == uep.ULTRAEP_EDATA
    bad[V // 2, 0] = -1 if tk[0][V // 2, 0] >= 0 else 0
    assert gp.gpu_dispatch(x, bad, 0, g, plan)[3] == uep.ULTRAEP_EDATA
    plan.host_ptr[E] = E + R * NS + 1
    assert gp.gpu_dispatch(x, tk[0], 0, g, plan)[3] == uep.ULTRAEP_EDATA


@pytest.mark.parametrize("V", [700, 2048, 2049, 5 * 2048 + 3, 10 * 2048, 12 * 2048])
def test_layout_in_place(V):
    """row_of_slot may be the ids' own memory: every id is read before a row
    takes its place, at one chunk of 2048 slots, at several and past the one
    launch."""
    R, E, NS = 8, 64, 2
    rng = np.random.default_rng(V)
    tk = np.minimum(rng.geometric(0.1, (R, V, 1)) - 1, E - 1).astype(np.int32)
    tk[rng.random(tk.shape) < 0.1] = -1
    g, og = gp.groups(R, E, NS, 1)
    load, _ = oracle.count(tk, E, R)
    plan = gp.gpu_plan(load, g)
    ids = gp.dev_i32(tk[3])
    off = torch.empty(R * g.S + 1, dtype=torch.int64, device=gp.DEV)
    ws = torch.empty(uep.ultraep_dispatch_ws_bytes(V, 1, g), dtype=torch.uint8, device=gp.DEV)
    st = gp.zero_status()
    uep.ultraep_dispatch_layout(ids, V, 1, 3, g, plan, ids, off, ws, st)
    torch.cuda.synchronize()
    assert int(st.item()) == 0
    x = np.zeros((V, 8), np.uint16)
    _, oros, ooff, _ = oracle.dispatch(x, tk[3], 3, og, oracle.plan(load, og))
    assert np.array_equal(ids.cpu().numpy().reshape(-1), oros.reshape(-1))
    assert np.array_equal(off.cpu().numpy(), ooff)


# the one launch's counts in 8, 4, 2 and 1 copies (as many as LDS holds), up to
# the chunks that each takes and past them, half of the ids one expert
@pytest.mark.parametrize("R,E,NS", [(64, 512, 4), (64, 640, 1), (64, 640, 4), (64, 704, 1)])
@pytest.mark.parametrize("V", [2 * 2048, 2 * 2048 + 65, 3 * 2048, 4 * 2048, 5 * 2048, 5 * 2048 + 1,
                               8 * 2048, 8 * 2048 + 1])
def test_layout_copies_of_the_counts(R, E, NS, V):
    rng = np.random.default_rng(V + E + NS)
    tk = rng.integers(-1, E, (R, V, 1)).astype(np.int32)
    tk[rng.random(tk.shape) < 0.5] = E // 3
    g, og = gp.groups(R, E, NS, 7)
    load, _ = oracle.count(tk, E, R)
    op = oracle.plan(load, og)
    plan = gp.gpu_plan(load, g)
    x = (np.arange(V * 8) & 0xFFFF).astype(np.uint16).reshape(V, 8)
    send, ros, off, st = gp.gpu_dispatch(x, tk[1], 1, g, plan)
    assert st == 0
    osend, oros, ooff, ost = oracle.dispatch(x, tk[1], 1, og, op)
    assert np.array_equal(ros, oros) and np.array_equal(off, ooff)
    assert np.array_equal(send, osend)


# the sums over chunk histograms where few threads share them (16 of E = 1, 9
# and 64, one of E = 600 with threads left over) and around their batches
# of 4, 4 and 12 loads per thread
@pytest.mark.parametrize("R,E", [(1, 1), (3, 9), (16, 64), (8, 600)])
@pytest.mark.parametrize("chunks", [11, 16 * 4 + 1, 16 * 8 + 1, 16 * 16 + 3])
def test_layout_chunk_sum_batches(R, E, chunks):
    V = chunks * 2048 - 77
    rng = np.random.default_rng(chunks + E)
    tk = rng.integers(-1, E, (V, 1)).astype(np.int32)
    load = np.tile(np.bincount(tk[tk >= 0], minlength=E).astype(np.int32), (R, 1))
    g, og = gp.groups(R, E, 1, 50)
    plan, op = gp.gpu_plan(load, g), oracle.plan(load, og)
    x = (np.arange(V * 8) & 0xFFFF).astype(np.uint16).reshape(V, 8)
    send, ros, off, st = gp.gpu_dispatch(x, tk, R - 1, g, plan)
    assert st == 0
    osend, oros, ooff, ost = oracle.dispatch(x, tk, R - 1, og, op)
    assert np.array_equal(ros, oros) and np.array_equal(off, ooff)
    assert np.array_equal(send, osend)
