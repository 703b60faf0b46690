"""The Python binding refuses tensors too small (or of the wrong element size)
for the shapes it is given, before the library is called, so that no kernel
runs past a caller's buffer.  No GPU needed: the check comes first."""
import os
import shutil
import subprocess
import sys

import pytest
import torch

import paper_2606_04101_amd as uep


def t(n, dtype=torch.int32):
    return torch.zeros(n, dtype=dtype)


G = uep.Group(4, 16, 2, 8)  # n_main = 4, S = 6, R * n_slot = 8


def test_count_buffers():
    with pytest.raises(ValueError, match="topk"):
        uep.ultraep_count(t(2 * 10 * 2 - 1), 10, 2, 16, 2, t(32), t(1))
    with pytest.raises(ValueError, match="counts"):
        uep.ultraep_count(t(40), 10, 2, 16, 2, t(31), t(1))
    with pytest.raises(ValueError, match="status"):
        uep.ultraep_count(t(40), 10, 2, 16, 2, t(32), None)


def test_plan_load():
    plan = type("P", (), {})()  # never reached
    for f in (uep.ultraep_plan, uep.ultraep_plan_replicate):
        with pytest.raises(ValueError, match="load"):
            f(t(4 * 16 - 1), G, plan, ws=t(1, torch.uint8))
    with pytest.raises(ValueError, match="load"):
        uep.ultraep_plan_reroute(t(63), G, plan)


def test_dispatch_buffers():
    T, k, H = 10, 2, 16
    ok = dict(x=t(T * H, torch.int16), topk=t(T * k), send=t(T * k * H, torch.int16),
              row_of_slot=t(T * k), block_off=t(4 * 6 + 1, torch.int64), status=t(1))
    for name, bad in [("x", t(T * H - 1, torch.int16)), ("send", t(T * k * H - 8, torch.int16)),
                      ("topk", t(T * k - 1)), ("row_of_slot", t(T * k - 1)),
                      ("block_off", t(4 * 6, torch.int64)), ("block_off", t(25, torch.int32))]:
        a = dict(ok, **{name: bad})
        with pytest.raises(ValueError, match=name):
            uep.ultraep_dispatch(a["x"], a["topk"], T, k, H, 0, G, None, a["send"],
                                 a["row_of_slot"], a["block_off"], t(1, torch.uint8), a["status"])
    with pytest.raises(ValueError, match="n_routed"):
        uep.ultraep_dispatch_scatter(ok["x"], T, k, H, ok["row_of_slot"], None, ok["send"])


def test_pack_and_relay_buffers():
    W, cap = 64, 3
    w = t(4 * W, torch.int16)
    with pytest.raises(ValueError, match="w_main"):
        uep.ultraep_pack_replicas(t(4 * W - 1, torch.int16), W, 0, G, None,
                                  t(cap * W, torch.int16), cap, t(5, torch.int64), t(1))
    with pytest.raises(ValueError, match="staging"):
        uep.ultraep_pack_replicas(w, W, 0, G, None, t(cap * W - 1, torch.int16), cap,
                                  t(5, torch.int64), t(1))
    with pytest.raises(ValueError, match="dest_off"):
        uep.ultraep_reroute_and_pack(t(64), G, None, w, W, 0, t(cap * W, torch.int16), cap,
                                     t(4, torch.int64), t(1))
    with pytest.raises(ValueError, match="relay_src"):
        uep.ultraep_pack_relay(w, t(2 * W - 1, torch.int16), W, 0, G, None, t(8),
                               t(cap * W, torch.int16), cap, t(5, torch.int64), t(1))
    with pytest.raises(ValueError, match="send_vol"):
        uep.ultraep_relay_plan(G, None, 4, t(8), t(3), t(4, torch.int64), t(1))
    with pytest.raises(ValueError, match="relay_stats"):
        uep.ultraep_relay_plan(G, None, 4, t(8), t(4), t(4), t(1))


def test_combine_and_reduce_buffers():
    T, k, H = 5, 3, 8
    args = dict(y=t(15 * H, torch.int16), gate=t(T * k, torch.float32), ros=t(T * k),
                out=t(T * H, torch.int16))
    for name, key, bad in [("y", "y", t(15 * H - 1, torch.int16)),
                           ("gate", "gate", t(T * k, torch.float16)),
                           ("row_of_slot", "ros", t(T * k - 1)),
                           ("out", "out", t(T * H, torch.float32))]:
        a = dict(args, **{key: bad})
        with pytest.raises(ValueError, match=name):
            uep.ultraep_combine(a["y"], 15, a["gate"], a["ros"], T, k, H, a["out"], t(1))
    with pytest.raises(ValueError, match="main_grad"):
        uep.ultraep_grad_reduce(t(4 * 8 - 1, torch.float32), t(8, torch.float32), 8, 0, G, None,
                                1, t(1))
    with pytest.raises(ValueError, match="rgrad"):
        uep.ultraep_grad_reduce(t(32, torch.float32), t(2 * 8, torch.int16), 8, 0, G, None, 2,
                                t(1))


def test_native_half_declines_host_tensors():
    """What the native half does not take it leaves to the code above: host
    tensors, missing ones, too few arguments and other types give None."""
    n = uep._load_native()
    assert n.count(t(40), 10, 2, 16, 2, t(32), t(1), 0) is None
    assert n.count(None, 0, 2, 16, 2, None, None, 0) is None
    assert n.count(t(40), 10.0, 2, 16, 2, t(32), t(1), 0) is None
    assert n.count(t(40), 1 << 70, 2, 16, 2, t(32), t(1), 0) is None
    assert n.count(t(40)) is None
    assert n.plan(t(64), G, object(), None, 0) is None
    assert n.plan(t(64), (4, 16, 2, 8), None, None, 0) is None


@pytest.mark.parametrize("native", ["missing", "no_library", "other_torch"])
def test_calls_without_the_native_half(native, tmp_path):
    """Where _native.so is absent or does not fit, calls go through ctypes:
    the same refusals, from the binding's checks and from the library."""
    src = os.path.dirname(uep.__file__)
    pkg = tmp_path / "paper_2606_04101_amd"
    pkg.mkdir()
    for f in ("__init__.py", "_build.py", "libultraep.so"):
        shutil.copy(os.path.join(src, f), pkg / f)
    if native == "no_library":
        (pkg / "_native.so").write_text("not a library")
    elif native == "other_torch":
        shutil.copy(os.path.join(src, "_native.so"), pkg / "_native.so")
    code = f"""
import sys, warnings
sys.path.insert(0, {str(tmp_path)!r})
import torch
import paper_2606_04101_amd as uep
if {native!r} == "other_torch":
    torch.__version__ = "0.1"
with warnings.catch_warnings(record=True) as w:
    warnings.simplefilter("always")
    for _ in range(2):
        try:
            uep.ultraep_dispatch_scatter(None, 0, 1, 7, None, None, None, stream=0)
        except uep.UltraEPError as e:
            assert e.code == uep.ULTRAEP_EINVAL
        else:
            raise AssertionError("not refused")
    try:
        uep.ultraep_count(torch.zeros(39, dtype=torch.int32), 10, 2, 16, 2, None, None, stream=0)
    except ValueError as e:
        assert "topk" in str(e)
    else:
        raise AssertionError("not refused")
assert [v.category for v in w if "ctypes" in str(v.message)] == [RuntimeWarning]
"""
    env = {k: v for k, v in os.environ.items() if k != "ULTRAEP_LIB"}
    r = subprocess.run([sys.executable, "-c", code], cwd=tmp_path, env=env, timeout=300,
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr


def test_library_builds_without_the_native_half(monkeypatch, tmp_path):
    """A torch without headers, or no host compiler: the library is built all
    the same, and no file of an earlier build is left to be loaded with it."""
    from paper_2606_04101_amd import _build
    for name in ("LIB", "NATIVE"):
        monkeypatch.setattr(_build, name, str(tmp_path / os.path.basename(getattr(_build, name))))
    stale = tmp_path / "_native.so"
    stale.write_text("earlier build")

    def fails():
        raise RuntimeError("no headers")
    done = []

    def run(cmd, **kw):
        done.append(cmd)
        open(cmd[cmd.index("-o") + 1], "w").close()
        return subprocess.CompletedProcess(cmd, 0, "", "")
    monkeypatch.setattr(_build, "build_native", fails)
    monkeypatch.setattr(_build.subprocess, "run", run)
    monkeypatch.setattr(_build, "HERE", str(tmp_path))
    with pytest.warns(RuntimeWarning, match="no headers"):
        assert _build.build() == str(tmp_path / "libultraep.so")
    assert len(done) == len(_build.SOURCES) + 1
    assert (tmp_path / "libultraep.so").exists() and not stale.exists()
