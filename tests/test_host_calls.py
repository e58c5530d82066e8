"""What the library asks of the HIP runtime, on a machine without a GPU.

The built library runs in a child process over a stand-in for the runtime
(``fake_hip.c``) that logs every launch, event and attribute call and runs no
kernel: the host side of a call (which kernels, on which streams, in which
order, with what set before) without its device side."""
from __future__ import annotations

import json
import os
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HERE = os.path.dirname(os.path.abspath(__file__))

# The child must not load torch (its HIP runtime would bind first): the
# marshalling module gets an empty stand-in for it.
PRELUDE = textwrap.dedent(r"""
    import ctypes, json, sys, types
    sys.path.insert(0, @ROOT@)
    sys.modules["torch"] = types.ModuleType("torch")
    fake = ctypes.CDLL(@FAKE@, mode=ctypes.RTLD_GLOBAL)
    fake.fake_log.restype = ctypes.c_char_p
    from paper_2609_40247_amd import herschel as H
    lib = H.load()

    def params(n=0, **kw):
        q = dict(window_begin=0, window_end=30 * 10**9, gap_threshold=0, n_procs=1, n_streams=4, n_threads=1,
                 n_names=2000, n_op_names=100, flags=3, workspace=1 << 40, workspace_bytes=1 << 50)
        q.update(kw)
        return H.HerschelParams(**q)

    EV = H.HerschelEvents(**{k: (1 << 44) + 256 * i for i, (k, _) in enumerate(H.HerschelEvents._fields_)})

    def outputs(*without):
        o = {k: (1 << 45) + 4096 * i for i, (k, _) in enumerate(H.HerschelOutputs._fields_)
             if k != "gap_capacity" and k not in without}
        return H.HerschelOutputs(gap_capacity=1 << 20, **o)

    def log():
        t = fake.fake_log().decode().splitlines()
        fake.fake_clear()
        return t

    def device(d=0, word=0, attr_result=0):
        fake.fake_set(d, word, attr_result)

    out = []
""")


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    from paper_2609_40247_amd import build, herschel
    if not os.path.exists(herschel.library_path("release")):
        build.build(checked=False)
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "fake_hip.c")], check=True)
    return so


def child(fake, body, **env):
    """Runs `body` over the stand-in; what it appends to `out`."""
    src = (PRELUDE + textwrap.dedent(body) + "\nprint(json.dumps(out))\n").replace("@ROOT@", repr(ROOT)).replace(
        "@FAKE@", repr(fake))
    r = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, timeout=120,
                       env={**os.environ, **env})
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.splitlines()[-1])


def launches(log):
    return [line.split()[1] for line in log if line.startswith("launch ")]


def test_calls_are_seen(fake):
    """The stand-in serves the library: a small window's launches, in order."""
    (code, log), = child(fake, """
        device()
        o = outputs()
        out.append((H.herschel_trace_analyze(EV, 1500, params(), o), log()))
    """)
    k = launches(log)
    assert code == 0 and len(k) == 9 and "k_finalize" in k[-1] and all("k_level" in x for x in k[:-1]), (code, k)


@pytest.mark.parametrize("entry", ["analyze", "static"])
def test_lds_limit_is_raised_on_every_device(fake, entry):
    """Launches with more dynamic LDS than the default 64 KB: the kernel's limit
    was raised on that device before, and a device that refuses it fails the
    call instead of the launch."""
    res = child(fake, f"""
        call = H.herschel_trace_analyze{"_static" if entry == "static" else ""}
        for d in (0, 1, 0, 3):
            device(d)
            out.append((d, call(EV, 1500, params(), outputs()), log()))
        device(5, 0, 1)
        out.append((5, call(EV, 1500, params(), outputs()), log()))
        device(5)
        out.append((5, call(EV, 1500, params(), outputs()), log()))
    """)
    raised = set()
    for d, code, log in res[:4] + res[5:]:
        assert code == 0
        big = 0
        for line in log:
            w = line.split()
            if w[0] == "attribute":
                raised.add((w[1], int(w[-1]), int(w[3])))
            elif w[0] == "launch" and int(w[7]) > 65536:
                big += 1
                assert any(f == w[1] and v == d and size >= int(w[7]) for f, v, size in raised), line
        assert big
    d, code, log = res[4]
    assert code == -5 and not launches(log)


def test_captured_op_name_tables_wait_for_the_sorted_lists(fake):
    """A window on three streams captured for replay keeps the edge from the
    refine pass to the op-name tables: without it the runtime lays the graph's
    branches out differently, and a replay took 266 us instead of 210."""
    (code, log), = child(fake, """
        device()
        p = params(flags=3 | H.REPLAY)
        out.append((H.herschel_trace_analyze(EV, 600_000, p, outputs()), log()))
    """)
    at = {}
    for i, line in enumerate(log):
        w = line.split()
        if w[0] == "launch":
            assert line.endswith("captured"), line
            at.setdefault(next(k for k in ("opnames_partial", "refine", w[1]) if k in w[1]), i)
    refine, tables = at["refine"], at["opnames_partial"]
    lists = next(line.split()[1] for line in log[refine:] if line.startswith("record "))
    stream = log[tables].split()[9]
    assert f"wait {lists} stream {stream}" in log[refine:tables], log
    assert code == 0 and sum(line.startswith("graph ") for line in log) == 1


@pytest.mark.parametrize("rows,captured", [(400_000, True), (600_000, False)])
def test_idle_coincidence_is_captured_on_one_stream_only(fake, rows, captured):
    """With the idle coincidence a window that takes three streams is launched
    directly also when replay is asked for."""
    (code, log), = child(fake, f"""
        device()
        out.append((H.herschel_trace_analyze(EV, {rows}, params(flags=7 | H.REPLAY), outputs()), log()))
    """)
    assert code == 0 and launches(log)
    assert any(line.startswith("capture ") for line in log) == captured


@pytest.mark.parametrize("rows", [350_000, 600_000, 20_000_000])
def test_inline_critical_path_launches(fake, rows):
    """A batch marks each window's critical path in line, with what a long path
    needs beyond the walk: launches with nothing to do in nearly every window.
    They are no more than the rounds of doubling over the window's events (two
    more for a small window, whose strides are two launches)."""
    (code, log), = child(fake, f"""
        import numpy as np
        device()
        offs = np.array([0, {rows}, {2 * rows}])
        out.append((H.herschel_trace_analyze_batch(EV, offs, [params(flags=19)] * 2, [outputs()] * 2), log()))
    """)
    needed = ("elist", "kernels", "host", "last", "ops", "rows", "local", "walk", "mark_local", "attr")
    rest = [k for k in launches(log) if "k_crit_" in k and not any(f"k_crit_{x}E" in k for x in needed)]
    rounds = (2 * rows - 1).bit_length() + 1
    assert code == 0 and len(rest) <= 2 * (rounds + (2 if rows <= 450_000 else 0)), rest[:40]


@pytest.mark.parametrize("flags,most", [(0, 450_000), (3, 450_000), (7, 450_000), (1, 450_000), (17, 360_000), (23, 360_000),
                                        (33, 280_000), (51, 280_000)])
def test_level_by_level_lines(fake, flags, most):
    """The largest windows that are launched level by level on the caller's
    stream, by their outputs (each line where three streams begin to win); with
    replay asked for and through the entry point that takes one stream, the same
    for all outputs."""
    res = child(fake, f"""
        device()
        for n in ({most}, {most} + 1):
            p = params(flags={flags}, n_graph_nodes=100)
            out.append((H.herschel_trace_analyze(EV, n, p, outputs()), log()))
        out.append((H.herschel_trace_analyze(EV, 450_000, params(flags={flags} | H.REPLAY, n_graph_nodes=100), outputs()), log()))
        out.append((H.herschel_trace_analyze_static(EV, 150_000, params(flags={flags}, n_graph_nodes=100), outputs()), log()))
    """)
    small = [any("k_level" in k for k in launches(log)) for _, log in res]
    assert all(code == 0 for code, _ in res) and small == [True, False, True, True], small
    assert not any(line.startswith(("record", "wait")) for line in res[0][1])
