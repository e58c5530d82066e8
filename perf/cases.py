"""Workloads for measuring the trace analyzer through its public entry points.

Every case is one profiling window (or a batch of windows) of the kind that
``paper_2609_40247_amd/synth.py`` describes: steps of kernels queued per device
stream, a launch for each kernel (or one per replayed graph), a forest of CPU
ops over the launches, rows in delivery order.  The generator below follows
the same recipe with torch on the GPU, so that a window of 24 million rows is
made in a fraction of a second; row counts depend on the case alone, contents
on the seed.  Times, ids and names have the distributions of the recipe:
log-normal kernel durations around 6 us, exponential queue gaps with 1% long
stalls, Zipf names, ids rising in launch order.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2609_40247_amd import herschel as H
from paper_2609_40247_amd.synth import EDGE_DTYPE

DEV = "cuda"
US, MS, S = 1_000, 1_000_000, 1_000_000_000
EPOCH = 1_765_000_000 * S
CPU_OP, LAUNCH, KERNEL = 0, 1, 2
DROP, BLOCK = 0.01, 4096
CONTAIN, OVERLAP, WAITS, SOL, CRIT, GRAPH = 1, 2, 4, 8, 16, 32

DEFAULTS = dict(entry="analyze", kernels=1000, per_step=1000, period_us=30_000, procs=1, streams=4, threads=1,
                names=2000, op_names=100, threshold_us=20, flags=3, order="delivery", ids="dense", edges=0, nodes=0,
                mixed=False, traces=1, smallest=0, chunk=1)


def _full(case: dict) -> dict:
    return {**DEFAULTS, **case}


def listed() -> list:
    return [
        # one decode step of a small service, the smallest window anyone asks for: a call is its launches and latency
        dict(name="one_step", kernels=500, per_step=500, streams=2, names=200),
        # the repository's tiny trace: a 10 s window of 20k kernels on two streams, nested three deep
        dict(name="tiny_window", kernels=20_000, per_step=20_000, period_us=10_000_000, streams=2, names=200,
             threshold_us=50),
        # the entry point for hosts that may not allocate (a serving loop's own analysis): 200 decode steps
        dict(name="static_window", entry="static", kernels=90_003, per_step=500),
        # the headline workload: 30 s of decode steps, 1000 kernels each, every default output
        dict(name="decode", kernels=1_001_000),
        # prefill beside decode: 8 streams (compute, communication, copies), long and short kernels together
        dict(name="prefill_decode", kernels=1_154_153, per_step=1153, streams=8, threads=2, mixed=True),
        # a node: 8 processes with clock offsets and cross-process dependency edges
        dict(name="node", kernels=1_001_000, procs=8, edges=20_000),
        # the batch of many windows per call, with only the aggregate outputs (names, busy / idle, gaps, latencies)
        dict(name="batch", entry="batch", kernels=2_000_000, smallest=200_000, traces=8, flags=0),
        # the same batch streamed from pinned host memory in chunks: windows kept by a collector
        dict(name="streamed", entry="chunked", kernels=400_000, smallest=50_000, traces=6, chunk=2, flags=0),
        # idle evidence: the GPU's idle time inside the CPU ops, by op name
        dict(name="idle_evidence", kernels=1_001_000, flags=CONTAIN | OVERLAP | WAITS),
        # the critical path of a shorter window, at an odd size
        dict(name="critical_path", kernels=500_557, per_step=997, flags=CONTAIN | OVERLAP | CRIT),
        # graph replay: one launch a step owns its 1000 kernels; operator efficiency from the ops' counts
        dict(name="graph_replay", kernels=200_000, streams=2, nodes=1000, flags=CONTAIN | SOL | GRAPH),
        # every output over a merged trace: 4 processes (two replay graphs), 16 streams,
        # opaque ids, rows in no order, a ragged size
        dict(name="merged_all", kernels=25_013, per_step=333, procs=4, streams=16, threads=3, order="shuffled",
             ids="sparse", edges=501, nodes=333, flags=63),
    ]


def draw(rng) -> dict:
    """A window of the same ranges: 1.5 thousand to 8 million rows."""
    what = rng.choice(["plain", "plain", "plain", "mixed", "node", "static", "batch", "streamed", "waits", "crit",
                       "graph", "merged"])
    span = lambda lo, hi: int(math.exp(rng.uniform(math.log(lo), math.log(hi)))) | 1  # noqa: E731
    c = dict(per_step=rng.randint(100, 2500), names=rng.choice([200, 2000, 3001]), op_names=rng.choice([37, 100, 333]))
    if what == "plain":
        c.update(kernels=span(500, 1_500_000), streams=rng.randint(1, 8), threads=rng.randint(1, 3),
                 order=rng.choice(["delivery", "delivery", "shuffled"]), ids=rng.choice(["dense", "dense", "sparse"]),
                 flags=rng.choice([0, 1, 2, 3, 3]))
    elif what == "mixed":
        c.update(kernels=span(50_000, 1_200_000), per_step=rng.randint(500, 1500), streams=8, threads=2, mixed=True)
    elif what == "node":
        p = rng.randint(2, 12)
        c.update(kernels=span(2_000, 2_000_000 // p), procs=p, edges=rng.randint(1, 20_000))
    elif what == "static":
        c.update(entry="static", kernels=span(500, 85_000))
    elif what == "batch":
        c.update(entry="batch", kernels=span(50_000, 800_000), smallest=20_000, traces=rng.randint(2, 7), flags=0)
    elif what == "streamed":
        c.update(entry="chunked", kernels=span(20_000, 300_000), smallest=10_000, traces=rng.randint(2, 6),
                 chunk=rng.randint(1, 3), flags=0)
    elif what == "waits":
        c.update(kernels=span(1_000, 1_000_000), streams=rng.randint(1, 8), flags=7)
    elif what == "crit":
        c.update(kernels=span(1_000, 800_000), procs=rng.randint(1, 2), flags=19)
    elif what == "graph":
        c.update(kernels=span(10_000, 600_000), nodes=1, streams=rng.randint(1, 4), flags=41)
        c["nodes"] = c["per_step"]
    else:
        p = rng.randint(1, 5)
        c.update(kernels=span(500, 300_000 // p), procs=p, streams=rng.randint(2, 20), threads=rng.randint(1, 4),
                 order="shuffled", ids="sparse", edges=rng.randint(1, 2000), nodes=1, flags=63)
        c["nodes"] = c["per_step"]
    return c


# ------------------------------------------------------------- the generator
def _kernels(g, K, per_step, period, t0, streams, weights, median, sigma):
    """Kernel timeline of one phase: start, end, stream and step, K each."""
    i = torch.arange(K, device=DEV)
    step = i // per_step
    n_steps = (K + per_step - 1) // per_step
    w = torch.tensor(weights, dtype=torch.float64, device=DEV)
    cdf = torch.cumsum(w / w.sum(), 0)
    which = torch.searchsorted(cdf, torch.rand(K, dtype=torch.float64, device=DEV, generator=g), right=True)
    stream = torch.tensor(streams, device=DEV)[which.clamp(max=len(streams) - 1)]
    dur = torch.empty(K, dtype=torch.float64, device=DEV).log_normal_(math.log(median), sigma, generator=g)
    dur = dur.round().clamp(min=1, max=2 * S).long()
    gap = torch.empty(K, dtype=torch.float64, device=DEV).exponential_(1 / (3 * US), generator=g).round().long()
    stall = torch.rand(K, device=DEV, generator=g) < 0.01
    gap += stall * torch.randint(200 * US, 5 * MS, (K,), device=DEV, generator=g)
    order = torch.sort(step * 64 + stream, stable=True).indices
    grp = (step * 64 + stream)[order]
    v = (gap + dur)[order]
    cs = torch.cumsum(v, 0)
    head = torch.ones(K, dtype=torch.bool, device=DEV)
    head[1:] = grp[1:] != grp[:-1]
    base = torch.cummax(torch.where(head, cs - v, torch.full_like(cs, -1)), 0).values
    rel_end = torch.empty_like(cs)
    rel_end[order] = cs - base
    length = torch.zeros(n_steps, dtype=torch.int64, device=DEV).scatter_reduce_(0, step, rel_end, "amax")
    before = torch.cumsum(length, 0) - length
    s = torch.cummax(t0 + torch.arange(n_steps, device=DEV) * period - before, 0).values + before
    end = s[step] + rel_end
    return end - dur, end, stream, step


def _ops(g, points, thread, step, want):
    """Exactly `want` CPU ops over launch points sorted by (thread, time): a
    nested forest, four levels deep, with leaf ops that launch nothing."""
    L, depth = len(points), 4
    last = torch.ones(L, dtype=torch.bool, device=DEV)  # no point of the same thread follows
    last[:-1] = thread[1:] != thread[:-1]
    far = torch.full((L,), 10_000, dtype=torch.int64, device=DEV)
    gapr = far.clone()
    gapr[:-1] = torch.where(last[:-1], far[:-1], points[1:] - points[:-1])
    gapl = far.clone()
    gapl[1:] = gapr[:-1]
    lam = torch.full((L,), depth, dtype=torch.int64, device=DEV)
    u = torch.rand(L, device=DEV, generator=g)
    for d, p in ((3, 1 / 1.5), (2, 1 / 6), (1, 1 / 50)):
        lam[u < p] = d
    lam[gapr < 8] = depth
    cut = last.clone()
    cut[:-1] |= step[1:] != step[:-1]
    lam[cut] = 0
    # about 2% of the launches, the first ones of a root, lie in no op
    start = torch.ones(L, dtype=torch.bool, device=DEV)
    start[1:] = lam[:-1] == 0
    root = torch.cumsum(start.long(), 0) - 1
    first = torch.nonzero(start).flatten()
    size = torch.diff(first, append=torch.tensor([L], device=DEV))
    orph = (size * 0.02 + torch.rand(len(size), device=DEV, generator=g)).floor().long()
    orph = torch.minimum(orph, size - 1)
    pos = torch.arange(L, device=DEV) - first[root]
    orphan = pos < orph[root]
    lam[pos == orph[root] - 1] = 0
    ts, te = [], []
    for d in range(depth):
        f = 0.4 * (depth - d) / depth
        b = torch.nonzero(lam <= d).flatten()
        a = torch.cat([torch.zeros(1, dtype=torch.int64, device=DEV), b[:-1] + 1])
        keep = ~orphan[a]
        a, b = a[keep], b[keep]
        ts.append(points[a] - (gapl[a] * f).floor().long())
        te.append(points[b] + 1 + ((gapr[b] - 1) * f).floor().long())
        if d == 0:
            thr = [thread[a]]
        else:
            thr.append(thread[a])
    ts, te, thr = torch.cat(ts), torch.cat(te), torch.cat(thr)
    if len(ts) < want:
        ok = torch.nonzero((lam > 0) & (gapr >= 40) & ~orphan).flatten()
        pick = ok[torch.randperm(len(ok), device=DEV, generator=g)[:want - len(ts)]]
        gp = gapr[pick]
        ts = torch.cat([ts, points[pick] + (gp * 0.42).ceil().long()])
        te = torch.cat([te, points[pick] + (gp * 0.58).floor().long()])
        thr = torch.cat([thr, thread[pick]])
    if len(ts) < want:  # markers of no length
        pick = torch.randint(0, L, (want - len(ts),), device=DEV, generator=g)
        ts, te, thr = torch.cat([ts, points[pick]]), torch.cat([te, points[pick]]), torch.cat([thr, thread[pick]])
    if len(ts) > want:
        keep = torch.randperm(len(ts), device=DEV, generator=g)[:want].sort().values
        ts, te, thr = ts[keep], te[keep], thr[keep]
    return ts, te, thr


def _zipf(g, names, count):
    cdf = torch.cumsum(torch.arange(1, names + 1, dtype=torch.float64, device=DEV) ** -1.1, 0)
    u = torch.rand(count, dtype=torch.float64, device=DEV, generator=g) * cdf[-1]
    return torch.searchsorted(cdf, u, right=True).clamp(max=names - 1)


def _prefill_kernels(c, K):
    return int(K * 0.45) if c["mixed"] else 0


def _replays(c, p) -> bool:
    """Process p replays a captured graph each step (of several processes, every other one)."""
    return c["nodes"] > 0 and (c["procs"] == 1 or p % 2 == 1)


def _counts(c, K, p=0):
    """(launches, kernels recorded, CPU ops) of process p with K decode kernels."""
    k = K + _prefill_kernels(c, K)
    launches = (K + c["per_step"] - 1) // c["per_step"] if _replays(c, p) else k
    return launches, k - int(k * DROP), launches


def rows(c, K) -> int:
    return sum(sum(_counts(c, K, p)) for p in range(c["procs"]))


def _window(c, K) -> int:
    return max(1, K // c["per_step"]) * c["period_us"] * US


def _process(g, c, K, p, offset):
    """Columns of one process, one tuple per kind: ts, te, corr, lane, name, node."""
    period = c["period_us"] * US
    if c["mixed"]:
        side = list(range(4, c["streams"]))
        share = [0.35, 0.35] + [0.3 / len(side)] * len(side)
        kern = [_kernels(g, K, c["per_step"], period, EPOCH - 5 * MS, [0, 1] + side, share, 6 * US, 1.2),
                _kernels(g, _prefill_kernels(c, K), 3459, 200 * MS, EPOCH - 5 * MS, [2, 3] + side, share, 40 * US, 1.5)]
        for i in range(2):
            kern[i] = kern[i] + (torch.full_like(kern[i][3], i),)
    else:
        k = _kernels(g, K, c["per_step"], period, EPOCH - 5 * MS, list(range(c["streams"])), [1.0] * c["streams"],
                     6 * US, 1.2)
        kern = [k + (k[2] % c["threads"],)]
    start, end, stream, step, thread = (torch.cat([k[i] for k in kern]) for i in range(5))
    n = len(start)
    if _replays(c, p):  # one launch per step, before the step's first kernel
        n_l, _, _ = _counts(c, K, p)
        head = torch.full((n_l,), 1 << 62, dtype=torch.int64, device=DEV).scatter_reduce_(0, step, start, "amin")
        owner, l_thread, l_step = step, torch.arange(n_l, device=DEV) % c["threads"], torch.arange(n_l, device=DEV)
        node = torch.arange(n, device=DEV) % c["per_step"]
    else:
        n_l, head = n, start
        owner, l_thread, l_step = torch.arange(n, device=DEV), thread, step
        node = torch.full((n,), -1, dtype=torch.int64, device=DEV)
    lat = torch.empty(n_l, dtype=torch.float64, device=DEV).exponential_(1 / (5 * US), generator=g).round().long()
    l_ts = head - lat
    l_te = l_ts + torch.randint(1000, 4001, (n_l,), device=DEV, generator=g)
    by_time = torch.sort(l_ts, stable=True).indices
    corr = torch.empty(n_l, dtype=torch.int64, device=DEV)
    corr[by_time] = (p << 40) + 1000 * p + 17 + torch.cumsum(torch.randint(1, 4, (n_l,), device=DEV, generator=g), 0)
    if c["ids"] == "sparse":  # a driver's opaque 64-bit ids
        corr = corr * -7046029254386353131
    o = by_time[torch.sort(l_thread[by_time], stable=True).indices]
    o_ts, o_te, o_thr = _ops(g, l_ts[o], l_thread[o], l_step[o], n_l)
    keep = torch.randperm(n, device=DEV, generator=g)[int(n * DROP):].sort().values
    zero = torch.zeros(len(o_ts), dtype=torch.int64, device=DEV)
    none = lambda t: torch.full_like(t, -1)  # noqa: E731
    api = (torch.rand(n_l, device=DEV, generator=g) < 0.05).long()
    kname = _zipf(g, c["names"], n)
    return [(o_ts + offset, o_te + offset, zero, o_thr, _zipf(g, c["op_names"], len(o_ts)), none(o_ts)),
            (l_ts + offset, l_te + offset, corr, l_thread, api, none(l_ts)),
            (start[keep] + offset, end[keep] + offset, corr[owner[keep]], stream[keep], kname[keep], node[keep])]


def _trace(c, K, seed):
    """(columns on the GPU, params) of one window."""
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1_000_003 + K) & ((1 << 62) - 1))
    P = c["procs"]
    offs = torch.randint(-50 * US, 50 * US + 1, (P,), device=DEV, generator=g).tolist() if P > 1 else [0]
    parts, group = [], []
    for p in range(P):
        for kind, part in enumerate(_process(g, c, K, p, offs[p])):
            parts.append(part)
            group.append(torch.full((len(part[0]),), 3 * p + kind, dtype=torch.int64, device=DEV))
    ts, te, corr, lane, name, node = (torch.cat([q[i] for q in parts]) for i in range(6))
    group = torch.cat(group)
    n = len(ts)
    if c["order"] == "shuffled":
        order = torch.randperm(n, device=DEV, generator=g)
    else:  # per (process, kind) by end time, in blocks ordered by their last end
        order = torch.sort(te, stable=True).indices
        order = order[torch.sort(group[order], stable=True).indices]
        gs = group[order]
        head = torch.ones(n, dtype=torch.bool, device=DEV)
        head[1:] = gs[1:] != gs[:-1]
        at = torch.arange(n, device=DEV)
        pos = at - torch.cummax(torch.where(head, at, torch.zeros_like(at)), 0).values
        blk = torch.cumsum((head | (pos % BLOCK == 0)).long(), 0) - 1
        final = torch.empty(int(blk[-1]) + 1, dtype=torch.int64, device=DEV)
        edge = torch.ones(n, dtype=torch.bool, device=DEV)
        edge[:-1] = blk[1:] != blk[:-1]
        final[blk[edge]] = te[order][edge]
        rank = torch.empty_like(final)
        rank[torch.sort(final, stable=True).indices] = torch.arange(len(final), device=DEV)
        order = order[torch.sort(rank[blk], stable=True).indices]
    i32 = lambda t: t[order].to(torch.int32).contiguous()  # noqa: E731
    cols = dict(ts=ts[order].contiguous(), te=te[order].contiguous(), corr=corr[order].contiguous(),
                pid=i32(group // 3), lane=i32(lane), name=i32(name), kind=(group[order] % 3).to(torch.uint8).contiguous())
    params = dict(window_begin=EPOCH, window_end=EPOCH + _window(c, K), gap_threshold=c["threshold_us"] * US,
                  n_procs=P, n_streams=c["streams"], n_threads=c["threads"], n_names=c["names"],
                  n_op_names=c["op_names"], clock_offset=np.array(offs, np.int64) if P > 1 else None,
                  stream_class=np.array([0, 0, 0, 0, 1, 1, 2, 2], np.uint8) if c["mixed"] else None,
                  edges=None, flags=c["flags"])
    if c["edges"]:  # a random kernel's end, and a kernel of another process
        E = c["edges"]
        k = torch.nonzero(cols["kind"] == KERNEL).flatten()
        a, b = (k[torch.randint(0, len(k), (E,), device=DEV, generator=g)] for _ in range(2))
        e = np.zeros(E, EDGE_DTYPE)
        for f, x in (("prod_pid", cols["pid"][a]), ("cons_pid", cols["pid"][b]), ("prod_corr", cols["corr"][a]),
                     ("cons_corr", cols["corr"][b])):
            e[f] = x.cpu().numpy()
        params["edges"] = e
    if c["flags"] & SOL:  # 2 GFLOP and 0.5 GB an op in the median; 2.5 PFLOP/s and 8 TB/s
        op = cols["kind"] == CPU_OP
        for f, med in (("flops", 2e9), ("bytes", 5e8)):
            v = torch.empty(n, dtype=torch.float64, device=DEV).log_normal_(math.log(med), 1.5, generator=g)
            cols[f] = torch.where(op, v.round().long(), torch.zeros_like(ts))
        params.update(peak_flops=2_500_000_000_000_000, peak_bytes=8_000_000_000_000,
                      ref_sol_ppm=torch.randint(0, 400_000, (c["op_names"],), device=DEV, generator=g).cpu().numpy())
    if c["flags"] & GRAPH:
        cols["graph_node"] = i32(node)
        params["n_graph_nodes"] = max(1, c["nodes"])
    return cols, params


def _lengths(c) -> list:
    """Kernels of each window of the case: spread between smallest and kernels."""
    T = c["traces"]
    if T == 1:
        return [c["kernels"]]
    lo, hi = min(c["smallest"], c["kernels"]), c["kernels"]
    return [int(lo + (hi - lo) * ((0.5 + 0.618034 * t) % 1.0)) for t in range(T - 1)] + [hi]


# --------------------------------------------------------------- the outputs
ALWAYS = ("busy", "idle", "name_count", "name_sum", "name_min", "name_max", "lat_hist", "gap_pid", "gap_stream",
          "gap_begin", "gap_end", "gap_flags", "counters", "opname_count", "opname_sum", "opname_min", "opname_max")
BY_FLAG = {CONTAIN: ("op_nkern", "op_first", "op_last", "op_ksum"),
           OVERLAP: ("pair_overlap", "class_busy", "class_overlap", "any_busy"),
           WAITS: ("dev_idle", "op_span", "op_idle"),
           SOL: ("op_mfu", "op_mbu", "op_sol", "opn_flops", "opn_bytes", "opn_time", "opn_sol", "opn_hot"),
           CRIT: ("crit_time", "crit_flags", "crit_proc"),
           GRAPH: ("launch_first", "launch_last", "gn_count", "gn_sum", "gn_min", "gn_max", "gn_offset")}
AGGREGATES = ALWAYS  # what a batch asks for


def _wanted(c) -> list:
    if c["entry"] in ("batch", "chunked"):
        return list(AGGREGATES)
    w = list(ALWAYS) + ["link", "aux"] + (["edge_wait", "edge_status"] if c["edges"] else [])
    for f, names in BY_FLAG.items():
        if c["flags"] & f:
            w += names
    return w


def _analyzer(params, n, workspace):
    an = H.Analyzer(params, n, workspace=workspace)
    for v in an.o.values():  # what a call leaves alone reads the same in every run
        v.fill_(3)
    return an


def prepare(case: dict, seed: int) -> dict:
    c = _full(case)
    made = [_trace(c, K, seed + 7919 * t) for t, K in enumerate(_lengths(c))]
    ns = [len(m[0]["ts"]) for m in made]
    st = dict(entry=c["entry"], wanted=_wanted(c), n=ns[0])
    if c["entry"] in ("analyze", "static"):
        cols, params = made[0]
        st.update(an=_analyzer(params, ns[0], workspace=c["entry"] == "analyze"), cols=cols, ev=H.events_struct(cols))
        return st
    ans = [H.Analyzer(m[1], 1, workspace=False) for m in made]  # their parameters; the outputs are below
    ws = torch.empty(max(H.herschel_workspace_size(n, a.params) for a, n in zip(ans, ns)), dtype=torch.uint8, device=DEV)
    plist = [ans[0]._params_struct(ws.data_ptr(), ws.numel())] + [a.params for a in ans[1:]]
    # every window's part of one tensor per output, each part on a 256-byte line
    P, NS = c["procs"], c["streams"]
    size = dict(busy=P * NS, idle=P * NS, lat_hist=64, counters=len(H.COUNTERS))
    size.update({"name_" + k: c["names"] for k in ("count", "sum", "min", "max")})
    size.update({"opname_" + k: c["op_names"] for k in ("count", "sum", "min", "max")})
    line = lambda x: (x + 255) // 256 * 256  # noqa: E731
    at = {k: np.cumsum([0] + [line(size.get(k, n + P * NS)) for n in ns]) for k in AGGREGATES}
    o = {k: torch.full((int(at[k][-1]),), 3, dtype=ans[0].o[k].dtype, device=DEV) for k in AGGREGATES}
    outs = [H.HerschelOutputs(gap_capacity=n + P * NS,
                              **{k: o[k].data_ptr() + int(at[k][t]) * o[k].element_size() for k in AGGREGATES})
            for t, n in enumerate(ns)]
    offs = np.cumsum([0] + ns).astype(np.int64)
    cols = {k: torch.cat([m[0][k] for m in made]) for k in made[0][0]}
    st.update(ans=ans, ws=ws, plist=plist, outs=outs, offs=offs, o=o)
    if c["entry"] == "batch":
        st.update(cols=cols, ev=H.events_struct(cols))
        return st
    host = {k: v.cpu().pin_memory() for k, v in cols.items()}
    room = max(int(offs[min(t + c["chunk"], len(ns))] - offs[t]) for t in range(0, len(ns), c["chunk"]))
    staging = [{k: torch.empty(room, dtype=v.dtype, device=DEV) for k, v in host.items()} for _ in range(2)]
    st.update(host=host, hev=H.events_struct(host), room=room, chunk=c["chunk"], staging=staging,
              sev=[H.events_struct(s) for s in staging])
    return st


def run(state: dict):
    e = state["entry"]
    if e == "analyze":
        code = state["an"].run(state["ev"], state["n"])
    elif e == "static":
        an = state["an"]
        code = H.herschel_trace_analyze_static(state["ev"], state["n"], an.params, an.outs, an.lib)
    elif e == "batch":
        code = H.herschel_trace_analyze_batch(state["ev"], state["offs"], state["plist"], state["outs"])
    else:
        code = H.herschel_trace_analyze_chunked(state["hev"], state["offs"], state["chunk"], state["sev"],
                                                state["room"], state["plist"], state["outs"])
    if code != H.OK:
        raise RuntimeError(H.herschel_strerror(code))
    if "an" in state:
        return {k: state["an"].o[k] for k in state["wanted"]}
    return state["o"]


def work(case: dict) -> dict:
    """Every input column once and every wanted output once."""
    c = _full(case)
    total = 0
    f, P, NS = c["flags"], c["procs"], c["streams"]
    for K in _lengths(c):
        L, k, ops = (sum(_counts(c, K, p)[i] for p in range(P)) for i in range(3))
        n = L + k + ops
        total += 37 * n + 16 * P * NS + 32 * c["names"] + 32 * c["op_names"] + 512 + 112 + 36 * c["edges"]
        total += 25 * P * K // 50  # gaps above the threshold, about one kernel in fifty
        if c["entry"] in ("analyze", "static"):
            total += 8 * n  # link, aux
        if f & CONTAIN:
            total += 28 * ops
        if f & OVERLAP:
            total += 8 * P * (NS * NS + 13)
        if f & WAITS:
            total += 16 * P * c["op_names"] + 8 * P
        if f & SOL:
            total += 16 * n + 24 * ops + 48 * c["op_names"]
        if f & CRIT:
            total += 9 * n + 64 * P
        if f & GRAPH:
            total += 4 * n + 16 * L + 40 * max(1, c["nodes"])
    return {"bytes": int(total), "flops": 0}


def tolerance(case: dict):
    return "exact"  # integer nanoseconds, counts and row indices


# ----------------------------------------------------- the same in plain torch
def _plain(c, cols, p) -> dict:
    """Busy and idle time, per-name tables and latencies of one window, in
    64-bit integers by sorting and scanning."""
    off = torch.zeros(c["procs"], dtype=torch.int64, device=DEV)
    if p["clock_offset"] is not None:
        off = torch.from_numpy(p["clock_offset"]).to(DEV)
    W0, W1 = p["window_begin"], p["window_end"]
    pid, kind, lane, name = (cols[k].long() for k in ("pid", "kind", "lane", "name"))
    ts, te = cols["ts"] - off[pid], cols["te"] - off[pid]
    adm = (ts >= W0) & (ts < W1)
    out = {}
    for pre, which, count in (("name", KERNEL, c["names"]), ("opname", CPU_OP, c["op_names"])):
        m = adm & (kind == which)
        q, d = name[m], (te - ts)[m]
        z = torch.zeros(count, dtype=torch.int64, device=DEV)
        out[pre + "_count"] = z.scatter_add(0, q, torch.ones_like(d))
        out[pre + "_sum"] = z.scatter_add(0, q, d)
        big = torch.iinfo(torch.int64)
        out[pre + "_min"] = torch.full_like(z, big.max).scatter_reduce(0, q, d, "amin")
        out[pre + "_max"] = torch.full_like(z, big.min).scatter_reduce(0, q, d, "amax")
    m = adm & (kind == KERNEL)
    W, NS = W1 - W0, c["streams"]
    seg, s, e = (pid * NS + lane)[m], ts[m] - W0, te[m].clamp(max=W1) - W0
    o = torch.sort(seg * (W + 1) + s, stable=True).indices
    seg, s, e = seg[o], s[o], e[o]
    reach = torch.cummax(seg * (W + 1) + e, 0).values - seg * (W + 1)  # 0 or more inside a segment
    prev = torch.zeros_like(reach)
    prev[1:] = torch.where(seg[1:] == seg[:-1], reach[:-1], torch.zeros_like(reach[:-1]))
    busy = torch.zeros(c["procs"] * NS, dtype=torch.int64, device=DEV)
    busy = busy.scatter_add(0, seg, (e - torch.maximum(s, prev)).clamp(min=0))
    out["busy"], out["idle"] = busy, W - busy
    # latencies: each kernel and its launch (ids are unique among launches)
    l, k = adm & (kind == LAUNCH), adm & (kind == KERNEL)
    key = cols["corr"] if c["ids"] != "sparse" else cols["corr"] * -1018231460777725123  # back to ids (p << 40) + i
    lk, lo = torch.sort(key[l])
    lt = ts[l][lo]
    if not len(lk):  # no launch admitted
        lk, lt = key.new_tensor([-1]), ts.new_zeros(1)
    at = torch.searchsorted(lk, key[k]).clamp(max=len(lk) - 1)
    hit = lk[at] == key[k]
    x = (ts[k] - lt[at])[hit]
    bins = torch.zeros_like(x)
    for b in range(62):
        bins += (x >= (1 << b)).long()
    out["lat_hist"] = torch.bincount(bins, minlength=64)
    return out


def exact(case: dict, seed: int):
    c = _full(case)
    got = [_plain(c, *_trace(c, K, seed + 7919 * t)) for t, K in enumerate(_lengths(c))]
    if c["entry"] in ("analyze", "static"):
        return {k: got[0].get(k) for k in _wanted(c)}
    full = {}
    for k in AGGREGATES:  # laid out as prepare() does, None where there is no such value
        if k not in got[0]:
            full[k] = None
            continue
        size = (len(got[0][k]) + 255) // 256 * 256
        full[k] = torch.full((size * len(got),), 3, dtype=torch.int64, device=DEV)
        for t, v in enumerate(got):
            full[k][size * t:size * t + len(v[k])] = v[k]
    return full
