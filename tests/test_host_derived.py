"""What the host derives for the team kernel, on the CPU: compact template
records (what they decode to, the sharing of state slots under random event
orders, that only an upload builds them) and bursts of ready nodes."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2607_11262_amd import api
from paper_2607_11262_amd.gen import workloads as W
from paper_2607_11262_amd.gen.graph import ALU, DATA, GLOAD, GSTORE, ORDER, SYNC, GraphBuilder
from paper_2607_11262_amd.gen.rng import SplitMix64
from single_sink import single_sink_graph
from templated import templated_graph
from windowed import windowed_graph

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2607_11262_amd", "csrc")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("compact") / "compact.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                           "-I/opt/rocm/include", os.path.join(HERE, "host_derived.cpp"),
                           os.path.join(CSRC, "gts_host_only.cpp"), "-L/opt/rocm/lib", "-lamdhip64", "-o", out])
    L = ctypes.CDLL(out)
    L.gts_test_words_after_check.restype = L.gts_test_compact.restype = ctypes.c_int64
    L.gts_test_compact.argtypes = [ctypes.c_void_p] * 3 + [ctypes.c_uint64]
    return L


def compact(lib, g):
    """Per kernel {template nodes, state slots, records [nodes, 8] or None}."""
    h, _keep = api._host_struct(g)
    K = len(g.kernel_warps)
    ks = np.zeros((K, 3), np.uint32)
    rec = np.zeros((g.n_nodes + 1, 8), np.uint32)
    n = lib.gts_test_compact(ctypes.byref(h), ks.ctypes.data, rec.ctypes.data, rec.size)
    assert 0 <= n <= rec.size
    return [(int(t), int(s), rec[b:b + t].astype(np.int64) if s else None) for t, b, s in ks]


def local_edges(g, k):
    """[(u, v, kind)] of the kernel's first CTA, local numbering."""
    c0 = int(g.kernel_cta_begin[k])
    a, e = int(g.cta_node_begin[c0]), int(g.cta_node_begin[c0 + 1])
    out = []
    for u in range(a, e):
        for s in np.asarray(g.succ[int(g.succ_ptr[u]):int(g.succ_ptr[u + 1])], np.int64):
            out.append((u - a, int(s & 0x3FFFFFFF) - a, int(s >> 30)))
    return out


def decode(r):
    """The node's successors [(node, slot, in-degree, at issue)] released at
    issue (compute nodes: all of them) and at completion, and whether it is a
    load / store."""
    first, second, mem = int(r[2] >> 28), int(r[3] >> 29) & 7, bool((r[3] >> 28) & 1)
    w = [(int(x & 0xFFF), int((x >> 12) & 1023), int((x >> 22) & 31), bool((x >> 27) & 1)) for x in r]
    return w[:first], (w[4:4 + second] if mem else []), mem


def run_events(rec, slots, rng, indeg):
    """Random order of issues and completions through the shared slots; returns
    the order in which nodes became ready."""
    n = len(rec)
    st = [0] * slots
    ready = [v for v in range(n) if indeg[v] == 0]
    out, flying = list(ready), []
    nodes = [decode(r) for r in rec]

    def release(succ):
        sv = [st[s] for _, s, _, _ in succ]  # read together, as the kernel does
        for (v, s, need, _), cnt in zip(succ, sv):
            if cnt + 1 == need:
                st[s] = 0
                ready.append(v)
                out.append(v)
            else:
                st[s] = cnt + 1

    while ready or flying:
        pick = rng.randint(0, len(ready) + len(flying) - 1)
        if pick < len(ready):
            u = ready.pop(pick)
            now, later, mem = nodes[u]
            release(now)
            if mem:
                flying.append(u)
        else:
            release(nodes[flying.pop(pick - len(ready))][1])
    assert all(c == 0 for c in st[:-1])  # the last slot takes words without a successor
    return out


@pytest.mark.parametrize("chunk", range(4))
def test_shared_slots(lib, chunk):
    """Every node becomes ready once, after all its predecessors released it,
    in random orders of the events."""
    for seed in range(chunk * 40, chunk * 40 + 40):
        rng = SplitMix64(seed, 31)
        g, sinks = single_sink_graph(rng, mixed=0.2 if seed % 4 == 0 else 0.0)
        ks = compact(lib, g)
        assert sum(s > 0 for _, s, _ in ks) == sinks, f"seed {seed}"
        for k, (n, slots, rec) in enumerate(ks):
            if rec is None:
                continue
            edges = local_edges(g, k)
            indeg = [0] * n
            for _, v, _ in edges:
                indeg[v] += 1
            got = []
            for u in range(n):
                now, later, mem = decode(rec[u])
                for v, slot, need, issue in now + later:
                    assert need == indeg[v] and slot < slots - 1 and (need > 1) == (slot < slots - 2)
                    assert issue == ((v, slot, need, issue) in now if mem else issue)
                    got.append((u, v, ORDER if issue else DATA))
            assert sorted(got) == sorted((u, v, ORDER if kd == ORDER else DATA) for u, v, kd in edges)
            for _ in range(3):
                order = run_events(rec, slots, rng, indeg)
                assert sorted(order) == list(range(n)), f"seed {seed} kernel {k}"
                at = {v: i for i, v in enumerate(order)}
                assert all(at[u] < at[v] for u, v, _ in edges)


def _joins(n):
    """A kernel of two CTAs: n compute nodes of two in-edges that wait at once."""
    b = GraphBuilder()
    b.kernel(4, 0)
    for _ in range(2):
        b.cta()
        src = [b.node(GLOAD, 256, 0xF) for _ in range(n)]
        mid = [b.node(ALU, 256, 0xF) for _ in range(n)]
        for i in range(n):
            b.edge(src[i], mid[i])
            b.edge(src[(i + 1) % n], mid[i])
        level = mid
        while len(level) > 1:
            nxt = []
            for i in range(0, len(level), 31):
                j = b.node(SYNC, 0, 0xF)
                for u in level[i:i + 31]:
                    b.edge(u, j)
                nxt.append(j)
            level = nxt
        out = b.node(GSTORE, 256, 0xF)
        b.edge(level[0], out)
    return b.build("joins")


@pytest.mark.parametrize("n,waiting", [(2, 3), (900, 930), (988, 1022), (989, 1023), (1900, 1965)])
def test_slot_limit(lib, n, waiting):
    """1022 nodes that wait at once fit the slots (none of the joins follows
    all of another's predecessors); one more does not."""
    g = _joins(n)
    (t_n, slots, _), = compact(lib, g)
    indeg = np.bincount([v for _, v, _ in local_edges(g, 0)], minlength=t_n)
    assert t_n > 0 and int((indeg >= 2).sum()) == waiting
    assert slots == (waiting + 2 if waiting <= 1022 else 0)


def test_refused_templates(lib):
    """Templates with several sinks have no compact records; none at all
    without templates."""
    for seed in range(20):
        g = templated_graph(SplitMix64(seed, 7))
        for k, (n, slots, _) in enumerate(compact(lib, g)):
            if n:
                succ = {u for u, _, _ in local_edges(g, k)}
                assert not slots or len(set(range(n)) - succ) == 1


def test_queries_build_no_records(lib):
    """A size query and a validation leave the compact records out: their
    cost (ancestor sets of every node) is an upload's alone."""
    for g in (_joins(900), W.gemm(512, 512, 512, 128, 128, 32, 2), single_sink_graph(SplitMix64(1, 31))[0]):
        h, _keep = api._host_struct(g)
        assert lib.gts_test_words_after_check(ctypes.byref(h)) == 0
        assert any(s for _, s, _ in compact(lib, g))


def burst(g):
    """Nodes, and loads and stores in one cycle, that one event readies on one
    SM, at least, written out."""
    ptr, succ = np.asarray(g.succ_ptr, np.int64), np.asarray(g.succ, np.int64)
    tgt, order = succ & 0x3FFFFFFF, succ >> 30 == ORDER
    src = np.repeat(np.arange(g.n_nodes), np.diff(ptr))
    cta = np.repeat(np.arange(len(g.cta_node_begin) - 1), np.diff(np.asarray(g.cta_node_begin, np.int64)))
    indeg = np.bincount(tgt, minlength=g.n_nodes)
    mem = np.isin(np.asarray(g.op_cls)[np.asarray(g.node_op, np.int64)], (GLOAD, GSTORE))
    alone = (indeg[tgt] == 1) & (cta[src] == cta[tgt])
    event = 2 * src + (order & mem[src])  # a compute node's releases are one event ...
    cycle = 2 * src + order               # ... in two cycles
    most = lambda x: int(np.bincount(x).max()) if len(x) else 0  # noqa: E731
    return (max(most(cta[indeg == 0]), most(event[alone])),
            max(most(cta[(indeg == 0) & mem]), most(cycle[alone & mem[tgt]])))


def test_burst(lib):
    def of(g):
        h, _keep = api._host_struct(g)
        out = (ctypes.c_uint32 * 2)()
        assert lib.gts_test_burst(ctypes.byref(h), out) == 0
        return tuple(out)
    for seed in range(200):
        g = windowed_graph(SplitMix64(seed, 17), nodes=(1, 12 if seed % 2 else 40))
        assert of(g) == burst(g), f"seed {seed}"
    for seed in range(40):
        g, _ = single_sink_graph(SplitMix64(seed, 18))
        assert of(g) == burst(g), f"seed {seed}"
    assert of(_joins(300)) == (300, 300)  # its loads
    b = GraphBuilder()  # one event in two cycles: 9 + 3 loads, and 20 other nodes
    b.kernel(4, 0)
    b.cta()
    u = b.node(ALU, 256, 0xF)
    late = [b.node(GLOAD, 256, 0xF) for _ in range(12)]
    other = [b.node(ALU, 256, 0xF) for _ in range(20)]
    out = b.node(GSTORE, 256, 0xF)
    for i, v in enumerate(late + other):
        b.edge(u, v, ORDER if i < 5 or i % 2 else DATA)
        b.edge(v, out)
    assert of(b.build("two_cycles")) == (32, 9)
    # the pending node beside a full list of qp + 240 / waves entries; the rings
    for sms, share in ((1, 240), (64, 240), (65, 120), (132, 80), (256, 60)):
        assert not lib.gts_test_team_overflows(8 + share + 1, 68, 8, 4, sms)
        assert lib.gts_test_team_overflows(8 + share + 2, 0, 8, 4, sms)
        assert lib.gts_test_team_overflows(69, 69, 8, 4, sms)
