"""GPU parity of the team kernel on its own (one workgroup per simulation, one
thread per SM): random graphs the windowed kernels accept, named workloads
and batches at the edges of its lists, shown to have run on it, bit-exact
against the oracle; and the hand-back of a simulation that overflows them."""
import numpy as np
import pytest

from paper_2607_11262_amd import api
from paper_2607_11262_amd.gen import hw as H
from paper_2607_11262_amd.gen import workloads as W
from paper_2607_11262_amd.gen.rng import SplitMix64
from test_gpu_windowed import (ALL, STATS_BYTES, STATUS_RETRY, _simultaneous_loads_graph, _wide_roots_graph, compare,
                               note)
from windowed import window_eligible, windowed_graph, windowed_machines

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def run_counted(torch, g, hws, flags, monkeypatch, kernel="team"):
    """One launch with GTS_KERNEL=kernel (None: the normal path); returns the
    outputs and every simulation's counter block."""
    if kernel:
        monkeypatch.setenv("GTS_KERNEL", kernel)
    try:
        dg = api.upload(g)
        hs = api.upload_hw(hws)
        B = hws.shape[0]
        stride = api.scratch_bytes(dg, 2, flags) - api.scratch_bytes(dg, 1, flags)
        scratch = torch.zeros(api.scratch_bytes(dg, B, flags), dtype=torch.uint8, device="cuda")
        out = api.alloc_outputs(dg, B, flags)
        api.simulate_hwset_into(dg, hs, 0, B, flags, *out, scratch)
        torch.cuda.synchronize()
        blk = scratch[:B * stride].view(B, stride)[:, stride - STATS_BYTES:].contiguous().view(torch.int64).cpu().numpy()
    finally:
        if kernel:
            monkeypatch.delenv("GTS_KERNEL")
    cyc, mk, st, dg_ = out
    return (cyc.cpu().numpy().view(np.uint32) if cyc is not None else None, mk.cpu().numpy().view(np.uint32),
            st.cpu().numpy(), dg_.cpu().numpy().view(np.uint64) if dg_ is not None else None), blk


def run_team_only(torch, g, hws, flags, monkeypatch):
    """The outputs of the team kernel alone and, per simulation, the windows
    and the wavefronts its counter block reports."""
    gpu, blk = run_counted(torch, g, hws, flags, monkeypatch)
    return gpu, blk[:, 0], blk[:, 11]


def check(torch, g, hws, flags, monkeypatch, what):
    gpu, windows, waves = run_team_only(torch, g, hws, flags, monkeypatch)
    st = gpu[2]
    assert not np.any(st == STATUS_RETRY), f"{what}: handed back sims {np.flatnonzero(st == STATUS_RETRY)}"
    ran = st != api.SIM_INFEASIBLE
    assert np.all(windows[ran] > 0) and np.all(waves[ran] == -(-hws[ran, 0].astype(int) // 64)), what
    compare(g, hws, flags, gpu)
    return int(ran.sum())


@pytest.mark.parametrize("chunk", range(8))
def test_team_random_graphs(torch_cuda, chunk, monkeypatch):
    """200 random graphs (cross-CTA edges into shared nodes, fan-outs above
    three, zero-work nodes) on machines of 1-256 SMs under all four flag
    combinations."""
    ran = 0
    for seed in range(chunk * 25, chunk * 25 + 25):
        rng = SplitMix64(seed, 89)
        g = windowed_graph(rng)
        assert window_eligible(g)
        hws = windowed_machines(rng, rng.randint(1, 8))
        flags = ALL | rng.choice([0, api.NO_CONTENTION, api.ORDER_AT_FINISH, api.NO_CONTENTION | api.ORDER_AT_FINISH])
        note(f"team random seed={seed} N={g.n_nodes} E={g.n_edges} n_sm={hws[:, 0].tolist()} flags={flags}")
        ran += check(torch_cuda, g, hws, flags, monkeypatch, f"seed {seed}")
    assert ran > 0


@pytest.mark.parametrize("name", ["gemm_512", "gemm_perwarp", "fa", "fa_causal", "decode_small", "decoder_tiny",
                                  "simultaneous_loads"])
def test_team_workloads(torch_cuda, name, monkeypatch):
    """Each workload on machines whose SM counts sit at the edges of one to
    four waves (the last also with more arrivals, and retirements, in one
    cycle than a batch holds)."""
    g = {
        "gemm_512": lambda: W.gemm(512, 512, 512, 128, 128, 32, 2),
        "gemm_perwarp": lambda: W.gemm(2048, 1024, 512, 64, 64, 32, 3, per_warp=True),
        "fa": lambda: W.flash_attention(1, 4, 1024),
        "fa_causal": lambda: W.flash_attention(1, 4, 1024, 128, 128, 64, causal=True),
        "decode_small": lambda: W.splitkv_decode(batch=6, kv_min=64, kv_max=4096, seed=9),
        "decoder_tiny": lambda: W.decoder_layer(tokens=256, hidden=512, heads=8, kv_heads=2, ffn=1024, d=64),
        "simultaneous_loads": _simultaneous_loads_graph,
    }[name]()
    for sms in ((1, 3, 64), (65, 100, 128), (129, 132, 192), (193, 255, 256)):
        hws = np.stack([H.preset("H100", n_sm=s, max_cta_per_sm=c, tensor_permille=t)
                        for s in sms for c, t in ((32, 1000), (2, 2500))])
        note(f"team {name} N={g.n_nodes} n_sm={sms}")
        check(torch_cuda, g, hws, ALL, monkeypatch, f"{name} {sms}")


def test_team_short_lists(torch_cuda, monkeypatch):
    """A batch that fills every CU (each workgroup gets the shortest lists and
    rings): more arrivals of one SM, pending retirements and ready nodes than
    LDS holds, on kernels in LDS and in global memory."""
    for g in (W.splitkv_decode(batch=3, kv_min=64, kv_max=4096, seed=9), W.gemm(512, 512, 512, 64, 64, 32, 4)):
        hws = np.concatenate([np.stack([H.preset("H100", n_sm=s, max_cta_per_sm=c) for s, c in
                                        ((192, 32), (40, 32), (7, 8), (1, 32))]), H.sample_h100_sweep(45, 1020)])
        note(f"team short lists N={g.n_nodes} B={hws.shape[0]}")
        check(torch_cuda, g, hws, ALL, monkeypatch, g.name)


def test_team_subpartitions(torch_cuda, monkeypatch):
    """One server word per class, and (with a record of eight subpartitions in
    the batch) one per subpartition lane."""
    g = W.gemm(1024, 512, 512, 128, 128, 32, 3)
    hws = H.sample_h100_sweep(78, 9)
    hws[:, H.FIELDS["n_subpart"]] = [1, 2, 3, 4] * 2 + [4]
    check(torch_cuda, g, hws, ALL, monkeypatch, "one word")
    hws[4, H.FIELDS["n_subpart"]] = 8
    check(torch_cuda, g, hws, ALL, monkeypatch, "one per lane")


def test_team_hands_back_overflow(torch_cuda, monkeypatch):
    """300 loads ready at once on one SM of a 256-SM machine fit no list: the
    team kernel hands the simulation back, and the normal path finishes it."""
    g = _wide_roots_graph()
    hws = np.stack([H.preset("H100", n_sm=256, max_cta_per_sm=2), H.preset("H100", n_sm=1, max_cta_per_sm=2)])
    gpu, _, _ = run_team_only(torch_cuda, g, hws, ALL, monkeypatch)
    assert gpu[2][1] == STATUS_RETRY
    res = api.simulate(api.upload(g), hws, ALL)
    torch_cuda.cuda.synchronize()
    compare(g, hws, ALL, api.to_numpy(res))


@pytest.mark.parametrize("kind", ["tiles", "addresses"])
def test_team_forced_on_other_modes(torch_cuda, kind, monkeypatch):
    """GTS_KERNEL=team takes no graph whose loads go through the LRU L2 or are
    split into transactions: the team kernel has neither, so the normal path
    runs them and every cycle is the oracle's."""
    g = W.gemm(512, 512, 512, 128, 128, 32, 2, tiles=True) if kind == "tiles" else \
        W.gemm_addressed(512, 512, 512, 128, 128, 32, 2)
    hws = np.stack([H.preset("H100", n_sm=s, l2_lines=H.l2_lines(mib)) for s in (4, 132) for mib in (0.01, 0.25)])
    note(f"team forced on {kind} N={g.n_nodes}")
    monkeypatch.setenv("GTS_KERNEL", "team")
    res = api.simulate(api.upload(g), hws, ALL)
    torch_cuda.cuda.synchronize()
    compare(g, hws, ALL, api.to_numpy(res))


def _many_releases_into_one_cta(n_sources, per_source):
    """One kernel: source CTAs of loads, and a last CTA whose nodes each wait
    for one of those loads (and join in a store)."""
    from paper_2607_11262_amd.gen.graph import ALU, GLOAD, GSTORE, MISS, SYNC, GraphBuilder
    b = GraphBuilder()
    b.kernel(4, 0)
    loads = []
    for c in range(n_sources):
        b.cta()
        mine = [b.node(GLOAD, 512 + 64 * ((c + i) % 5), 0xF, MISS if i % 2 else 0) for i in range(per_source)]
        out = b.node(GSTORE, 256, 0xF, MISS)
        for u in mine:
            b.edge(u, out)
        loads += mine
    b.cta()
    heads = [b.node(ALU, 256, 0xF) for _ in loads]
    join = b.node(SYNC, 0, 0xF)
    out = b.node(GSTORE, 256, 0xF)
    for u in heads:
        b.edge(u, join)
    b.edge(join, out)
    for u, v in zip(loads, heads):
        b.edge(u, v)
    return b.build("many_releases")


@pytest.mark.parametrize("sms", [70, 130, 200, 256])
def test_team_releases_past_the_lds_list(torch_cuda, sms, monkeypatch):
    """Loads of CTAs on all waves ready the nodes of one CTA: its SM's list
    runs past its part in LDS with entries that other waves write."""
    g = _many_releases_into_one_cta(sms - 1, 1)
    g2 = _many_releases_into_one_cta(16, 5)
    for gr in (g, g2):
        assert window_eligible(gr)
        # a fast memory: many loads finish in one window
        hws = np.stack([H.preset("H100", n_sm=sms, max_cta_per_sm=2, rate_l2=4096 << 16, rate_dram=4096 << 16,
                                 lat_l2=200 + 50 * i, lat_dram=200 + 90 * i) for i in range(4)])
        note(f"team releases n_sm={sms} N={gr.n_nodes}")
        gpu, _, _ = run_team_only(torch_cuda, gr, hws, ALL, monkeypatch)
        if gr is g2:
            check(torch_cuda, gr, hws, ALL, monkeypatch, f"releases {sms}")
        res = api.simulate(api.upload(gr), hws, ALL)  # the longer list is handed back where it does not fit
        torch_cuda.cuda.synchronize()
        compare(gr, hws, ALL, api.to_numpy(res))


def _fan_out(width, kind):
    """CTAs of one node after another, then `width` nodes that one event
    readies, on a CTA of its own per SM."""
    from paper_2607_11262_amd.gen.graph import ALU, DATA, GLOAD, GSTORE, MISS, ORDER, SYNC, GraphBuilder
    b = GraphBuilder()
    b.kernel(4, 0)
    for _ in range(4):
        b.cta()
        u = b.node(GLOAD, 256, 0xF, MISS)
        for _i in range(8):
            a, v = b.node(ALU, 64, 0xF), b.node(GLOAD, 256, 0xF)
            b.edge(u, a)
            b.edge(a, v)
            u = v
        if kind == "compute":
            v = b.node(ALU, 64, 0xF)
            b.edge(u, v)
            u = v
        mid = [b.node(GLOAD if kind == "loads" else ALU, 64 + i % 5, 0xF) for i in range(width)]
        join, out = b.node(SYNC, 0, 0xF), b.node(GSTORE, 256, 0xF)
        for m in mid:
            b.edge(u, m, ORDER if kind == "issue" else DATA)
            b.edge(m, join)
        b.edge(join, out)
        if kind == "issue":
            b.edge(u, out)
    return b.build("fan_out")


@pytest.mark.parametrize("kind", ["issue", "completion", "compute", "loads"])
def test_team_bursts(torch_cuda, kind, monkeypatch):
    """What the rule that leaves such graphs to the windowed kernel rests on:
    a burst past the lists (of loads: past the rings, 64 entries beside at most
    16 in LDS) is handed back by every simulation of the batch, one that fits
    by none."""
    for width, fits in ((60, True), (81 if kind == "loads" else 300, False)):
        g = _fan_out(width, kind)
        assert window_eligible(g)
        hws = np.stack([H.preset("H100", n_sm=s, max_cta_per_sm=1) for s in (132, 256, 44, 4)])
        gpu, _, _ = run_team_only(torch_cuda, g, hws, ALL, monkeypatch)
        assert np.all((gpu[2] == STATUS_RETRY) != fits), (width, gpu[2])
        res = api.simulate(api.upload(g), hws, ALL)
        torch_cuda.cuda.synchronize()
        compare(g, hws, ALL, api.to_numpy(res))


@pytest.mark.parametrize("width", [31, 32, 33, 38, 39, 40, 41, 100, 230])
def test_team_lists_in_scratch(torch_cuda, width, monkeypatch):
    """Ready lists on both sides of the end of their LDS part and of the eight
    entries read at a time behind it, with the longest (4 simulations) and the
    shortest LDS parts (2048)."""
    for kind in ("issue", "compute"):
        g = _fan_out(width, kind)
        for B in (4, 2048):
            hws = np.stack([H.preset("H100", n_sm=s, max_cta_per_sm=1) for s in (64, 1, 40, 3)] * (B // 4))
            hws[:, H.FIELDS["rate_alu"]] += np.arange(B, dtype=np.uint32) % 61 << 12
            check(torch_cuda, g, hws, api.OUT_DIGEST, monkeypatch, f"width {width} {kind} B {B}")


def _late_diamonds(levels):
    """A kernel that ends at cycle ~0xF0000000, then a templated one whose root
    finishes past the last cycle, followed by levels of four nodes joined by
    one.  The root's finish wraps to 0x08000000, below the window's end."""
    from paper_2607_11262_amd.gen.graph import GLOAD, GSTORE, SYNC, TENSOR, GraphBuilder
    b = GraphBuilder()
    b.kernel(4, 0)
    b.cta()
    u = b.node(GLOAD, 64, 0xF)
    for cls, work in ((SYNC, 0), (SYNC, 0), (SYNC, 0), (TENSOR, 0x3000), (GSTORE, 64)):
        v = b.node(cls, work, 0xF)
        b.edge(u, v)
        u = v
    b.kernel(4, 0)
    for _ in range(2):
        b.cta()
        x = b.node(TENSOR, 0x1800, 0xF)
        for _l in range(levels):
            y = [b.node(TENSOR, 0, 0xF) for _ in range(4)]
            j = b.node(TENSOR, 0, 0xF)
            for v in y:
                b.edge(x, v)
                b.edge(v, j)
            x = j
        out = b.node(GSTORE, 64, 0xF)
        b.edge(x, out)
    return b.build("late_diamonds")


def test_team_gives_up_past_the_last_cycle(torch_cuda, monkeypatch):
    """A simulation that passes the last cycle in a kernel run from LDS ends
    there: its cycles stay past the end.  (Were they to wrap, each level of
    joins could become ready twice as often as the one before.)"""
    g = _late_diamonds(40)
    assert window_eligible(g) and api.templates(g)["templated_kernels"] == 1
    hws = np.stack([H.toy(n_sm=s, n_subpart=1, rate_tensor=1, lat_tensor=0, lat_sync=1 << 30, max_cta_per_sm=2)
                    for s in (1, 2, 65)])
    gpu, _, _ = run_team_only(torch_cuda, g, hws, ALL, monkeypatch)
    assert np.all(gpu[2] == STATUS_RETRY)
    res = api.simulate(api.upload(g), hws, ALL)
    torch_cuda.cuda.synchronize()
    compare(g, hws, ALL, api.to_numpy(res))
    assert np.all(res.status.cpu().numpy() == api.SIM_OVERFLOW)
