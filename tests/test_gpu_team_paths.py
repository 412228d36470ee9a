"""GPU parity of the team kernel's rarer paths, each shown to have run by the
counts of its counter block: kernels run from LDS on random graphs, switches
between kernels in LDS and in global memory, batches served in doubles or
ordered by 64-bit keys, and the hand-backs of a kernel longer than 2^27
cycles and of a list that overflows bit by bit."""
import numpy as np
import pytest

import oracle
from paper_2607_11262_amd import api
from paper_2607_11262_amd.gen import hw as H
from paper_2607_11262_amd.gen import workloads as W
from paper_2607_11262_amd.gen.graph import ALU, GLOAD, GSTORE, MISS, SYNC, GraphBuilder
from paper_2607_11262_amd.gen.rng import SplitMix64
from single_sink import single_sink_graph
from test_gpu_team import run_counted, torch_cuda  # noqa: F401 (fixture)
from test_gpu_windowed import ALL, STATUS_RETRY, compare, note
from windowed import window_eligible, windowed_machines

pytestmark = pytest.mark.gpu

IN_LDS, IN_DOUBLES, BY_64_BITS = 13, 14, 15  # words of the counter block


def on_team(torch, g, hws, flags, monkeypatch, what, may_overflow=False):
    """Every simulation ran on the team kernel to the end, exactly (or, if it
    may, outgrew its lists: many CTAs on a few SMs of a batch of larger
    machines); returns the blocks of those that ran and which they are."""
    gpu, blk = run_counted(torch, g, hws, flags, monkeypatch)
    back = gpu[2] == STATUS_RETRY
    assert may_overflow or not back.any(), f"{what}: handed back sims {np.flatnonzero(back)}"
    compare(g, hws[~back], flags, tuple(a[~back] if a is not None else None for a in gpu))
    ran = ~back & (gpu[2] != api.SIM_INFEASIBLE)
    return blk[ran], ran


@pytest.mark.parametrize("chunk", range(8))
def test_random_kernels_in_lds(torch_cuda, chunk, monkeypatch):
    """Random single-sink kernels (in-degrees to 31, up to eight successors,
    SYNC and SMEM nodes, ORDER beside DATA edges, several op classes), every
    fourth graph among ragged ones that run from global memory, with and
    without contention."""
    in_lds = kernels = sims = finished = 0
    for seed in range(chunk * 25, chunk * 25 + 25):
        rng = SplitMix64(seed, 61)
        g, sinks = single_sink_graph(rng, mixed=0.5 if seed % 4 == 0 else 0.0)
        assert window_eligible(g)
        hws = windowed_machines(rng, rng.randint(1, 8))
        flags = ALL | rng.choice([0, 0, api.NO_CONTENTION])
        note(f"team LDS seed={seed} N={g.n_nodes} E={g.n_edges} n_sm={hws[:, 0].tolist()} flags={flags}")
        blk, ran = on_team(torch_cuda, g, hws, flags, monkeypatch, f"seed {seed}",
                           may_overflow=True)
        narrow = hws[ran][:, H.FIELDS["n_subpart"]] <= 4  # eight lanes may need a word each
        assert np.all(blk[:, IN_LDS] <= sinks)
        in_lds += int(blk[narrow, IN_LDS].sum())
        kernels += sinks * int(narrow.sum())
        sims += hws.shape[0]
        finished += int(ran.sum())
    note(f"team LDS chunk={chunk}: {in_lds} of {kernels} kernels from LDS, {finished} of {sims} simulations")
    assert in_lds > kernels // 2 and finished > sims // 2


def test_order_at_finish_runs_from_global_memory(torch_cuda, monkeypatch):
    """ORDER edges released at the finish are not in the compact records."""
    rng = SplitMix64(3, 62)
    g, sinks = single_sink_graph(rng)
    hws = windowed_machines(rng, 6)
    blk, _ = on_team(torch_cuda, g, hws, ALL | api.ORDER_AT_FINISH, monkeypatch, "order at finish", may_overflow=True)
    assert sinks and len(blk) and np.all(blk[:, IN_LDS] == 0)


def test_kernels_switch_between_lds_and_global_memory(torch_cuda, monkeypatch):
    """LDS -> global -> LDS: a decoder layer's GEMMs around its causal
    attention, and random graphs with ragged kernels between."""
    g = W.decoder_layer(tokens=256, hidden=512, heads=8, kv_heads=2, ffn=1024, d=64)
    hws = np.stack([H.preset("H100", n_sm=s, max_cta_per_sm=4) for s in (2, 64, 132, 200)])
    blk, _ = on_team(torch_cuda, g, hws, ALL, monkeypatch, "decoder")
    assert np.all(blk[:, IN_LDS] > 1) and np.all(blk[:, IN_LDS] < len(g.kernel_warps))
    mixed = 0
    for seed in range(12):
        rng = SplitMix64(seed, 63)
        g, sinks = single_sink_graph(rng, n_kernels=(4, 4), mixed=0.5)
        blk, _ = on_team(torch_cuda, g, windowed_machines(rng, 4), ALL, monkeypatch, f"mixed seed {seed}",
                         may_overflow=True)
        mixed += int(np.sum((blk[:, IN_LDS] > 0) & (blk[:, IN_LDS] < len(g.kernel_warps))))
    assert mixed > 0


@pytest.mark.parametrize("in_lds", [True, False])
def test_slow_memory_is_served_in_doubles(torch_cuda, in_lds, monkeypatch):
    """Occupancies on both sides of 2^21 cycles, where a batch's sum no longer
    fits 32 bits, and a backlog past 2^29 cycles."""
    g = W.gemm(256, 256, 128, 128, 128, 32, 2) if in_lds else W.splitkv_decode(batch=2, kv_min=64, kv_max=512, seed=9)
    hws = []
    for rate in (1 << 16, 1 << 10, 300, 256, 255, 100, 40):  # Q16 bytes per cycle
        r = H.preset("H100", n_sm=70, max_cta_per_sm=2)
        r[H.FIELDS["rate_l2"]] = rate * 4
        r[H.FIELDS["rate_dram"]] = rate
        hws.append(r)
    hws = np.stack(hws)
    gpu, blk = run_counted(torch_cuda, g, hws, ALL, monkeypatch)
    note(f"slow memory in_lds={in_lds} status={gpu[2].tolist()} doubles={blk[:, IN_DOUBLES].tolist()}")
    done = gpu[2] != STATUS_RETRY  # kernels in LDS end before 2^27 cycles
    assert blk[0, IN_DOUBLES] == 0 and np.any(blk[done, IN_DOUBLES] > 0)
    if not in_lds:
        assert np.all(done)
    res = api.to_numpy(api.simulate(api.upload(g), hws, ALL))
    compare(g, hws, ALL, res)
    for b in np.flatnonzero(done):
        assert gpu[2][b] == res[2][b] and gpu[1][b] == res[1][b] and gpu[3][b] == res[3][b]
        assert res[2][b] != api.SIM_OK or np.array_equal(gpu[0][b], res[0][b])


def test_long_kernel_is_handed_back(torch_cuda, monkeypatch):
    """A kernel in LDS counts its slots' cycles in 27 bits: the records that
    make it longer are handed back, the others not, and the windowed kernel
    finishes them."""
    g = W.gemm(512, 512, 512, 128, 128, 32, 2)
    hws = np.stack([H.preset("H100", n_sm=8, max_cta_per_sm=1) for _ in range(6)])
    hws[:, H.FIELDS["rate_tensor"]] = [1 << 16, 16420, 16395, 16384, 16350, 1 << 10]
    flags = ALL
    omk = oracle.simulate_batch(g, hws, flags, want_nodes=False, threads=4)[0].astype(np.int64)
    gpu, blk = run_counted(torch_cuda, g, hws, flags, monkeypatch)
    note(f"long kernel makespans={omk.tolist()} status={gpu[2].tolist()}")
    back = gpu[2] == STATUS_RETRY
    assert np.array_equal(back, omk >= 1 << 27) and back.any() and not back.all()
    assert np.all(blk[:, IN_LDS] == 1)
    alone, wblk = run_counted(torch_cuda, g, hws, flags, monkeypatch, kernel="window")
    assert not np.any(alone[2] == STATUS_RETRY)
    gpu, blk = run_counted(torch_cuda, g, hws, flags, monkeypatch, kernel=None)
    assert np.array_equal(blk[back, :6], wblk[back, :6])  # the windowed kernel's counts
    compare(g, hws, flags, gpu)


def test_list_that_overflows_bit_by_bit(torch_cuda, monkeypatch):
    """No single event readies more than 12 nodes, but 144 are ready at once
    on one SM: handed back, and finished by the windowed kernel."""
    b = GraphBuilder()
    b.kernel(4, 0)
    for _ in range(3):
        b.cta()
        root, join, out = b.node(GLOAD, 256, 0xF, MISS), b.node(SYNC, 0, 0xF), None
        for i in range(12):
            u = b.node(GLOAD, 256, 0xF)
            b.edge(root, u)
            for _j in range(12):
                v = b.node(ALU, 1 << 14, 0xF)
                b.edge(u, v)
                b.edge(v, join)
        out = b.node(GSTORE, 256, 0xF)
        b.edge(join, out)
    g = b.build("grows")
    assert window_eligible(g)
    hws = np.stack([H.preset("H100", n_sm=s, max_cta_per_sm=1) for s in (256, 200, 64)])
    gpu, _ = run_counted(torch_cuda, g, hws, ALL, monkeypatch)
    assert np.all(gpu[2] == STATUS_RETRY)
    alone, wblk = run_counted(torch_cuda, g, hws, ALL, monkeypatch, kernel="window")
    assert not np.any(alone[2] == STATUS_RETRY)
    gpu, blk = run_counted(torch_cuda, g, hws, ALL, monkeypatch, kernel=None)
    assert np.array_equal(blk[:, :6], wblk[:, :6])
    compare(g, hws, ALL, gpu)


def test_wide_ids_are_ordered_by_64_bits(torch_cuda, monkeypatch):
    """65,792 CTAs of 34 nodes: CTA and node number need 23 bits, one more than
    the 32-bit order keys hold."""
    g = W.gemm(256 * 64, 257 * 64, 11 * 32, 64, 64, 32, 2)
    hws = np.stack([H.preset("H100", n_sm=s, max_cta_per_sm=2) for s in (132, 60)])
    blk, _ = on_team(torch_cuda, g, hws, api.OUT_DIGEST, monkeypatch, "wide ids")
    assert np.all(blk[:, IN_LDS] == 1) and np.all(blk[:, BY_64_BITS] > 0)
    small = W.gemm(512, 512, 512, 128, 128, 32, 2)
    blk, _ = on_team(torch_cuda, small, hws, ALL, monkeypatch, "short ids")
    assert np.all(blk[:, BY_64_BITS] == 0)


def test_steps_of_all_waves_are_counted(torch_cuda, monkeypatch):
    """Three CTAs on SMs of three waves, one of them short: with one busy SM
    per wave every step issues one node."""
    b = GraphBuilder()
    b.kernel(4, 0)
    for n in (2, 30, 11):
        b.cta()
        u = b.node(GLOAD, 256, 0xF)
        for i in range(n):
            v = b.node(GLOAD if i % 3 == 0 else ALU, 256, 0xF)
            b.edge(u, v)
            u = v
        v = b.node(GSTORE, 256, 0xF)
        b.edge(u, v)
    g = b.build("three_chains")
    hws = np.stack([H.preset("H100", n_sm=132), H.preset("H100", n_sm=192)])
    blk, _ = on_team(torch_cuda, g, hws, ALL, monkeypatch, "three chains")
    assert np.all(blk[:, 2] == g.n_nodes) and np.all(blk[:, 1] == blk[:, 2])
