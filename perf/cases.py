"""The measured cases: batches of tile-graph simulations as programs run them.

A program builds a tile graph, uploads it, and simulates it under one or many
hardware records: alone (how long does this kernel take on this machine?), a
few machines, or a design sweep of thousands; with every node's (start,
finish) cycles, or with makespan / status / digest only.  The cases take the
graph families this package generates -- GEMM, flash attention, split-KV
decode, a decoder layer, the fused GEMM + SiLU organisations, cluster-fused
attention, and GEMMs whose tiles go through the LRU L2 by id or by address --
from a single small GEMM to sweeps of 1.6e9 simulated nodes, through the two
entry points: `api.simulate` (records from host memory, outputs and scratch
allocated per call) and `api.simulate_hwset_into` (records resident on the
GPU, outputs and scratch kept by the caller).

Everything computed is a whole number (cycles, status, a 64-bit digest), so
results are compared bit for bit.
"""
from __future__ import annotations

import numpy as np
import torch

from paper_2607_11262_amd import api
from paper_2607_11262_amd.gen import clusterfusion as CF
from paper_2607_11262_amd.gen import hw as H
from paper_2607_11262_amd.gen import pipelining as PL
from paper_2607_11262_amd.gen import workloads as W

NODES, DIGEST = api.OUT_NODES | api.OUT_DIGEST, api.OUT_DIGEST


def listed():
    return [
        # the smallest call: one small GEMM on one machine, records from the
        # host, every node's cycles back (784 nodes; launches and latency)
        dict(name="one_gemm_512", family="gemm", M=512, N=512, K=512, BM=128, BN=128, BK=32, S=2, per_warp=False,
             machines="a100", records=1, nodes=True, entry="simulate"),
        # one prefill attention on one machine: a single simulation's latency
        # (82,944 nodes on one wavefront)
        dict(name="one_flash_2048", family="flash", batch=1, heads=32, seqlen=2048, causal=False, machines="h100",
             records=1, nodes=True, entry="simulate"),
        # the 1024^3 GEMM of the A100 study: a handful of machines
        dict(name="gemm_1024_a100", family="gemm", M=1024, N=1024, K=1024, BM=128, BN=128, BK=32, S=2,
             per_warp=False, machines="a100", records=16, nodes=True, entry="hwset"),
        # design sweep, a small GEMM (24,832 nodes) under 4096 machines
        dict(name="sweep_gemm_25k", family="gemm", M=1024, N=2048, K=1024, BM=64, BN=128, BK=32, S=2,
             per_warp=False, machines="h100", records=4096, nodes=False, entry="hwset"),
        # design sweep, a large GEMM (401,408 nodes) under 4096 machines: the
        # most simulated nodes of all
        dict(name="sweep_gemm_401k", family="gemm", M=8192, N=8192, K=1024, BM=64, BN=128, BK=64, S=3,
             per_warp=False, machines="h100", records=4096, nodes=False, entry="hwset"),
        # prefill attention, 256 machines, per-node cycles for all of them
        dict(name="flash_prefill_256", family="flash", batch=2, heads=32, seqlen=4096, causal=False, machines="h100",
             records=256, nodes=True, entry="hwset"),
        # split-KV decode: many short ragged CTAs, cross-CTA reductions
        dict(name="splitkv_decode_1024", family="splitkv", batch=16, kv_max=32768, lens=1004, machines="h100",
             records=1024, nodes=True, entry="hwset"),
        # a decoder layer's nine kernels, 64 machines: the longest simulation
        dict(name="decoder_layer_64", family="decoder", tokens=256, machines="h100", records=64, nodes=True,
             entry="hwset"),
        # GEMM + SiLU organisations: a single SM, thousands of machines
        dict(name="gemm_silu_4096", family="silu", org="pingpong", BM=256, BN=128, BK=64, drop="full",
             machines="hopper1", records=4096, nodes=True, entry="simulate"),
        # cluster-fused attention over an SM-cluster network (one event at a
        # time: the general kernel)
        dict(name="cluster_attention_2048", family="cluster", cluster=4, comm="noc", machines="noc", records=2048,
             nodes=False, entry="hwset"),
        # a GEMM whose tiles go through an LRU L2 of 4-64 MiB
        dict(name="lru_gemm_2048", family="gemm_tiles", M=4096, N=2048, K=1024, BM=128, BN=64, BK=64, S=3,
             machines="h100_l2", records=2048, nodes=False, entry="hwset"),
        # a GEMM of addressed tiles: 128-B transactions under an LRU of lines
        dict(name="txn_gemm_1024", family="gemm_addr", M=1024, N=512, K=512, BM=128, BN=64, BK=32, S=3, layout="nk",
             pad=8, machines="h100_l2", records=1024, nodes=False, entry="hwset"),
    ]


def _log(rng, lo, hi):
    """A whole number, uniform over its logarithm."""
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


# per family: how often drawn, most simulated nodes of a pass, most nodes of
# a graph (a pass of few records lasts as long as one simulation)
_DRAWN = dict(gemm=(5, 6e8, 400_000), flash=(3, 2e8, 400_000), splitkv=(2, 1e8, 120_000), decoder=(1, 1.2e8, 2_600_000),
              silu=(1, 5e6, 4_000), cluster=(1, 4e7, 60_000), gemm_tiles=(2, 2e8, 120_000), gemm_addr=(1, 4e6, 8_000))


def _draw_graph(rng, family):
    if family in ("gemm", "gemm_tiles", "gemm_addr"):
        small = family == "gemm_addr"
        BM, BN = rng.choice((64, 128) if small else (64, 128, 256)), rng.choice((64, 128) if small else (64, 128, 256))
        BK = rng.choice((32, 64))
        # whole tiles in each dimension, any number of them (not powers of two)
        c = dict(M=BM * _log(rng, 1, 12 if small else 96), N=BN * _log(rng, 1, 12 if small else 96),
                 K=BK * _log(rng, 1, 20 if small else 160), BM=BM, BN=BN, BK=BK, S=rng.choice((2, 3, 4)))
        if family == "gemm":
            c["per_warp"] = rng.random() < 0.2
        if family == "gemm_addr":
            c.update(layout=rng.choice(("kn", "nk")), pad=rng.choice((0, 8)))
        return c
    if family == "flash":
        causal = rng.random() < 0.3
        return dict(batch=_log(rng, 1, 4), heads=_log(rng, 1, 32), seqlen=128 * _log(rng, 1, 32), causal=causal)
    if family == "splitkv":
        return dict(batch=_log(rng, 1, 20), kv_max=_log(rng, 1024, 32768), lens=rng.randrange(1 << 20))
    if family == "decoder":
        return dict(tokens=128 * rng.randint(1, 2))
    if family == "silu":
        BM, BN, BK = rng.choice(PL.TILES)
        return dict(org=rng.choice(PL.ORGANIZATIONS), BM=BM, BN=BN, BK=BK, drop=rng.choice(sorted(PL.ABLATIONS)))
    return dict(cluster=rng.choice(CF.CLUSTER_SIZES), comm=rng.choice(CF.COMMS))


def _nodes(c):
    """Nodes of a drawn case's graph, closely enough to bound its cost."""
    f = c["family"]
    if f.startswith("gemm"):
        per_step = 6 if c.get("per_warp") else 3
        return (c["M"] // c["BM"]) * (c["N"] // c["BN"]) * (per_step * (c["K"] // c["BK"]) + 1)
    if f == "flash":
        n = c["batch"] * c["heads"] * (c["seqlen"] // 128) * (5 * (c["seqlen"] // 64) + 2)
        return n * 0.6 if c["causal"] else n
    if f == "splitkv":
        return c["batch"] * 8 * 24 * (1 + c["kv_max"] // 1024)
    if f == "decoder":
        return 10_000 * c["tokens"]
    return 3_000 if f == "silu" else 3_700 * c["cluster"]


def draw(rng):
    while True:
        family = rng.choice([f for f, (weight, _, _) in _DRAWN.items() for _ in range(weight)])
        _, most_sims, most_nodes = _DRAWN[family]
        c = dict(family=family, **_draw_graph(rng, family))
        n = _nodes(c)
        if n > most_nodes:
            continue
        top = int(min(4096, most_sims // n))
        if family == "decoder":
            top = min(top, 64)
        if top < 1:
            continue
        c["records"] = _log(rng, 1, top)
        c["machines"] = dict(silu="hopper1", cluster="noc", gemm_tiles="h100_l2", gemm_addr="h100_l2").get(
            family, "a100" if family == "gemm" and rng.random() < 0.25 else "h100")
        c["nodes"] = n * c["records"] <= 2e8 and rng.random() < 0.5
        # infeasible machines leave rows of api.simulate's fresh per-node
        # output unwritten: it is drawn where every machine fits the kernels
        c["entry"] = "simulate" if (not c["nodes"] or c["machines"] in ("hopper1", "noc")) and rng.random() < 0.4 else "hwset"
        return c


def _graph(c):
    f = c["family"]
    if f == "gemm":
        return W.gemm(c["M"], c["N"], c["K"], c["BM"], c["BN"], c["BK"], c["S"], per_warp=c["per_warp"])
    if f == "gemm_tiles":
        return W.gemm(c["M"], c["N"], c["K"], c["BM"], c["BN"], c["BK"], c["S"], tiles=True)
    if f == "gemm_addr":
        return W.gemm_addressed(c["M"], c["N"], c["K"], c["BM"], c["BN"], c["BK"], c["S"], pad=c["pad"],
                                b_layout=c["layout"])
    if f == "flash":
        return W.flash_attention(c["batch"], c["heads"], c["seqlen"], causal=c["causal"])
    if f == "splitkv":
        return W.splitkv_decode(c["batch"], kv_max=c["kv_max"], seed=c["lens"])
    if f == "decoder":
        return W.decoder_layer(c["tokens"])
    if f == "silu":
        return PL.gemm_silu(c["org"], c["BM"], c["BN"], c["BK"], drop=PL.ABLATIONS[c["drop"]])
    return CF.cluster_attention(c["cluster"], comm=c["comm"])


def _machines(kind, seed, B):
    if kind == "a100":
        return H.sample_a100_sweep(seed, B)
    if kind == "noc":
        return CF.sample_noc_machines(seed, B)
    if kind == "hopper1":
        return PL.sample_hopper_1sm(seed, B)
    hw = H.sample_h100_sweep(seed, B)
    if kind == "h100_l2":  # an LRU L2 of 4-64 MiB, in 128-B lines
        hw[:, 26] = (np.random.default_rng(seed).integers(4, 65, size=B) * (1 << 20)) // 128
    return hw


def prepare(case, seed):
    g, hw = _graph(case), _machines(case["machines"], seed, case["records"])
    if case["records"] == 1 and case["machines"] == "h100":
        # a single machine is a product's (132 SMs, 228 KiB), its rates sampled
        hw[:, 0], hw[:, 4] = H.preset("H100")[0], H.preset("H100")[4]
    flags = NODES if case["nodes"] else DIGEST
    dg = api.upload(g)
    if case["entry"] == "simulate":
        return dict(graph=dg, hw=hw, flags=flags)
    B = hw.shape[0]
    # cleared once: an infeasible machine leaves its row of cycles unwritten
    outs = [t.zero_() if t is not None else None for t in api.alloc_outputs(dg, B, flags)]
    scratch = torch.empty(max(api.scratch_bytes(dg, B, flags), 1), dtype=torch.uint8, device="cuda")
    return dict(graph=dg, hwset=api.upload_hw(hw), B=B, flags=flags, outs=outs, scratch=scratch)


def run(state):
    g, flags = state["graph"], state["flags"]
    if "hw" in state:
        r = api.simulate(g, state["hw"], flags)
        outs = (r.cycles, r.makespan, r.status, r.digest)
    else:
        outs = state["outs"]
        api.simulate_hwset_into(g, state["hwset"], 0, state["B"], flags, *outs, state["scratch"])
    return {k: v for k, v in zip(("cycles", "makespan", "status", "digest"), outs) if v is not None}


def work(case):
    """What a pass cannot do without: the graph (op 2 B, warps 2 B, successor
    offset 4 B and in-degree 2 B per node, 4 B per edge) and every 128-B
    record read once; makespan, status and digest, and with per-node output 8
    B per node, written once per record; per simulated node its start (a
    maximum of ready and free cycles), finish, server update and digest term,
    and per edge a maximum and a count."""
    g = _graph(case)
    B = case["records"]
    out = 16 + (8 * g.n_nodes if case["nodes"] else 0)
    return {"bytes": 10 * g.n_nodes + 4 * g.n_edges + (128 + out) * B, "flops": (12 * g.n_nodes + 2 * g.n_edges) * B}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """Whole numbers only: there is no rounding to measure against 64 bits
    (the tests compare them with a serial list scheduler, bit for bit)."""
    return None
