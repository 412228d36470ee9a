"""Seeded graphs whose kernels run from compact template records (test helper).

Each kernel replicates one random CTA graph that ends in one store which every
other node reaches over DATA / SYNC edges.  It keeps to what those records
hold -- in-degrees up to 31, eight successors of a compute node, four at issue
(ORDER) and four at completion of a load or store -- and goes to those bounds:
wide joins and fan-outs, SYNC and SMEM nodes, ORDER edges beside DATA, several
op classes per kernel.  Between them, with probability `mixed`, kernels whose
CTAs differ in shape (no template: they run from global memory)."""
from paper_2607_11262_amd.gen.graph import (ALU, DATA, GLOAD, GSTORE, MISS, ORDER, SFU, SMEM, SYNC, SYNC_EDGE, TENSOR,
                                            GraphBuilder)

MOST_IN, MOST_COMPUTE, MOST_ISSUE, MOST_END = 31, 8, 4, 4


def _local(rng, n):
    """Classes of n local nodes and their edges {(u, v): kind}."""
    cls = [rng.choice([TENSOR, ALU, SFU, SMEM, SYNC, GLOAD, GLOAD, GSTORE]) for _ in range(n - 1)] + [GSTORE]
    edges = {}
    indeg, at_issue, at_end = [0] * n, [0] * n, [0] * n

    def fits(u, v, kind, reserve):
        # `reserve`: one edge at completion is kept for u's way to the sink
        if u >= v or (u, v) in edges or indeg[v] >= MOST_IN:
            return False
        spare = 1 if reserve and at_end[u] == 0 and kind == ORDER else 0
        if cls[u] in (GLOAD, GSTORE):
            return at_issue[u] < MOST_ISSUE if kind == ORDER else at_end[u] < MOST_END
        return at_issue[u] + at_end[u] + spare < MOST_COMPUTE

    def add(u, v, kind, reserve=True):
        if not fits(u, v, kind, reserve):
            return False
        edges[(u, v)] = kind
        indeg[v] += 1
        if kind == ORDER:
            at_issue[u] += 1
        else:
            at_end[u] += 1
        return True

    for v in range(1, n):
        for _ in range(rng.randint(0, 3)):
            add(rng.randint(max(0, v - rng.choice([1, 4, 40])), v - 1), v, rng.choice([DATA, DATA, ORDER, SYNC_EDGE]))
    for _ in range(rng.randint(0, 2)):  # a wide join, up to the largest in-degree
        v = rng.randint(1, n - 1)
        for _ in range(rng.choice([8, 31, 40])):
            add(rng.randint(0, v - 1), v, rng.choice([DATA, ORDER, SYNC_EDGE]))
    for _ in range(rng.randint(0, 3)):  # a wide fan-out
        u = rng.randint(0, n - 2)
        for _ in range(rng.randint(4, 10)):
            add(u, rng.randint(u + 1, n - 1), rng.choice([DATA, ORDER]))
    for u in range(n - 1):  # every node's way to the sink
        if at_end[u]:
            continue
        for v in [rng.randint(u + 1, n - 1) for _ in range(4)] + list(range(u + 1, n)):
            if (u, v) in edges:  # an ORDER edge, or a full target
                continue
            if add(u, v, DATA, False):
                break
        else:
            return None
    return cls, edges


def single_sink_graph(rng, n_kernels=(1, 4), n_local=(2, 80), n_ctas=(2, 40), mixed=0.0, work=1 << 14):
    """Returns the graph and the number of its single-sink kernels."""
    b = GraphBuilder()
    sinks = 0
    kernels = rng.randint(*n_kernels)
    for _k in range(kernels):
        local = None
        while local is None:
            n = rng.randint(*n_local)
            local = _local(rng, n)
        cls, edges = local
        ragged = rng.randint(0, 999) < 1000 * mixed
        sinks += not ragged
        # at most 16 ops, and CTAs of up to three op classes (two with more than
        # two kernels: class x op entries stay within a graph's 128), which
        # differ in work or the L2-miss flag
        palette = {c: [(rng.randint(1, work), rng.choice([1, 3, 0xF])) for _ in range(2)] for c in set(cls)}
        ops = [(c, *rng.choice(palette[c])) for c in cls]
        variants = [(0, 0)] + [(rng.randint(0, work), rng.randint(0, 1)) for _ in range(rng.randint(0, 2 if kernels <= 2 else 1))]
        b.kernel(4, rng.choice([0, 1024, 8192]))
        for c in range(rng.randint(*n_ctas)):
            b.cta()
            more, miss = variants[rng.randint(0, len(variants) - 1)]
            # a ragged kernel's CTAs drop nodes from the front
            drop = rng.randint(0, n - 2) if ragged and n > 2 else 0
            if ragged and c == 0:
                drop = 0
            ids = {}
            for i in range(drop, n):
                cl, w, warps = ops[i]
                ids[i] = b.node(cl, 0 if cl == SYNC else w + more, warps, MISS if cl in (GLOAD, GSTORE) and miss else 0)
            for (u, v), kind in sorted(edges.items()):
                if u >= drop:
                    b.edge(ids[u], ids[v], kind)
        if ragged:  # at least two shapes
            b.cta()
            b.node(GSTORE, rng.randint(1, work), 1)
    return b.build("single_sink"), sinks
