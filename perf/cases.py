"""What a user of this library has it do, as cases that can be timed.

A case names an operation, a graph family and its sizes.  The families are
those of the benchmark and the tests: G(n, q) ("er") and R-MAT with
(a,b,c,d) = (.57,.19,.19,.05) ("rmat"), undirected and simple, as symmetric
CSRs resident in device memory; the graphs are drawn on the GPU from the
seed.  Operations: the six compressions through their single-graph calls,
many graphs as one batch, jobs through the in-process server, and the degree
divergence metric.  Output buffers have the case's capacity, as a program
that compresses many graphs of one size keeps them, and columns past the
written entries stay zero: the buffers are cleared when they are made, and no
call writes there.
"""
import math

import numpy as np
import torch

from paper_1912_08950_amd import slim

DEV = "cuda:0"
A, B, C = 0.57, 0.19, 0.19  # R-MAT quadrant probabilities

OPS = {"tr": slim.OP_TR, "tr2": slim.OP_TR2, "mctr": slim.OP_MCTR, "eotr": slim.OP_EOTR,
       "es": slim.OP_ES}
# operations of the server's jobs, in turn, and their deletion probabilities
SERVE_OPS = (slim.OP_TR, slim.OP_ES, slim.OP_TR2, slim.OP_MCTR)
SERVE_P = (0.2, 0.5, 0.8)


def listed():
    return [
        # the smallest configuration of the benchmark (2000 vertices, average
        # degree 16): latency of one call, for the edge kernel and for the
        # triangle pipeline
        {"name": "es_er2000", "op": "es", "kind": "er", "n": 2000, "d": 16.0, "p": 0.5},
        {"name": "tr_er2000", "op": "tr", "kind": "er", "n": 2000, "d": 16.0, "p": 0.5},
        # a ragged mid-size graph (no power of two, fractional degree); a
        # selected triangle loses two edges
        {"name": "tr2_rmat_90001", "op": "tr2", "kind": "rmat", "n": 90001, "d": 23.5, "p": 0.8},
        # R-MAT scale 20, a mid-size single graph of the benchmark
        {"name": "tr_rmat20", "op": "tr", "kind": "rmat", "n": 1 << 20, "d": 32.0, "p": 0.5},
        # the headline workload: R-MAT scale 24, edge factor 16
        {"name": "tr_rmat24", "op": "tr", "kind": "rmat", "n": 1 << 24, "d": 32.0, "p": 0.5},
        # the variants that list triangles more than once
        {"name": "mctr_rmat20", "op": "mctr", "kind": "rmat", "n": 1 << 20, "d": 32.0, "p": 0.5},
        {"name": "eotr_rmat20", "op": "eotr", "kind": "rmat", "n": 1 << 20, "d": 32.0, "p": 0.5},
        # the edge kernels at full size: sampling at scale 24, sparsification
        # with weights at scale 22 (upsilon = p m / n with p = 0.5)
        {"name": "es_rmat24", "op": "es", "kind": "rmat", "n": 1 << 24, "d": 32.0, "p": 0.5},
        {"name": "spectral_rmat22", "op": "spectral", "kind": "rmat", "n": 1 << 22, "d": 32.0,
         "p": 8.0},
        # the benchmark's mixed population (half G(n,q), half R-MAT, n
        # log-uniform in [1e3, 2e5], degree 4..64) as one batch
        {"name": "batch_tr_256", "op": "batch", "kind": "mix", "n": 200000, "d": 64.0, "p": 0.5,
         "count": 256},
        # a burst of small mixed jobs through the server, results copied out
        {"name": "serve_burst_16", "op": "serve", "kind": "mix", "n": 20000, "d": 64.0, "p": 0.5,
         "count": 16},
        # accuracy metric after a compression, over bounded-degree vertices
        {"name": "kl_4m", "op": "kl", "kind": "degrees", "n": 1 << 22, "d": 128.0, "p": 0.05},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    op = rng.choice(("tr", "tr", "tr2", "mctr", "eotr", "es", "spectral", "batch", "serve", "kl"))
    p = rng.choice((0.2, 0.5, 0.8, rng.uniform(0.0, 1.0)))
    if op in ("batch", "serve"):
        count = int(_log_uniform(rng, 2, 300)) if op == "batch" else rng.randint(2, 20)
        n = int(_log_uniform(rng, 2000, 200000 if op == "batch" else 20000))
        return {"op": op, "kind": "mix", "n": n, "d": rng.uniform(8.0, 64.0), "p": p,
                "count": count}
    if op == "kl":
        # the largest degrees occur often enough to stay in the output, so
        # that the divergence is finite
        n = int(_log_uniform(rng, 4096, 1 << 24))
        return {"op": op, "kind": "degrees", "n": n,
                "d": float(rng.randint(4, int(math.sqrt(n)) // 4)), "p": rng.uniform(0.01, 0.5)}
    kind = rng.choice(("er", "rmat"))
    d = rng.uniform(4.0, 64.0)
    # entries at most: what keeps a case below the headline one in time
    # (G(n,q) has few triangles)
    most = {"tr": 1e8, "tr2": 1e8, "mctr": 4e7, "eotr": 2.4e7, "es": 4e8, "spectral": 2e8}[op]
    n = int(_log_uniform(rng, 1000, min(1 << 24, most / d)))
    if op == "spectral":
        p = rng.uniform(0.5, 1.0) * d / 4
    return {"op": op, "kind": kind, "n": n, "d": d, "p": p}


# ------------------------------------------------------------------ inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _csr(u, v, n):
    """Symmetric sorted CSR of the undirected simple graph on pairs (u, v)."""
    keep = u != v
    u, v = u[keep], v[keep]
    key = torch.cat((u * n + v, v * n + u))
    del u, v
    key = _unique(key)
    starts = torch.arange(n + 1, device=DEV, dtype=torch.int64) * n
    row_off = torch.searchsorted(key, starts)
    return row_off, key.remainder_(n).to(torch.int32)


def _unique(key):
    key = torch.sort(key).values
    first = torch.ones_like(key, dtype=torch.bool)
    torch.ne(key[1:], key[:-1], out=first[1:])
    return key[first]


def _exactly(u, v, n, m, g):
    """m distinct pairs of [0, n): of (u, v), drawn without order, or all of
    them and uniform ones for what is missing."""
    key = _unique(torch.where(u < v, u * n + v, v * n + u)[u != v])
    while key.numel() < m:
        a, b = (torch.randint(n, (2 * m,), device=DEV, generator=g) for _ in range(2))
        more = torch.where(a < b, a * n + b, b * n + a)[a != b]
        key = _unique(torch.cat((key, more[:4 * (m - key.numel())])))
    key = key[torch.randperm(key.numel(), device=DEV, generator=g)[:m]]
    return key // n, key % n


def _samples(kind, n, d):
    """Pairs drawn for a graph: a bound on its undirected edges."""
    size = 1 << max(1, math.ceil(math.log2(n)))
    return max(1, int(round(n * d / 2 * (1 if kind == "er" else (size / n) ** 2))))


def _graph(kind, n, d, seed, edges=None):
    """CSR of a graph of n vertices and average degree near d; with `edges`,
    of exactly so many undirected edges."""
    g = _gen(seed)
    m = _samples(kind, n, d)
    if kind == "er":
        u = torch.randint(n, (m,), device=DEV, generator=g)
        v = torch.randint(n, (m,), device=DEV, generator=g)
    else:
        scale = max(1, math.ceil(math.log2(n)))
        u = torch.zeros(m, dtype=torch.int32, device=DEV)
        v = torch.zeros(m, dtype=torch.int32, device=DEV)
        r = torch.empty(m, dtype=torch.float32, device=DEV)
        for _ in range(scale):
            r.uniform_(generator=g)
            bu = r >= A + B
            bv = ((r >= A) & ~bu) | (r >= A + B + C)
            u.mul_(2).add_(bu)
            v.mul_(2).add_(bv)
        del r, bu, bv
        # ids through a random bijection; endpoints past n are dropped
        perm = torch.randperm(1 << scale, device=DEV, generator=g)
        u, v = perm[u.long()], perm[v.long()]
        if 1 << scale > n:
            keep = (u < n) & (v < n)
            u, v = u[keep], v[keep]
    if edges is not None:
        u, v = _exactly(u, v, n, edges, g)
    return _csr(u, v, n)


def _mix_sizes(case):
    """(kind, n, d, undirected edges) of the mixed population: even indices
    G(n,q), odd R-MAT (of whose samples a fifth may be duplicates)."""
    out = []
    for i in range(case["count"]):
        a, b = (i * 0.6180339887498949 + 0.5) % 1.0, (i * 0.7548776662466927 + 0.5) % 1.0
        n = int(1000 * (case["n"] / 1000) ** a)
        d = 4.0 + (case["d"] - 4.0) * b
        out.append(("rmat" if i % 2 else "er", n, d, int((0.4 if i % 2 else 0.48) * n * d)))
    return out


def _mix(case, seed):
    return [_graph(kind, n, d, seed * 1000003 + i, m)
            for i, (kind, n, d, m) in enumerate(_mix_sizes(case))]


def _offsets(deg):
    return torch.cat((torch.zeros(1, dtype=torch.int64, device=DEV), torch.cumsum(deg, 0)))


def _degrees(case, seed):
    """Row offsets of an input whose degrees fall off as 1/k^2 up to a bound,
    and of an output in which a share p of the vertices lost about half of
    their entries."""
    g = _gen(seed)
    x = torch.rand(case["n"], device=DEV, generator=g, dtype=torch.float64)
    deg = (1.0 / (1.0 - x)).clamp(max=case["d"]).floor()
    hit = torch.rand(case["n"], device=DEV, generator=g) < case["p"]
    half = torch.binomial(deg, torch.full_like(deg, 0.5), generator=g)
    return _offsets(deg.long()), _offsets(torch.where(hit, half, deg).long())


def prepare(case, seed):
    op = case["op"]
    if op == "kl":
        ro_p, ro_q = _degrees(case, seed)
        # the workspace that a program keeps
        out = torch.empty(1, dtype=torch.float64, device=DEV)
        ws = torch.empty(16 * (case["n"] + 1) + (64 << 10), dtype=torch.uint8, device=DEV)
        return {"op": op, "p": ro_p, "q": ro_q, "out": out, "ws": ws}
    if op in ("batch", "serve"):
        graphs = [slim.Graph(ro, col) for ro, col in _mix(case, seed)]
        if op == "batch":
            b = slim.Batch(graphs, [(slim.OP_TR, case["p"], seed + i)
                                    for i in range(len(graphs))])
            b.col_all.zero_()
            return {"op": op, "batch": b}
        jobs = [(SERVE_OPS[i % len(SERVE_OPS)], SERVE_P[i % len(SERVE_P)], seed + i)
                for i in range(len(graphs))]
        # host arrays that collect the results
        cols = [np.zeros(2 * m, dtype=np.uint32) for _, _, _, m in _mix_sizes(case)]
        return {"op": op, "graphs": graphs, "jobs": jobs, "cols": cols,
                "server": slim.Server(4 << 30)}
    g = slim.Graph(*_graph(case["kind"], case["n"], case["d"], seed))
    bufs = slim.Buffers(g, slim.OP_SPECTRAL if op == "spectral" else OPS[op])
    cap = 2 * _samples(case["kind"], case["n"], case["d"])
    bufs.out_col = torch.zeros(cap, dtype=torch.int32, device=DEV)
    if bufs.out_w is not None:
        bufs.out_w = torch.zeros(cap, dtype=torch.float32, device=DEV)
    return {"op": op, "graph": g, "bufs": bufs, "p": case["p"], "seed": seed}


def run(state):
    op = state["op"]
    if op == "kl":
        return {"kl": slim.degree_kl(state["p"], state["q"], out=state["out"], ws=state["ws"])}
    if op == "batch":
        b = state["batch"]
        b.run()
        return {"row_off": b.row_off_all, "col": b.col_all, "stats": b.stats_all}
    if op == "serve":
        s = state["server"]
        tickets = [s.submit(g, *job) for g, job in zip(state["graphs"], state["jobs"])]
        out = {}
        for i, (t, dst) in enumerate(zip(tickets, state["cols"])):
            ro, col, st = s.result_numpy(t)
            dst[:col.size] = col
            out["job%d" % i] = {"row_off": ro, "col": dst, "m_out": st["m_out"]}
            s.release(t)
        return out
    b, p, seed = state["bufs"], state["p"], state["seed"]
    if op == "spectral":
        slim.spectral_sparsify(state["graph"], p, seed, b)
        return {"row_off": b.out_row_off, "col": b.out_col, "weight": b.out_w, "stats": b.stats}
    if op == "tr":
        slim.triangle_reduce(state["graph"], p, seed, b)
    elif op == "es":
        slim.edge_sample(state["graph"], p, seed, b)
    else:
        slim.compress(state["graph"], OPS[op], p, seed, b)
    return {"row_off": b.out_row_off, "col": b.out_col, "stats": b.stats}


def work(case):
    """Bytes: the CSR read once and the output written once, with the share
    of the entries that the operation is expected to keep; duplicate samples
    of the generators are not taken off."""
    op, n, d = case["op"], case["n"], case["d"]
    if op == "kl":
        return {"bytes": 16 * (n + 1) + 8, "flops": 0}
    if op in ("batch", "serve"):
        # mean of 1000 (n/1000)^a over a in [0, 1), mean degree (4 + d) / 2
        n = case["count"] * 1000 * (n / 1000 - 1) / math.log(n / 1000)
        d = (4.0 + d) / 2
    nnz = n * d
    keep = 1 - case["p"] if op == "es" else 0.25 if op == "spectral" else 0.5
    out = 4 * nnz * keep * (2 if op == "spectral" else 1)
    return {"bytes": 16 * n + 4 * nnz + out, "flops": 0}


# ------------------------------------------------- values in 64 bits
def _philox_word0(x0, x1, x2, x3, k0, k1):
    """Word 0 of Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) over int64
    tensors of 32-bit values."""
    mask = 0xFFFFFFFF
    for _ in range(10):
        a, b = x0 * 0xD2511F53, x2 * 0xCD9E8D57  # wraps in 64 bits, as the products do
        x0, x1, x2, x3 = (((b >> 32) & mask) ^ x1 ^ k0, b & mask,
                          ((a >> 32) & mask) ^ x3 ^ k1, a & mask)
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return x0


def exact(case, seed):
    op = case["op"]
    if op == "kl":
        ro_p, ro_q = _degrees(case, seed)
        p, q = (torch.bincount(torch.diff(r), minlength=int(case["d"]) + 1).double()
                for r in (ro_p, ro_q))
        p, q = p[:int(case["d"]) + 1], q[:int(case["d"]) + 1]
        t = torch.where(p > 0, p / case["n"] * torch.log2(p / q), torch.zeros_like(p))
        return {"kl": t.sum().reshape(1)}
    if op != "spectral":
        return None
    ro, col = _graph(case["kind"], case["n"], case["d"], seed)
    deg = torch.diff(ro)
    row = torch.repeat_interleave(torch.arange(case["n"], device=DEV), deg)
    col = col.long()
    pe = (case["p"] / torch.minimum(deg[row], deg[col]).double()).clamp(max=1.0)
    a, b = torch.minimum(row, col), torch.maximum(row, col)
    del row, col
    w0 = _philox_word0(a, b, torch.zeros_like(a), torch.full_like(a, 2), seed & 0xFFFFFFFF,
                       (seed >> 32) & 0xFFFFFFFF)
    kept = 1.0 / pe[w0 < torch.floor(pe * 4294967296.0).long()]
    cap = 2 * _samples(case["kind"], case["n"], case["d"])
    weight = torch.zeros(cap, dtype=torch.float64, device=DEV)
    weight[:kept.numel()] = kept
    return {"row_off": None, "col": None, "weight": weight, "stats": None}
