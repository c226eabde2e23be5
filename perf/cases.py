"""Performance cases: what a user of this library has it do.

Each case is one pass through the package's public entry points on inputs
that are already on the device: whole s-line graph ensembles from the
smallest query to the full power-law workload, the dual, rows streamed out
of a hypergraph whose line graph does not fit in memory, a batch replayed
as one HIP graph, a burst of served queries, and the later stages on an
emitted line graph (components, squeezing, symmetric CSR).

The inputs follow the laws of the package's own synthetic workloads
(``hypergen``), drawn on the device so that the full sizes are ready in a
fraction of a second: members by successive sampling (draw from the vertex
weights, drop repeats, redraw the deficit, for a bounded number of rounds),
rows sorted, the vertex CSR the exact transpose. A case names one hypergraph;
the seed permutes its hyperedge and vertex ids, so that every seed is another
input with the same amount of work and the same number of edges.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2201_11326_amd as slg

DEV = "cuda"
ROUNDS = 48  # redraws of a row's missing members


# -- inputs -----------------------------------------------------------------
@functools.lru_cache(maxsize=8)
def _cdf(n: int, exponent: float) -> np.ndarray:
    return np.cumsum(np.arange(1, n + 1, dtype=np.float64) ** (-exponent))


@functools.lru_cache(maxsize=8)
def _zipf_cdf(alpha: float, lo: int, hi: int) -> np.ndarray:
    return np.cumsum(np.arange(lo, hi + 1, dtype=np.float64) ** (-alpha))


def _weighted(gen, count: int, cdf: np.ndarray) -> torch.Tensor:
    """`count` indices drawn with the weights whose running sum is `cdf`."""
    u = torch.rand(count, generator=gen, device=DEV, dtype=torch.float64) * float(cdf[-1])
    return torch.searchsorted(torch.from_numpy(cdf).to(DEV), u, right=True).clamp_(max=len(cdf) - 1)


def _csr(rows: int, cols: int, key: torch.Tensor):
    """CSR of the sorted distinct keys row * cols + col."""
    ptr = torch.zeros(rows + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(torch.bincount(key // cols, minlength=rows), 0, out=ptr[1:])
    return ptr, (key % cols).to(torch.int32)


def _shuffled(gen, count: int) -> torch.Tensor:
    return torch.argsort(torch.rand(count, generator=gen, device=DEV), stable=True)


def _incidence(law: str, m: int, n: int, order: str, member: int, seed: int):
    """Both CSRs (he_ptr, he_idx, v_ptr, v_idx) of a hypergraph of m
    hyperedges over n vertices, on the device."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(11326 + 7919 * m + member)
    exponent = 0.0
    if law == "uniform":  # sizes 2..20, members uniform
        sizes = torch.randint(2, 21, (m,), generator=gen, device=DEV)
    elif law == "power_law":  # Zipf(2.1) sizes on [2, 5000], vertex weight ~ rank^-0.8
        sizes = _weighted(gen, m, _zipf_cdf(2.1, 2, 5000)) + 2
        exponent = 0.8
    elif law == "skewed":  # log-normal sizes, vertex weight ~ rank^-1.5
        z = torch.randn(m, generator=gen, device=DEV, dtype=torch.float64)
        sizes = torch.exp(1.5 + z).round_().clamp_(max=10000).to(torch.int64)
        exponent = 1.5
    else:  # a batch member: Zipf(2.1) sizes from 1, members uniform
        sizes = _weighted(gen, m, _zipf_cdf(2.1, 1, 1000)) + 1
    sizes.clamp_(max=n)
    row = torch.arange(m, device=DEV)
    need, held, parts = sizes, torch.zeros(0, dtype=torch.int64, device=DEV), []
    for _ in range(ROUNDS):
        at = torch.repeat_interleave(row, need)
        if at.numel() == 0:
            break
        if exponent:
            v = _weighted(gen, at.numel(), _cdf(n, exponent))
        else:
            v = torch.randint(0, n, (at.numel(),), generator=gen, device=DEV)
        new = torch.unique(torch.cat([held, at * n + v]))  # held: members of the unfinished rows
        need = sizes - torch.bincount(new // n, minlength=m)
        done = need[new // n] <= 0
        parts.append(new[done])
        held = new[~done]
        sizes = torch.where(need > 0, sizes, torch.zeros_like(sizes))
    key = torch.cat(parts + [held])
    # the seed's hyperedge and vertex ids
    gen.manual_seed(int(seed) * 1000003 + member + 1)
    new_v, new_row = _shuffled(gen, n), _shuffled(gen, m)
    if order == "ascending":  # ids as after relabelling by size: shuffled among equal sizes only
        size = torch.bincount(key // n, minlength=m)
        by_size = new_row[torch.argsort(size[new_row], stable=True)]
        new_row = torch.empty_like(by_size)
        new_row[by_size] = row
    key = torch.sort(new_row[key // n] * n + new_v[key % n]).values
    he_ptr, he_idx = _csr(m, n, key)
    v_ptr, v_idx = _csr(n, m, torch.sort((key % n) * m + key // n).values)
    return he_ptr, he_idx, v_ptr, v_idx


@functools.lru_cache(maxsize=1)
def _context() -> slg.Context:
    """The one context of the program."""
    return slg.Context()


@functools.lru_cache(maxsize=1)
def _server():
    return _context().server(workers=8, mem_budget_bytes=64 << 30)


def _s(case) -> list:
    return [int(x) for x in case["s"].split(",")]


def _hypergraph(case, seed: int):
    he_ptr, he_idx, v_ptr, v_idx = _incidence(case["law"], case["m"], case["n"], case.get("order", "as drawn"), 0, seed)
    m, n = case["m"], case["n"]
    if case.get("dual"):  # the s-clique graph: the roles of vertices and hyperedges swapped
        m, n, he_ptr, he_idx, v_ptr, v_idx = n, m, v_ptr, v_idx, he_ptr, he_idx
    return m, n, he_ptr, he_idx, v_ptr, v_idx


def _members(case):
    """(hyperedges, s) of every member of a batch or a server's pool: sizes
    log-uniform in [m_lo, m_hi]. They belong to the case, not to its seed,
    so that passes on other inputs are the same amount of work."""
    rng = np.random.default_rng(case["family"])
    out = []
    for _ in range(case["count"]):
        m = int(math.exp(rng.uniform(math.log(case["m_lo"]), math.log(case["m_hi"]))))
        out.append((m, int(rng.integers(1, 9))))
    return out


# -- cases ------------------------------------------------------------------
def listed():
    return [
        # the smallest query: the package's smoke workload; launches and read-backs
        {"name": "tiny_uniform", "kind": "line_graph", "law": "uniform", "m": 1000, "n": 2000, "s": "1,2,3,4"},
        # one query of the served pool's small members, alone
        {"name": "small_skewed", "kind": "line_graph", "law": "skewed", "m": 3163, "n": 1581, "s": "1,2,3,5,8"},
        # an ordinary hypergraph, the whole ensemble
        {"name": "power_law_50k", "kind": "line_graph", "law": "power_law", "m": 50021, "n": 100003, "s": "1,2,4,8"},
        # the power-law workload at full size, the whole ensemble in memory (27 GB of output)
        {"name": "power_law_full", "kind": "line_graph", "law": "power_law", "m": 500000, "n": 1000000, "s": "1,2,4,8"},
        # one high-order line graph of the relabelled (size-sorted) hypergraph: pruning, counting, few edges
        {"name": "ascending_s3", "kind": "line_graph", "law": "power_law", "m": 200003, "n": 399989, "s": "3",
         "order": "ascending"},
        # s-clique graphs: the dual of the power-law workload
        {"name": "dual_200k", "kind": "line_graph", "law": "power_law", "m": 200000, "n": 400000, "s": "1,2,4,8",
         "dual": True},
        # strongly skewed vertex degrees, in memory: rows whose partners fill most of E_s
        {"name": "skewed_300k", "kind": "line_graph", "law": "skewed", "m": 300007, "n": 150001, "s": "8,16"},
        # the large skewed workload at full size: a row range streamed out in chunks and collected
        {"name": "stream_10m", "kind": "stream", "law": "skewed", "m": 10000000, "n": 5000000, "s": "16", "from": 0.35,
         "two_paths": 120000000000, "chunk_bytes": 2 << 30, "room": 1500000000},
        # the batched family: 256 small hypergraphs, one HIP-graph replay
        {"name": "batch_256", "kind": "batch", "law": "batch", "family": 11330, "count": 256, "m_lo": 1000,
         "m_hi": 200000},
        # later stages on an emitted L_1: its s-connected components and compact ids, its symmetric CSR
        {"name": "components_200k", "kind": "components", "law": "power_law", "m": 200000, "n": 400000, "s": "1"},
        {"name": "symmetric_200k", "kind": "symmetric", "law": "power_law", "m": 200000, "n": 400000, "s": "1"},
        # a burst of served queries over a pool of small resident graphs and two ordinary ones
        {"name": "served_burst", "kind": "served", "law": "skewed", "family": 11331, "count": 24, "m_lo": 1000,
         "m_hi": 10000, "requests": 48, "ordinary_m": 50000},
    ]


def _log(rng, lo: int, hi: int) -> int:
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["small", "small", "skewed", "power", "power", "power", "dual", "stream", "batch", "components",
                       "symmetric", "served"])
    if kind == "small":
        m = _log(rng, 600, 10000)
        law = rng.choice(["uniform", "skewed"])
        s = sorted(rng.sample([1, 2, 3, 4, 5, 8], rng.randint(1, 6)))
        return {"kind": "line_graph", "law": law, "m": m, "n": m * 2 if law == "uniform" else max(m // 2, 1),
                "s": ",".join(map(str, s))}
    if kind == "skewed":
        m = _log(rng, 20000, 300000)
        return {"kind": "line_graph", "law": "skewed", "m": m, "n": m // 2, "s": rng.choice(["8,16", "8", "12,16,24"])}
    if kind == "power":
        m = _log(rng, 20000, 500000)
        return {"kind": "line_graph", "law": "power_law", "m": m, "n": 2 * m + rng.randint(0, 99),
                "s": rng.choice(["1,2,4,8", "1,2,4,8", "2", "2,3,5", "3", "4,8", "1,2,3,4,5,8"]),
                "order": rng.choice(["as drawn", "as drawn", "ascending"])}
    if kind == "dual":
        m = _log(rng, 20000, 400000)
        return {"kind": "line_graph", "law": "power_law", "m": m, "n": 2 * m, "s": rng.choice(["1,2,4,8", "2,4", "3"]),
                "dual": True}
    if kind == "stream":
        m = _log(rng, 1000000, 10000000)
        paths = min(_log(rng, 20000000000, 120000000000), int(m * (m / 400.0)))
        return {"kind": "stream", "law": "skewed", "m": m, "n": m // 2, "s": "16", "from": round(rng.uniform(0, 0.9), 2),
                "two_paths": paths, "chunk_bytes": 1 << 30, "room": paths // 80}
    if kind == "batch":
        return {"kind": "batch", "law": "batch", "family": rng.randint(1, 10 ** 6), "count": _log(rng, 16, 256),
                "m_lo": 1000, "m_hi": _log(rng, 20000, 200000)}
    if kind == "served":
        return {"kind": "served", "law": "skewed", "family": rng.randint(1, 10 ** 6), "count": rng.randint(8, 24),
                "m_lo": 1000, "m_hi": 10000, "requests": rng.randint(16, 48), "ordinary_m": _log(rng, 20000, 50000)}
    m = _log(rng, 20000, 200000)
    return {"kind": kind, "law": "power_law", "m": m, "n": 2 * m + 1, "s": rng.choice(["1", "2"])}


# -- one pass ---------------------------------------------------------------
def prepare(case, seed):
    ctx, kind = _context(), case["kind"]
    state = {"case": case, "ctx": ctx, "kind": kind}
    if kind in ("batch", "served"):
        graphs, thresholds = [], []
        for i, (m, s) in enumerate(_members(case)):
            n = 2 * m if kind == "batch" else max(m // 2, 1)
            inc = _incidence(case["law"], m, n, "as drawn", i, seed)
            graphs.append(ctx.register(m, n, *inc))
            thresholds.append(s)
        if kind == "batch":
            b = ctx.batch(graphs, thresholds)
            # the batch's own output arrays, rewritten by every replay
            state.update(graphs=graphs, batch=b, views=[b.result(g) for g in range(len(graphs))])
            return state
        for i in range(2):  # two ordinary graphs beside the small ones
            m = case["ordinary_m"]
            graphs.append(ctx.register(m, 2 * m, *_incidence("power_law", m, 2 * m, "as drawn", 4000 + i, seed)))
        rng = np.random.default_rng(case["family"])
        choices = np.asarray([1, 2, 3, 4, 5, 8])
        requests = []
        for r in range(case["requests"]):
            g = int(rng.integers(0, case["count"])) if r % 12 else case["count"] + (r // 12) % 2
            requests.append((g, sorted(int(x) for x in rng.choice(choices, size=int(rng.integers(1, 7)), replace=False))))
        torch.cuda.synchronize()  # the resident graphs are complete before any slot's stream reads them
        state.update(graphs=graphs, requests=requests, server=_server())
        return state
    m, n, *inc = _hypergraph(case, seed)
    state["s"], state["inputs"] = _s(case), inc
    g = state["graph"] = ctx.register(m, n, *inc)
    if kind == "stream":  # the row range of this many 2-paths, as equal-work shards are cut
        prefix = ctx.work_prefix(g, state["s"][0])
        r0 = int(np.searchsorted(prefix, case["from"] * prefix[-1]))
        r1 = int(np.searchsorted(prefix, min(prefix[r0] + case["two_paths"], prefix[-1])))
        state["rows"] = (r0, max(r1, r0))
        # the program's own arrays for the collected edges
        state["out"] = [{"row_ptr": torch.zeros(m + 1, dtype=torch.int64, device=DEV),
                         **{k: torch.zeros(case["room"], dtype=torch.int32, device=DEV) for k in ("row", "col", "w")}}
                        for _ in state["s"]]
    elif kind in ("components", "symmetric"):
        state["lg"] = ctx.line_graph(g, state["s"])[0]
    return state


def _arrays(lg):
    return {"row_ptr": lg.row_ptr, "row": lg.row, "col": lg.col, "w": lg.w}


def _joined(lgs):
    """The line graphs of many queries, array by array."""
    return {"row_ptr": torch.cat([x.row_ptr for x in lgs]), "row": torch.cat([x.row for x in lgs]),
            "col": torch.cat([x.col for x in lgs]), "w": torch.cat([x.w for x in lgs])}


def run(state):
    ctx, kind = state["ctx"], state["kind"]
    if kind == "line_graph":
        return [_arrays(lg) for lg in ctx.line_graph(state["graph"], state["s"])]
    if kind == "stream":
        at = [0] * len(state["s"])

        def take(k, s, r0, r1, e0, row_ptr, row, col, w):  # a chunk's arrays live until the next but one
            out, n = state["out"][k], row.numel()
            out["row_ptr"][r0:r1 + 1] = row_ptr + e0
            for name, part in (("row", row), ("col", col), ("w", w)):
                out[name][e0:e0 + n] = part
            at[k] = e0 + n

        ctx.line_graph_stream(state["graph"], state["s"], state["case"]["chunk_bytes"], take, rows=state["rows"])
        return [dict(out, edges=e) for out, e in zip(state["out"], at)]
    if kind == "batch":
        state["batch"].run()
        return _joined(state["views"])
    if kind == "components":
        labels, count = ctx.components(state["graph"], state["s"][0], state["lg"])
        new_id, kept = ctx.squeeze(state["graph"].m, state["lg"])
        return {"labels": labels, "count": count, "new_id": new_id, "kept": kept}
    if kind == "symmetric":
        ptr, col, w = ctx.symmetrize(state["lg"])
        return {"ptr": ptr, "col": col, "w": w}
    srv = state["server"]
    tickets = [srv.submit(state["graphs"][g], s) for g, s in state["requests"]]
    return _joined([lg for t in tickets for lg in srv.wait(t).outs])


# -- what a pass cannot do without ------------------------------------------
def _two_paths(he_ptr, he_idx, v_ptr, v_idx, s_min: int) -> float:
    """2-paths e_i -> v -> e_j (i < j) between hyperedges of at least s_min members."""
    keep = (he_ptr[1:] - he_ptr[:-1] >= s_min)[v_idx.long()]
    run_sum = torch.zeros(v_idx.numel() + 1, dtype=torch.int64, device=DEV)
    torch.cumsum(keep, 0, out=run_sum[1:])
    d = (run_sum[v_ptr[1:]] - run_sum[v_ptr[:-1]]).double()
    return float((d * (d - 1) / 2).sum())


def _bytes(x) -> float:
    if isinstance(x, torch.Tensor):
        return float(x.numel() * x.element_size())
    if isinstance(x, dict):
        return sum(_bytes(v) for v in x.values())
    return sum(_bytes(v) for v in x) if isinstance(x, (list, tuple)) else 8.0


def work(case):
    """Every input read once and every output written once; one addition per
    2-path (components and the symmetric CSR: one step per edge)."""
    kind, state = case["kind"], prepare(case, 1)
    out = run(state)
    if kind in ("batch", "served"):
        nbytes, flops = _bytes(out), 0.0
        asked = (zip(range(len(state["graphs"])), ([s] for s in state["batch"].s)) if kind == "batch"
                 else state["requests"])
        for g, s in asked:
            inc = state["graphs"][g]._tensors
            nbytes += _bytes(list(inc))
            flops += _two_paths(*inc, s[0])
        return {"bytes": nbytes, "flops": flops}
    if kind == "components":
        e = state["lg"].num_edges
        return {"bytes": 8.0 * e + 16.0 * case["m"], "flops": float(e)}
    if kind == "symmetric":
        e = state["lg"].num_edges
        return {"bytes": _bytes(_arrays(state["lg"])) + _bytes(out), "flops": float(e)}
    if kind == "stream":
        nbytes = sum(12.0 * x["edges"] + 8.0 * (state["rows"][1] - state["rows"][0]) for x in out)
        return {"bytes": _bytes(state["inputs"]) + nbytes, "flops": float(case["two_paths"])}
    flops = _two_paths(*state["inputs"], state["s"][0])
    return {"bytes": _bytes(state["inputs"]) + _bytes(out), "flops": flops}


def exact(case, seed):
    """L_s of a small hypergraph from the product of its incidence matrix
    with its own transpose, in 64 bits."""
    if case["kind"] != "line_graph" or case["m"] > 6000 or case["n"] > 12000:
        return None
    m, n, he_ptr, he_idx, _, _ = _hypergraph(case, seed)
    h = torch.zeros(m, n, dtype=torch.float64)
    at = torch.repeat_interleave(torch.arange(m), (he_ptr[1:] - he_ptr[:-1]).cpu())
    h[at, he_idx.long().cpu()] = 1.0
    overlap = torch.triu(h @ h.t(), diagonal=1)
    out = []
    for s in _s(case):
        row, col = torch.nonzero(overlap >= s, as_tuple=True)
        ptr = torch.zeros(m + 1, dtype=torch.int64)
        torch.cumsum(torch.bincount(row, minlength=m), 0, out=ptr[1:])
        out.append({"row_ptr": ptr, "row": row.to(torch.int32), "col": col.to(torch.int32),
                    "w": overlap[row, col].round().to(torch.int32)})
    return out
