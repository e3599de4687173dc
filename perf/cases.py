"""Workloads of the bitruss library, with their inputs: what bench runs and
profiles of single entry points time.

Each case is one call (or one submit-and-drain of the serving engine) as a
user's program makes it, on graphs of the shapes that the package's own
generators draw: uniform pairs, Chung-Lu power laws (the 5M-edge workload
and its scaled copies), hub-heavy Chung-Lu, the many-small-graphs pool and
the large request graphs.  The graphs are drawn on the GPU from the seed, so
another seed is another graph of the same sizes.
"""
import math
import random

import numpy as np
import torch

from paper_2001_06111_amd import binding, synth

DEV = "cuda"


def listed():
    return [
        # Supports of a small graph, the smallest call: launches and host
        # waits are all of it.
        {"name": "support-uniform-10k", "call": "support", "shape": "uniform", "m": 10_000},
        # The same from static scratch (graph capture, tight serving loops),
        # near the largest graph that entry point takes.
        {"name": "noalloc-chunglu-250k", "call": "noalloc", "shape": "chunglu", "m": 250_000},
        # Supports of the 5M-edge power-law workload.
        {"name": "support-chunglu-5m", "call": "support", "shape": "chunglu", "m": 5_000_000},
        # Supports of the 20M-edge hub-heavy workload, the largest input.
        {"name": "support-hub-20m", "call": "support", "shape": "hub", "m": 20_000_000},
        # Bitruss numbers of one small graph (the plain small workload).
        {"name": "decompose-uniform-10k", "call": "decompose", "shape": "uniform", "m": 10_000},
        # One graph of ordinary size, an odd edge count.
        {"name": "decompose-chunglu-200k", "call": "decompose", "shape": "chunglu", "m": 200_003},
        # The single-graph headline: 5M edges.
        {"name": "decompose-chunglu-5m", "call": "decompose", "shape": "chunglu", "m": 5_000_000},
        # Progressive compression on a hub-heavy graph, which it is for.
        {"name": "pc-hub-400k", "call": "pc", "shape": "hub", "m": 400_000},
        # A batch of graphs as the pool draws them (200 to 200,000 edges).
        {"name": "batch-pool-192", "call": "batch", "shape": "pool", "graphs": 192,
         "m_max": 200_000, "sizes": 1},
        # A batch of small graphs alone (the serving engine's small class).
        {"name": "batch-small-512", "call": "batch", "shape": "pool", "graphs": 512,
         "m_max": 16_000, "sizes": 2},
        # The serving engine: a burst of pool requests submitted and drained.
        {"name": "serve-pool-24", "call": "serve", "shape": "pool", "graphs": 24,
         "m_max": 200_000, "sizes": 3},
        # Connected components of a k-bitruss, a query on finished numbers.
        {"name": "components-chunglu-1m", "call": "components", "shape": "chunglu",
         "m": 1_000_000, "k": 8},
    ]


def _log_int(rng, lo, hi):
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    call = rng.choice(["support", "support", "noalloc", "decompose", "decompose", "decompose",
                       "pc", "batch", "batch", "serve", "components"])
    if call in ("batch", "serve"):
        m_max = _log_int(rng, 2_000, 200_000)
        return {"call": call, "shape": "pool",
                "graphs": _log_int(rng, 3, (24 if call == "serve" else 160)), "m_max": m_max,
                "sizes": rng.randrange(1000)}
    shape = rng.choice(["uniform", "chunglu", "chunglu", "hub"])
    top = {"support": {"uniform": 5_000_000, "chunglu": 5_000_000, "hub": 15_000_000},
           "noalloc": {"uniform": 250_000, "chunglu": 250_000, "hub": 200_000},
           "decompose": {"uniform": 4_000_000, "chunglu": 4_000_000, "hub": 300_000},
           "pc": {"uniform": 200_000, "chunglu": 400_000, "hub": 300_000},
           "components": {"uniform": 1_000_000, "chunglu": 1_000_000, "hub": 200_000}}[call][shape]
    case = {"call": call, "shape": shape, "m": _log_int(rng, 1_000, top)}
    if call == "components":
        case["k"] = rng.choice([0, 1, 2, 5, 13, 40])
    return case


# --- sizes -------------------------------------------------------------------

def _single_size(case):
    """(n_upper, n_lower, edges) of a single-graph case."""
    m, shape = case["m"], case["shape"]
    if shape == "uniform":  # the 1,000 x 1,500 workload's aspect and density
        f = math.sqrt(m / 10_000)
        nu, nl = max(8, round(1000 * f)), max(8, round(1500 * f))
    elif shape == "chunglu":  # synth.scaled_chunglu's
        f = m / 5_000_000
        nu, nl = max(8, round(200_000 * f)), max(8, round(500_000 * f))
    else:  # the hub-heavy workload's aspect
        f = m / 20_000_000
        nu, nl = max(8, round(100_000 * f)), max(8, round(2_000_000 * f))
    return nu, nl, min(m, nu * nl // 4)


def _pool_sizes(case):
    """Graph sizes as synth.batch_graph draws them, up to m_max edges."""
    r = random.Random(case["sizes"])
    out = []
    for _ in range(case["graphs"]):
        nu = int(math.exp(r.uniform(math.log(50), math.log(20_000))))
        nl = int(math.exp(r.uniform(math.log(50), math.log(20_000))))
        m = int(math.exp(r.uniform(math.log(200), math.log(case["m_max"]))))
        out.append((nu, nl, min(m, nu * nl // 4)))
    return out


# --- graphs ------------------------------------------------------------------

def _csr(nu, nl, keys):
    keys = torch.sort(keys).values
    u = torch.div(keys, nl, rounding_mode="floor")
    row_ptr = torch.zeros(nu + 1, dtype=torch.int64, device=DEV)
    row_ptr[1:] = torch.cumsum(torch.bincount(u, minlength=nu), 0)
    return binding.DeviceGraph(nu, nl, row_ptr, (keys - u * nl).to(torch.int32))


def _first_distinct(pairs, m):
    """The first m distinct keys of a stream; pairs(k) draws the next k."""
    keys = torch.empty(0, dtype=torch.int64, device=DEV)
    while True:
        keys = torch.cat([keys, pairs(max(m, 1024))])
        order = torch.sort(keys, stable=True)
        new = torch.ones_like(order.values, dtype=torch.bool)
        new[1:] = order.values[1:] != order.values[:-1]
        first = torch.sort(order.indices[new]).values
        keys = keys[first]
        if keys.numel() >= m:
            return keys[:m]


def _uniform(nu, nl, m, gen):
    def pairs(k):
        u = torch.randint(nu, (k,), generator=gen, device=DEV)
        return u * nl + torch.randint(nl, (k,), generator=gen, device=DEV)
    return _csr(nu, nl, _first_distinct(pairs, m))


def _chung_lu(nu, nl, m, su, sl, cap_u, cap_l, rng, gen):
    ends = []
    for n, s, cap in ((nu, su, cap_u), (nl, sl, cap_l)):
        w = np.empty(n)
        w[rng.permutation(n)] = synth.expected_degrees(n, m, s, cap)
        ends.append(torch.from_numpy(np.cumsum(w)).to(DEV))

    def side(c, k):
        x = torch.rand(k, generator=gen, device=DEV, dtype=torch.float64) * c[-1]
        return torch.searchsorted(c, x, right=True).clamp_(max=c.numel() - 1)
    return _csr(nu, nl, _first_distinct(lambda k: side(ends[0], k) * nl + side(ends[1], k), m))


def _graph(case, seed):
    nu, nl, m = _single_size(case)
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    if case["shape"] == "uniform":
        return _uniform(nu, nl, m, gen)
    # Hubs hold up to 1% of the edges; four times the mean degree always fits.
    cap_u = min(float(nl), max(m / 100, 4.0 * m / nu))
    cap_l = min(float(nu), max(m / 100, 4.0 * m / nl))
    su, sl = (2.1, 2.5) if case["shape"] == "chunglu" else (1.8, 2.3)
    return _chung_lu(nu, nl, m, su, sl, cap_u, cap_l, rng, gen)


def _pool(case, seed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device=DEV).manual_seed(seed)
    return [_chung_lu(nu, nl, m, 2.2, 2.2, float(nl), float(nu), rng, gen)
            for nu, nl, m in _pool_sizes(case)]


# --- calls -------------------------------------------------------------------

def prepare(case, seed):
    state = {"case": case}
    if case["shape"] == "pool":
        state["graphs"] = _pool(case, seed)
        if case["call"] == "serve":
            state["engine"] = binding.BtEngine(slots=2)
            state["next"] = 0
    else:
        state["graph"] = _graph(case, seed)
        if case["call"] == "noalloc":
            state["sup"] = torch.empty(state["graph"].m, dtype=torch.int64, device=DEV)
        if case["call"] == "components":
            state["phi"] = binding.bt_decompose(state["graph"], want_sup=False)[1]
    torch.cuda.synchronize()
    return state


def run(state):
    case = state["case"]
    call = case["call"]
    if call == "support":
        return list(binding.bt_support(state["graph"]))
    if call == "noalloc":
        return list(binding.bt_support_noalloc(state["graph"], out_sup=state["sup"]))
    if call == "decompose":
        return list(binding.bt_decompose(state["graph"])[:2])
    if call == "pc":
        return list(binding.bt_decompose_pc(state["graph"])[:2])
    if call == "components":
        return list(binding.bt_bitruss_components(state["graph"], state["phi"], case["k"]))
    if call == "batch":
        sups, phis, _ = binding.bt_decompose_batch(state["graphs"])
        return [torch.cat(sups), torch.cat(phis)]
    eng, first = state["engine"], state["next"]
    state["next"] += len(state["graphs"])
    for i, g in enumerate(state["graphs"]):
        eng.bt_engine_submit(g, first + i, want_sup=True)
    eng.bt_engine_drain()
    done = eng.bt_engine_poll()
    assert len(done) == len(state["graphs"]) and all(s == binding.BT_OK for _, s in done)
    res = [eng.results.pop(first + i) for i in range(len(state["graphs"]))]
    return [torch.cat([r[1] for r in res]), torch.cat([r[2] for r in res])]


def work(case):
    """Each graph (row_ptr, col) read once, each int64 output written once."""
    sizes = _pool_sizes(case) if case["shape"] == "pool" else [_single_size(case)]
    per_edge = {"support": 4 + 8, "noalloc": 4 + 8, "components": 4 + 8 + 4}.get(case["call"],
                                                                             4 + 16)
    return {"bytes": sum(8 * (nu + 1) + per_edge * m for nu, nl, m in sizes), "flops": 0}


# --- exact values of the small cases -----------------------------------------

def _supports(a):
    """Support of each pair of the dense 0/1 matrix a (where it is 1)."""
    return ((a @ a.T) @ a - a.sum(1, keepdim=True) - a.sum(0, keepdim=True) + 1) * a


def exact(case, seed):
    if case["call"] not in ("support", "noalloc", "decompose", "pc") or case["m"] > 250_000:
        return None
    nu, nl, m = _single_size(case)
    if nu * nl > 300_000_000:
        return None
    g = _graph(case, seed)
    rows = torch.repeat_interleave(torch.arange(nu, device=DEV), torch.diff(g.row_ptr))
    cols = g.col.to(torch.int64)
    a = torch.zeros(nu, nl, dtype=torch.float64, device=DEV)
    a[rows, cols] = 1.0
    s = _supports(a)
    sup = s[rows, cols].round().to(torch.int64)
    if case["call"] in ("support", "noalloc"):
        return [sup, int(sup.sum().item()) // 4]
    if m > 12_000 or case["shape"] != "uniform":
        return [sup, None]
    # Remove every pair of support at most k, again and again, for k = 0, 1, ...
    phi = torch.zeros_like(a)
    k = 0.0
    while bool(a.any()):
        low = (a > 0) & (s < k + 0.5)
        if bool(low.any()):
            phi[low] = k
            a[low] = 0.0
            s = _supports(a)
        else:
            k += 1
    return [sup, phi[rows, cols].round().to(torch.int64)]
