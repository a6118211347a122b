"""The calls whose speed matters to a user of the library, as cases that can be timed.

Every case goes through the Python binding: one graph counted or enumerated, a batch of
graphs, or requests put to a server.  Graphs are drawn with numpy from the seed alone, in the
families the repository's workloads use: Erdos-Renyi, Chung-Lu power laws (exponent 2.1,
weights capped at sqrt(E / 10)), a dense skewed graph with planted blocks, and graphs with
hubs of more than 1024 neighbours.  The results are whole numbers: counts, 64-bit hashes
(as signed 64-bit values) and record arrays.
"""
import math

import numpy as np
import torch

import paper_2401_05039_amd as mbe


# --------------------------------------------------------------------------------- cases

def listed():
    return [
        # the smallest call: a graph of a few dozen vertices (a membership table), where the
        # fixed cost of a call is what a user waits for
        _count("count tiny, device", "er", n_u=24, n_v=20, edges=99),
        # a small study graph handed over as host arrays, default options
        _count("count er 200x300, host", "er", device=False, n_u=200, n_v=300, edges=3000),
        # the same size listed biclique by biclique into host memory (the binding sizes the
        # buffer itself)
        _enumerate("enumerate er 200x300, host", "er", device=False, n_u=200, n_v=300, edges=3000),
        # a medium sparse interaction graph of odd sizes, by a caller that must not allocate
        _count("count power law 12k, noalloc", "powerlaw", noalloc=True, n_u=12_345, n_v=6_789, edges=123_457),
        # the headline workload: a large sparse power-law graph on the device
        _count("count power law 100k", "powerlaw", n_u=100_000, n_v=50_000, edges=1_000_000),
        # all bicliques of a medium power-law graph written to device memory
        _enumerate("enumerate power law 20k, device", "powerlaw", n_u=20_000, n_v=10_000, edges=200_000),
        # a slice of the top-level candidates of a dense skewed graph (how a graph too heavy for
        # one call is split over calls or devices): few top-level candidates, huge subtrees
        _count("count skewed slice", "skewed", n_u=20_000, n_v=5_000, edges=2_000_000, root_lo=2000, roots=12),
        # hubs with more neighbours than the fixed mask classes hold
        _count("count hubs", "hubs", n_u=1_500, n_v=6_000, edges=40_000, hubs=16, hub_lo=1_100, hub_hi=3_000),
        # the embedded pruning of candidates and the pivot rule, as a user studying them calls them
        _count("count power law 8k, pruned", "powerlaw", prune=1, n_u=8_000, n_v=4_000, edges=80_000),
        _count("count power law 8k, pivot", "powerlaw", prune=2, n_u=8_000, n_v=4_000, edges=80_000),
        # many independent graphs of mixed sizes and densities in one call
        {"name": "batch of 128", "do": "batch", "graphs": 128, "lo": 50, "hi": 800},
        # a burst of requests to a running server, one in ten of them large
        {"name": "serve 40 requests", "do": "serve", "graphs": 40, "lo": 50, "hi": 400, "big": 10_000},
    ]


def draw(rng):
    """One more case of the same ranges."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["count er", "enumerate er", "count power law", "count power law", "enumerate power law",
                       "skewed", "hubs", "prune", "batch", "serve"])
    if kind in ("count er", "enumerate er"):
        n_u, n_v = log_int(20, 400), log_int(20, 400)
        g = dict(family="er", n_u=n_u, n_v=n_v, edges=max(1, int(n_u * n_v * rng.uniform(0.01, 0.06))))
        device = rng.random() < 0.5
        if kind == "count er":
            return {"do": "count", "device": device, "noalloc": rng.random() < 0.3, **g}
        return {"do": "enumerate", "device": device, **g}
    if kind in ("count power law", "enumerate power law"):
        n_u = log_int(1_000, 100_000 if kind == "count power law" else 20_000)
        g = dict(family="powerlaw", n_u=n_u, n_v=int(n_u * rng.uniform(0.4, 0.7)), edges=int(n_u * rng.uniform(5, 10)))
        if kind == "count power law":
            return {"do": "count", "device": rng.random() < 0.7, "steal_k": rng.choice([0, 0, 3]),
                    "noalloc": n_u < 15_000 and rng.random() < 0.3, **g}
        return {"do": "enumerate", "device": True, **g}
    if kind == "skewed":
        return {"do": "count", "device": True, "family": "skewed", "n_u": 20_000, "n_v": 5_000, "edges": 2_000_000,
                "root_lo": rng.randrange(1500, 4500), "roots": log_int(1, 8)}
    if kind == "hubs":
        return {"do": "count", "device": rng.random() < 0.5, "family": "hubs", "n_u": log_int(200, 1_500),
                "n_v": rng.randrange(4_000, 6_001), "edges": log_int(5_000, 40_000), "hubs": rng.randrange(2, 17),
                "hub_lo": 1_025, "hub_hi": rng.randrange(1_100, 3_000)}
    if kind == "prune":
        n_u = log_int(500, 8_000)
        return {"do": "count", "device": True, "family": "powerlaw", "prune": rng.choice([1, 2]), "n_u": n_u,
                "n_v": int(n_u * rng.uniform(0.4, 0.6)), "edges": int(n_u * rng.uniform(5, 10))}
    if kind == "batch":
        return {"do": "batch", "graphs": log_int(4, 128), "lo": 50, "hi": log_int(100, 800)}
    return {"do": "serve", "graphs": log_int(4, 40), "lo": 50, "hi": log_int(100, 400), "big": log_int(2_000, 10_000)}


def _count(name, family, device=True, **kw):
    return {"name": name, "do": "count", "family": family, "device": device, **kw}


def _enumerate(name, family, device=True, **kw):
    return {"name": name, "do": "enumerate", "family": family, "device": device, **kw}


# -------------------------------------------------------------------------------- graphs

class Graph:
    """A bipartite graph as the two sorted CSR arrays the binding takes."""

    def __init__(self, n_u, n_v, u_off, u_adj, v_off, v_adj):
        self.n_u, self.n_v = n_u, n_v
        self.u_off, self.u_adj, self.v_off, self.v_adj = u_off, u_adj, v_off, v_adj

    def cuda(self):
        return Graph(self.n_u, self.n_v, *[torch.from_numpy(a).cuda() for a in
                                           (self.u_off, self.u_adj, self.v_off, self.v_adj)])


def _from_keys(n_u, n_v, keys):
    """The graph of the distinct edges u * n_v + v."""
    def csr(n, rows, cols):
        off = np.zeros(n + 1, dtype=np.int32)
        np.cumsum(np.bincount(rows, minlength=n), out=off[1:])
        return off, cols.astype(np.int32)

    keys = np.sort(keys)
    u, v = keys // n_v, keys % n_v
    back = np.sort(v * n_u + u)
    return Graph(n_u, n_v, *csr(n_u, u, v), *csr(n_v, back // n_u, back % n_u))


def _distinct(sample, m):
    """m distinct edges in the order they were first drawn."""
    keys = np.zeros(0, dtype=np.int64)
    while keys.size < m:
        keys = np.concatenate([keys, sample(int((m - keys.size) * 1.1) + 64)])
        _, first = np.unique(keys, return_index=True)
        keys = keys[np.sort(first)]
    return keys[:m]


def _er(rng, n_u, n_v, m):
    return _distinct(lambda k: rng.integers(0, n_u * n_v, k), min(m, n_u * n_v // 2))


def _weights(n, gamma, total, cap):
    """Power-law weights that sum to total, none above cap."""
    w = np.arange(1, n + 1, dtype=np.float64) ** (-1.0 / (gamma - 1.0))
    w *= total / w.sum()
    for _ in range(100):
        over = w >= cap
        rest = total - cap * over.sum()
        if not (w > cap).any() or rest <= 0 or over.all():
            break
        w[over] = cap
        w[~over] *= rest / w[~over].sum()
    return np.minimum(w, cap)


def _power_law(rng, n_u, n_v, m, gamma=2.1):
    cap = float(math.isqrt(max(m // 10, 1)))
    cdf = []
    for n, c in ((n_u, min(cap, n_v)), (n_v, min(cap, n_u))):
        s = np.cumsum(_weights(n, gamma, m, c))
        cdf.append(s / s[-1])
    pu, pv = rng.permutation(n_u), rng.permutation(n_v)

    def sample(k):
        u = np.minimum(np.searchsorted(cdf[0], rng.random(k), side="right"), n_u - 1)
        v = np.minimum(np.searchsorted(cdf[1], rng.random(k), side="right"), n_v - 1)
        return pu[u] * n_v + pv[v]
    return _distinct(sample, m)


def _skewed(rng, n_u, n_v, m):
    """A dense power-law background and 50 planted complete blocks."""
    blocks = []
    for _ in range(50):
        a, b = rng.integers(10, 41, 2)
        us, vs = rng.choice(n_u, a, replace=False), rng.choice(n_v, b, replace=False)
        blocks.append((us[:, None] * n_v + vs[None, :]).ravel())
    return np.unique(np.concatenate([_power_law(rng, n_u, n_v, m, gamma=1.9)] + blocks))


def _hubs(rng, n_u, n_v, m, hubs, lo, hi):
    """A sparse background and, on the candidate side, hubs of lo to hi neighbours."""
    keys = [_er(rng, n_u, n_v, m)]
    for u in rng.choice(n_u, hubs, replace=False):
        keys.append(u * n_v + rng.choice(n_v, int(rng.integers(lo, hi + 1)), replace=False))
    return np.unique(np.concatenate(keys))


def _graph(case, rng):
    n_u, n_v, m = case["n_u"], case["n_v"], case["edges"]
    keys = {"er": lambda: _er(rng, n_u, n_v, m), "powerlaw": lambda: _power_law(rng, n_u, n_v, m),
            "skewed": lambda: _skewed(rng, n_u, n_v, m),
            "hubs": lambda: _hubs(rng, n_u, n_v, m, case["hubs"], case["hub_lo"], case["hub_hi"])}[case["family"]]()
    g = _from_keys(n_u, n_v, keys)
    return g.cuda() if case["device"] else g


def _mixed(case, rng):
    """Graphs of mixed sizes (log-uniform in [lo, hi]) and densities, half of them power laws;
    where the case has large ones, every tenth is a power law of up to that many vertices."""
    out = []
    for i in range(case["graphs"]):
        if case.get("big") and i % 10 == 5:
            n_u = int(round(math.exp(rng.uniform(math.log(case["big"] / 4), math.log(case["big"])))))
            out.append(_from_keys(n_u, n_u // 2, _power_law(rng, n_u, n_u // 2, 10 * n_u)))
            continue
        n_u, n_v = (int(round(math.exp(x))) for x in rng.uniform(math.log(case["lo"]), math.log(case["hi"]), 2))
        m = max(1, int(rng.uniform(0.01, 0.1) * n_u * n_v))
        out.append(_from_keys(n_u, n_v, (_er if rng.random() < 0.5 else _power_law)(rng, n_u, n_v, m)))
    return out


# ------------------------------------------------------------------------- prepare and run

_server = None


def _the_server():
    """One server for the whole process, as a serving program has."""
    global _server
    if _server is None:
        _server = mbe.Server(hbm_budget_bytes=16 << 30)
    return _server


def prepare(case, seed):
    rng = np.random.default_rng(seed)
    state = {"case": case}
    if case["do"] == "batch":
        state["graphs"] = _mixed(case, rng)
    elif case["do"] == "serve":
        state["graphs"] = _mixed(case, rng)
        state["server"] = _the_server()
    else:
        state["graph"] = _graph(case, rng)
        state["options"] = mbe.Options(root_lo=case.get("root_lo", 0),
                                       root_hi=case.get("root_lo", 0) + case["roots"] if case.get("roots") else 0,
                                       steal_k=case.get("steal_k", 0), prune=case.get("prune", 0))
        if case["do"] == "enumerate":
            # room for the records, more than these graphs have: on the device the buffer they
            # are written to, on the host where the program gathers them
            room = 48 * case["edges"] + 1024
            state["records"] = (torch.zeros(room, dtype=torch.int32, device="cuda") if case["device"]
                                else np.zeros(room, dtype=np.int32))
    return state


def _answer(r):
    h = r["hash"]
    return [r["count"], h - (1 << 64) if h >= 1 << 63 else h, r["out_ints"], r["side"]]


def run(state):
    case = state["case"]
    if case["do"] == "batch":
        return np.array([_answer(r) for r in mbe.mbe_count_batch(state["graphs"])], dtype=np.int64)
    if case["do"] == "serve":
        tickets = [state["server"].submit(g) for g in state["graphs"]]
        return np.array([_answer(state["server"].wait(t)[0]) for t in tickets], dtype=np.int64)
    if case["do"] == "enumerate":
        kept = state["records"]
        if case["device"]:
            r, _ = mbe.mbe_enumerate(state["graph"], state["options"], out=kept)
        else:
            r, records = mbe.mbe_enumerate(state["graph"], state["options"])
            kept[:len(records)] = records
        return {"answer": _answer(r), "records": kept}
    count = mbe.mbe_count_noalloc if case.get("noalloc") else mbe.mbe_count
    return {"answer": _answer(count(state["graph"], state["options"]))}


def work(case):
    """The CSR arrays read once, the answers written once (the records that an enumeration
    writes depend on the graph and are left out)."""
    if case["do"] in ("batch", "serve"):
        # of a log-uniform size: the mean of n, and of n squared (two independent sides)
        span = math.log(case["hi"] / case["lo"])
        mean = (case["hi"] - case["lo"]) / span
        n, big = case["graphs"], case["graphs"] // 10 if case.get("big") else 0
        edges, ends = (n - big) * 0.055 * mean * mean, (n - big) * 2 * mean
        if big:
            size = 0.75 * case["big"] / math.log(4)
            edges, ends = edges + big * 10 * size, ends + big * 1.5 * size
        return {"bytes": 4.0 * (2 * edges + ends) + 32.0 * n, "flops": 0.0}
    edges = case["edges"]
    if case["family"] == "hubs":
        edges += case["hubs"] * (case["hub_lo"] + case["hub_hi"]) / 2
    return {"bytes": 4.0 * (2 * edges + case["n_u"] + case["n_v"] + 2) + 32.0, "flops": 0.0}


# ---------------------------------------------------------------------------------- exact

def _mix(z):
    mask = (1 << 64) - 1
    z ^= z >> 30
    z = z * 0xBF58476D1CE4E5B9 & mask
    z ^= z >> 27
    z = z * 0x94D049BB133111EB & mask
    return z ^ z >> 31


def exact(case, seed):
    """For the small Erdos-Renyi graphs: the maximal bicliques from their definition, B being
    every intersection of rows of U and A all vertices that hold it."""
    if case.get("family") != "er":
        return None
    mask, k = (1 << 64) - 1, 0x9E3779B97F4A7C15
    g = _graph({**case, "device": False}, np.random.default_rng(seed))
    rows = [g.u_adj[g.u_off[u]:g.u_off[u + 1]].tolist() for u in range(g.n_u)]
    bits = [sum(1 << v for v in r) for r in rows]
    sides = set()
    for b in bits:
        sides |= {b & s for s in sides} | {b}
        sides.discard(0)
        if len(sides) > 200_000:
            return None
    found, total = [], 0
    for s in sides:
        a = [u for u in range(g.n_u) if bits[u] & s == s]
        b = [v for v in range(g.n_v) if s >> v & 1]
        hb = sum(_mix(k * (2 * v + 2) & mask) for v in b)
        total += _mix(sum(_mix(k * (2 * u + 1) & mask) for u in a) + _mix(hb + k & mask) & mask)
        found.append((a, b))
    found.sort()
    records = [x for a, b in found for x in (len(a), len(b), *a, *b)]
    answer = _answer({"count": len(found), "hash": total & mask, "out_ints": len(records),
                      "side": 2 if g.n_v < g.n_u else 1})
    if case["do"] == "enumerate":
        room = 48 * case["edges"] + 1024
        return {"answer": answer, "records": np.array(records + [0] * (room - len(records)), dtype=np.int32)}
    return {"answer": answer}
