"""GPU parity of skim_build_sketches against the CPU oracle (bit-exact sketches,
sizes and estimates), on random small graphs, the tiny config, a mid-size
power-law graph spanning many rank windows, edge cases, invalid inputs, and
the full 1M-node Chung-Lu configuration."""
import numpy as np
import pytest

from workloads import from_edges
from workloads.configs import make_config, make_graph
from brute import random_small_graph
from gpu_util import gpu_build, log

pytestmark = pytest.mark.gpu

THRS = [0xFFFFFFFF, 0xFFFFFFFF // 2, 0xFFFFFFFF // 4, 0xFFFFFFFF // 20]


def _check(oracle_lib, g, ell, k, seed):
    R, S, E, work, _ = gpu_build(g, ell, k, seed)
    R0, S0, _ = oracle_lib.build_alg2(g, seed, ell, k)
    E0 = oracle_lib.estimates(R0, S0, k, ell)
    assert np.array_equal(R, R0), "sketch ranks differ"
    assert np.array_equal(S, S0), "sketch sizes differ"
    assert np.array_equal(E, E0), "estimates differ"  # IEEE, same operation order
    return work


@pytest.mark.parametrize("ell,k", [(1, 2), (2, 3), (16, 4), (16, 16), (64, 64), (7, 5), (64, 256)])
def test_random_small_graphs(oracle_lib, ell, k):
    rng = np.random.default_rng(1000 * ell + k)
    for trial in range(6):
        n = int(rng.integers(1, 60))
        m = int(rng.integers(0, 4 * n)) if n > 1 else 0
        src, dst, thr = random_small_graph(rng, n, m, THRS) if n > 1 else ([], [], [])
        g = from_edges(n, src, dst, thr if len(src) else None)
        seed = int(rng.integers(0, 2 ** 63))
        log(f"random graph ell={ell} k={k} trial={trial} n={n} m={g.m} seed={seed}")
        _check(oracle_lib, g, ell, k, seed)


def test_tiny_config(oracle_lib):
    cfg = make_config("tiny-ic")
    g = make_graph(cfg)
    log("tiny-ic")
    work = _check(oracle_lib, g, cfg["ell"], cfg["k"], cfg["seed"])
    assert work["windows"] >= 1


def test_deterministic_graph_and_no_edges(oracle_lib):
    rng = np.random.default_rng(3)
    src, dst, _ = random_small_graph(rng, 200, 900, [0xFFFFFFFF])
    log("p=1 graph")
    _check(oracle_lib, from_edges(200, src, dst, 0xFFFFFFFF), 8, 16, 5)
    log("no edges")
    _check(oracle_lib, from_edges(300, [], []), 16, 8, 6)


def test_deep_path_many_levels(oracle_lib):
    # a p=1 path of 3000 nodes: reverse searches 3000 levels deep
    n = 3000
    g = from_edges(n, list(range(n - 1)), list(range(1, n)), 0xFFFFFFFF)
    log("deep path")
    _check(oracle_lib, g, 4, 8, 11)


def test_powerlaw_many_windows(oracle_lib):
    from workloads.graphs import Graph, chung_lu_graph, wc_thresholds
    rp, col = chung_lu_graph(20000, 320000, 2.1, 55)
    g = Graph(20000, rp, col, wc_thresholds(rp, col, 20000))
    log("chung-lu 20k wc l=64 k=64")
    work = _check(oracle_lib, g, 64, 64, 1)
    log(f"work {work}")
    assert work["windows"] >= 4 and work["restarts"] == 0
    log("chung-lu 20k uniform p=0.1 l=32 k=16")
    g2 = Graph(20000, rp, col, np.full(col.size, 0xFFFFFFFF // 10, dtype=np.uint32))
    _check(oracle_lib, g2, 32, 16, 2)


def test_hub_lists_spread_over_the_grid(oracle_lib):
    # live in-lists longer than 4096 entries (a p = 1 in-star of 6000
    # leaves into a hub, the hub feeding a chain, plus random p = 1/2 edges):
    # the searches from the chain visit the hub and expand its list on the
    # whole grid (k_expand_heavy) as well as in the tails and levels
    rng = np.random.default_rng(77)
    leaves, chain = 6000, 300
    n = 1 + leaves + chain
    src = list(range(1, leaves + 1)) + [0] + list(range(leaves + 1, n - 1))
    dst = [0] * leaves + [leaves + 1] + list(range(leaves + 2, n))
    thr = [0xFFFFFFFF] * len(src)
    extra = 20000
    es, ed = rng.integers(0, n, extra), rng.integers(0, n, extra)
    seen = set(zip(src, dst))
    for a, b in zip(es.tolist(), ed.tolist()):
        if a != b and (a, b) not in seen:
            seen.add((a, b))
            src.append(a)
            dst.append(b)
            thr.append(0xFFFFFFFF // 2)
    g = from_edges(n, src, dst, thr)
    for ell, k, seed in ((64, 16, 5), (8, 64, 6)):
        log(f"hub lists n={n} m={g.m} l={ell} k={k}")
        _check(oracle_lib, g, ell, k, seed)


def test_medium_lists_spread_over_the_workgroup(oracle_lib):
    # live in-lists of 17 to 4096 sources (p = 1 in-stars of 20 to 3000
    # leaves into 12 hubs that feed each other) next to short random lists:
    # a workgroup lays a chunk's long lists end to end, a wave its entries'
    # short ones
    rng = np.random.default_rng(78)
    sizes = [20, 33, 64, 100, 257, 300, 511, 700, 1000, 1500, 2048, 3000]
    hubs = len(sizes)
    n = hubs + sum(sizes)
    src, dst, thr = [], [], []
    nxt = hubs
    for h, sz in enumerate(sizes):
        for leaf in range(nxt, nxt + sz):
            src.append(leaf)
            dst.append(h)
            thr.append(0xFFFFFFFF)
        nxt += sz
        src.append(h)
        dst.append((h + 1) % hubs)
        thr.append(0xFFFFFFFF // 2)
    seen = set(zip(src, dst))
    for a, b in zip(rng.integers(0, n, 3 * n).tolist(), rng.integers(0, n, 3 * n).tolist()):
        if a != b and (a, b) not in seen:
            seen.add((a, b))
            src.append(a)
            dst.append(b)
            thr.append(0xFFFFFFFF // 3)
    g = from_edges(n, src, dst, thr)
    for ell, k, seed in ((64, 16, 8), (16, 64, 9)):
        log(f"medium lists n={n} m={g.m} l={ell} k={k}")
        _check(oracle_lib, g, ell, k, seed)


def test_deterministic_repeat():
    cfg = make_config("tiny-ic")
    g = make_graph(cfg)
    a = gpu_build(g, 16, 16, 1)
    b = gpu_build(g, 16, 16, 1)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[2], b[2])


@pytest.mark.parametrize("bad", ["unsorted", "duplicate", "self_loop", "head_range", "row_ptr"])
def test_invalid_graph_rejected(bad):
    import torch
    import paper_1408_6282_amd as sk
    from workloads.graphs import Graph
    rp = np.array([0, 2, 3, 3], dtype=np.uint64)
    col = np.array([1, 2, 2], dtype=np.uint32)
    if bad == "unsorted":
        col = np.array([2, 1, 2], dtype=np.uint32)
    elif bad == "duplicate":
        col = np.array([1, 1, 2], dtype=np.uint32)
    elif bad == "self_loop":
        col = np.array([0, 2, 2], dtype=np.uint32)
    elif bad == "head_range":
        col = np.array([1, 7, 2], dtype=np.uint32)
    elif bad == "row_ptr":
        rp = np.array([0, 3, 2, 3], dtype=np.uint64)
    g = Graph(3, rp, col, np.full(3, 0xFFFFFFFF, dtype=np.uint32))
    G = sk.DeviceGraph.from_host(g, "cuda:0")
    ranks = torch.full((3 * 4,), 7, dtype=torch.int64, device="cuda:0")
    size = torch.full((3,), 7, dtype=torch.int32, device="cuda:0")
    with pytest.raises(sk.SkimError) as ei:
        sk.skim_build_sketches(G, 4, 4, 1, ranks, size)
    assert ei.value.status == sk.SKIM_EINVAL
    assert (ranks.cpu() == 7).all() and (size.cpu() == 7).all()  # outputs untouched


def test_bad_parameters():
    import torch
    import paper_1408_6282_amd as sk
    g = from_edges(4, [0], [1])
    G = sk.DeviceGraph.from_host(g, "cuda:0")
    ranks = torch.empty(4 * 4, dtype=torch.int64, device="cuda:0")
    size = torch.empty(4, dtype=torch.int32, device="cuda:0")
    for ell, k in [(0, 4), (65, 4), (4, 1), (4, 257)]:
        with pytest.raises(sk.SkimError) as ei:
            sk.skim_build_sketches(G, ell, k, 1, ranks, size)
        assert ei.value.status == sk.SKIM_EINVAL


# Launch shapes of the full-size parity runs: the defaults, the shapes the
# autotuner picks on this workload (the launch the bench times), the widest
# windows and batches, every level by pull, and pull from 2^21 entries.
CL_SHAPES = {
    "default": None,
    "tuned": dict(small_frontier=262144, small_batch=16, large_batch=2, thread_frontier=524288,
                  heavy_visits=4, sort_frontier=0, window_span=3, first_span=5),
    "wide": dict(small_frontier=1 << 24, small_batch=64, large_batch=64, thread_frontier=1 << 30,
                 heavy_visits=1000, sort_frontier=0, window_span=8, first_span=16),
    "pull": dict(pull_frontier=1),
    "pull-2m": dict(pull_frontier=1 << 21),
}


@pytest.fixture(scope="module")
def chung_lu_1m():
    cfg = make_config("chung-lu-1m")
    log("generating chung-lu-1m")
    return cfg, make_graph(cfg)


@pytest.mark.slow
@pytest.mark.parametrize("shape", list(CL_SHAPES))
def test_chung_lu_1m_full_parity(chung_lu_1m, shape):
    # every sketch, size and estimate of the full workload equals the
    # oracle's Algorithm 2 (by the digests its committed script stored)
    import paper_1408_6282_amd as sk
    from gpu_util import check_digests, golden
    cfg, g = chung_lu_1m
    sk.skim_set_build_params(CL_SHAPES[shape])
    try:
        log(f"gpu build chung-lu-1m, {shape} shapes")
        R, S, E, work, _ = gpu_build(g, cfg["ell"], cfg["k"], cfg["seed"])
    finally:
        sk.skim_set_build_params(None)
    log(f"gpu work {work}")
    check_digests(golden("chung_lu_1m"), g, R, S, E)


@pytest.mark.parametrize("n,deg,denom,ell,k,hub", [
    (300, 6, 1, 64, 256, False),     # one word to eight, every pair reaches every source
    (2000, 8, 2, 64, 32, True),      # a hub: in-lists cut into chunks, two and more
    (2000, 8, 2, 7, 64, False),      # few instances
    (9001, 8, 2, 1, 64, False),      # one instance
    (20000, 6, 2, 33, 16, True),     # several nodes per workgroup and round
])
def test_dense_windows(oracle_lib, n, deg, denom, ell, k, hub):
    """Graphs whose optimistic first window overflows: the windows after it
    keep their sources as bit sets per pair."""
    rng = np.random.default_rng(n + k)
    e = rng.integers(0, n, size=(deg * n, 2))
    if hub:
        e = np.concatenate([e, np.stack([np.arange(1, n), np.zeros(n - 1, dtype=np.int64)], 1)])
    e = np.unique(e, axis=0)
    e = e[e[:, 0] != e[:, 1]]
    g = from_edges(n, e[:, 0], e[:, 1], 0xFFFFFFFF // denom)
    log(f"dense windows n={n} m={g.m} ell={ell} k={k} hub={hub}")
    R, S, E, work, _ = gpu_build(g, ell, k, 5)
    assert work["restart_flags"] & 16, "the first window was meant to overflow"
    wr, ws, _ = oracle_lib.build_alg2(g, 5, ell, k)
    assert np.array_equal(S, ws)
    assert np.array_equal(R, wr)
    assert np.array_equal(E, oracle_lib.estimates(wr, ws, k, ell))
    R2, _, _, _, _ = gpu_build(g, ell, k, 5)
    assert np.array_equal(R, R2)


@pytest.mark.parametrize("n,fan,denom,ell,k", [
    (400, 64, 1, 4, 8),      # in-lists of one step of a wave
    (400, 65, 1, 4, 8),      # ... and cut after it
    (3000, 400, 1, 64, 64),  # cut several times, more entries than a stack holds
    (3000, 130, 3, 16, 16),
])
def test_tails_lists_and_stacks(oracle_lib, n, fan, denom, ell, k):
    """Small frontiers that meet long in-lists: a cycle whose every 50th node
    has `fan` in-edges."""
    rng = np.random.default_rng(fan)
    e = [np.stack([np.arange(n), (np.arange(n) + 1) % n], 1)]
    for v in range(0, n, 50):
        e.append(np.stack([rng.choice(n, fan, replace=False), np.full(fan, v)], 1))
    e = np.unique(np.concatenate(e), axis=0)
    e = e[e[:, 0] != e[:, 1]]
    g = from_edges(n, e[:, 0], e[:, 1], 0xFFFFFFFF // denom)
    log(f"tails n={n} fan={fan} ell={ell} k={k}")
    _check(oracle_lib, g, ell, k, 9)


@pytest.mark.parametrize("ell,k", [(4, 256), (64, 16), (16, 64)])
def test_select_segment_sizes(oracle_lib, ell, k):
    """Nodes of every record count about the sizes where the selection changes
    its sort (64, 128, 256, 512 records), and of a few thousand."""
    rng = np.random.default_rng(ell)
    n = 1600
    fans = [14, 15, 16, 17, 30, 31, 32, 33, 62, 63, 64, 65, 126, 127, 128, 129, 200, 255, 256, 257,
            400, 511, 512, 513, 700, 1500]
    e = np.concatenate([np.stack([rng.choice(np.arange(len(fans), n), f, replace=False),
                                  np.full(f, v)], 1) for v, f in enumerate(fans)])
    g = from_edges(n, e[:, 0], e[:, 1], 0xFFFFFFFF)
    log(f"segment sizes ell={ell} k={k}")
    _check(oracle_lib, g, ell, k, 21)


@pytest.mark.parametrize("n", [1, 2, 4095, 4096, 4097, 32767, 32769])
def test_scan_sizes(oracle_lib, n):
    """Node counts at the edges of the single-workgroup prefix sum's rounds and
    of its range."""
    src = np.arange(0, n - 1, 3)
    g = from_edges(n, src, src + 1, 0xFFFFFFFF)
    log(f"scan sizes n={n}")
    _check(oracle_lib, g, 2, 4, 3)


def test_dense_windows_count_the_same_work():
    # windows of source bit sets report the visits and live-edge scans of the
    # per-source search (out-lists for pulled levels keep the build to that one;
    # no level is long enough to be pulled)
    import paper_1408_6282_amd as sk
    from workloads.graphs import Graph, rmat_graph, trivalency_thresholds
    rp, col = rmat_graph(14, 1 << 18, (0.57, 0.19, 0.19, 0.05), 5)
    g = Graph(1 << 14, rp, col, trivalency_thresholds(col.size, 5))
    try:
        sk.skim_timing_reset()
        sk.skim_timing_enable("k_dense_level")
        sk.skim_set_build_params(dict(first_span=1))
        R, S, _, work, _ = gpu_build(g, 64, 32, 3)
        dense = sk.skim_timing_read("k_dense_level")[1]
        sk.skim_timing_reset()
        sk.skim_set_build_params(dict(pull_frontier=0xFFFFFFFF))
        R0, S0, _, work0, _ = gpu_build(g, 64, 32, 3)
        assert dense and not sk.skim_timing_read("k_dense_level")[1]
    finally:
        sk.skim_timing_enable(None)
        sk.skim_set_build_params(None)
    log(f"work {work} by source {work0}")
    assert np.array_equal(R, R0) and np.array_equal(S, S0)
    assert work["visits"] == work0["visits"] and work["scans"] == work0["scans"]


@pytest.mark.parametrize("n,fan,denom,ell,k", [
    (2000, 512, 1, 4, 8),    # the longest list a wave of the tails walks by itself
    (2000, 513, 1, 4, 8),    # ... and past it
    (2500, 1200, 2, 16, 16),
    (3000, 300, 1, 16, 4),   # stacks that fill in few steps
])
def test_tails_hand_back_hubs_and_full_stacks(oracle_lib, n, fan, denom, ell, k):
    """Small frontiers that meet hubs, as in-lists (every 100th node of a cycle) and
    as sources all over: what the tails hand back goes on level by level."""
    rng = np.random.default_rng(n + fan)
    e = [np.stack([np.arange(n), (np.arange(n) + 1) % n], 1)]
    for v in range(0, n, 100):
        e.append(np.stack([rng.choice(n, fan, replace=False), np.full(fan, v)], 1))
        e.append(np.stack([np.full(20, v), rng.choice(n, 20, replace=False)], 1))
    e = np.unique(np.concatenate(e), axis=0)
    e = e[e[:, 0] != e[:, 1]]
    g = from_edges(n, e[:, 0], e[:, 1], 0xFFFFFFFF // denom)
    log(f"tails hand back n={n} fan={fan} ell={ell} k={k}")
    _check(oracle_lib, g, ell, k, 9)


def test_no_dense_windows_where_pairs_are_full():
    # few visits are left once the core's pairs hold k: those windows search by
    # source (the first windows of this graph visit a pair five times on average)
    import paper_1408_6282_amd as sk
    from workloads.graphs import Graph, rmat_graph, trivalency_thresholds
    rp, col = rmat_graph(15, 1 << 17, (0.57, 0.19, 0.19, 0.05), 5)
    g = Graph(1 << 15, rp, col, trivalency_thresholds(col.size, 5))
    try:
        sk.skim_timing_reset()
        sk.skim_timing_enable("k_dense_seed")
        _, _, _, work, _ = gpu_build(g, 32, 7, 5)
        dense = sk.skim_timing_read("k_dense_seed")[1]
    finally:
        sk.skim_timing_enable(None)
    log(f"work {work}, dense windows {dense}")
    assert work["restarts"] or dense == 0


def test_build_with_an_allocation_failing():
    # each allocation of a build with dense windows fails in turn: the call
    # returns SKIM_ENOMEM with its outputs untouched or, from the bit sets on,
    # makes the same sketches without them
    import torch
    import paper_1408_6282_amd as sk
    from workloads.graphs import Graph, rmat_graph, trivalency_thresholds
    rp, col = rmat_graph(14, 1 << 18, (0.57, 0.19, 0.19, 0.05), 5)
    g = Graph(1 << 14, rp, col, trivalency_thresholds(col.size, 5))
    G = sk.DeviceGraph.from_host(g, "cuda:0")
    ell, k = 64, 32
    ranks = torch.empty(g.n * k, dtype=torch.int64, device="cuda:0")
    size = torch.empty(g.n, dtype=torch.int32, device="cuda:0")

    def build(nth):
        ranks.fill_(7)
        size.fill_(7)
        sk.skim_timing_reset()
        sk.skim_debug_inject(sk.SKIM_FAULT_ALLOC_NTH, nth)
        try:
            sk.skim_build_sketches(G, ell, k, 3, ranks, size)
            ok = True
        except sk.SkimError as e:
            assert e.status == sk.SKIM_ENOMEM
            ok = False
        finally:
            sk.skim_debug_inject(sk.SKIM_FAULT_ALLOC_NTH, 0)
        torch.cuda.synchronize()
        return ok, sk.skim_timing_read("k_dense_seed")[1]

    try:
        sk.skim_set_build_params(dict(first_span=1))
        sk.skim_timing_enable("k_dense_seed")
        ok, dense = build(0)
        assert ok and dense
        wr, ws = ranks.clone(), size.clone()
        refused, without = 0, 0
        for nth in range(1, 120):
            log(f"build with allocation {nth} failing")
            ok, d = build(nth)
            if ok:
                assert torch.equal(ranks, wr) and torch.equal(size, ws), nth
                without += d < dense
            else:
                assert (ranks == 7).all() and (size == 7).all(), nth
                refused += 1
        assert refused and without
    finally:
        sk.skim_timing_enable(None)
        sk.skim_set_build_params(None)
