"""GPU parity of skim_query_batch against the oracle: bottom-k and Cohen-Kaplan
estimators, batched and one-launch-per-query paths (identical bits), set
semantics, per-query status, and a sample of the batched lognormal workload."""
import numpy as np
import pytest

from workloads import from_edges, lognormal_query_sets, uniform_query_sets
from workloads.configs import make_config, make_graph
from brute import random_small_graph
from gpu_util import gpu_build, gpu_query, log

pytestmark = pytest.mark.gpu


def _sets(sets):
    off = np.zeros(len(sets) + 1, dtype=np.uint64)
    off[1:] = np.cumsum([len(s) for s in sets])
    nodes = np.array([x for s in sets for x in s], dtype=np.uint32)
    return off, nodes


@pytest.fixture(scope="module")
def tiny(oracle_lib):
    cfg = make_config("tiny-ic")
    g = make_graph(cfg)
    R, S, E, _, (rt, st) = gpu_build(g, cfg["ell"], cfg["k"], cfg["seed"])
    return cfg, g, R, S, rt, st


def test_single_node_queries(oracle_lib, tiny):
    cfg, g, R, S, rt, st = tiny
    off = np.arange(g.n + 1, dtype=np.uint64)
    nodes = np.arange(g.n, dtype=np.uint32)
    for estimator, fn in [(0, oracle_lib.union_query), (1, oracle_lib.ck_query)]:
        want, _ = fn(R, S, cfg["k"], cfg["ell"], off, nodes)
        got, status = gpu_query(rt, st, g.n, cfg["k"], cfg["ell"], off, nodes, estimator)
        assert np.array_equal(got, want) and (status == 0).all()


@pytest.mark.parametrize("estimator", [0, 1])
def test_random_sets_batched_and_plain(oracle_lib, tiny, estimator):
    cfg, g, R, S, rt, st = tiny
    off, nodes = uniform_query_sets(600, g.n, 17, 1, 512)
    fn = oracle_lib.union_query if estimator == 0 else oracle_lib.ck_query
    want, _ = fn(R, S, cfg["k"], cfg["ell"], off, nodes)
    got, status = gpu_query(rt, st, g.n, cfg["k"], cfg["ell"], off, nodes, estimator, mode=0)
    plain, _ = gpu_query(rt, st, g.n, cfg["k"], cfg["ell"], off, nodes, estimator, mode=1)
    assert (status == 0).all()
    assert np.array_equal(got, want)
    assert np.array_equal(plain, got)


def test_set_semantics_and_status(oracle_lib, tiny):
    cfg, g, R, S, rt, st = tiny
    sets = [[], [3, 3, 3], [3], [1, 5000], [2, 0], list(range(1000)), [999, 0, 999]]
    off, nodes = _sets(sets)
    for estimator in (0, 1):
        got, status = gpu_query(rt, st, g.n, cfg["k"], cfg["ell"], off, nodes, estimator)
        assert got[0] == 0.0 and status[0] == 0
        assert got[1] == got[2]
        assert status[3] == -1 and got[3] == 0.0
        assert (status[[0, 1, 2, 4, 5, 6]] == 0).all()
        fn = oracle_lib.union_query if estimator == 0 else oracle_lib.ck_query
        want, wst = fn(R, S, cfg["k"], cfg["ell"], off, nodes)
        assert np.array_equal(got, want) and np.array_equal(status, wst)


def test_lognormal_batch_sample(oracle_lib, tiny):
    cfg, g, R, S, rt, st = tiny
    off, nodes = lognormal_query_sets(50_000, g.n, 104)
    want, _ = oracle_lib.union_query(R, S, cfg["k"], cfg["ell"], off, nodes)
    got, status = gpu_query(rt, st, g.n, cfg["k"], cfg["ell"], off, nodes, 0)
    assert (status == 0).all() and np.array_equal(got, want)


def test_random_graph_sketch_shapes(oracle_lib):
    rng = np.random.default_rng(9)
    for ell, k in [(1, 2), (64, 64), (8, 200)]:
        src, dst, thr = random_small_graph(rng, 50, 150, [0xFFFFFFFF // 3, 0xFFFFFFFF])
        g = from_edges(50, src, dst, thr)
        R, S, _, _, (rt, st) = gpu_build(g, ell, k, 3)
        off, nodes = uniform_query_sets(200, 50, 5, 1, 50)
        for estimator, fn in [(0, oracle_lib.union_query), (1, oracle_lib.ck_query)]:
            want, _ = fn(R, S, k, ell, off, nodes)
            got, _ = gpu_query(rt, st, 50, k, ell, off, nodes, estimator)
            log(f"ell={ell} k={k} est={estimator}")
            assert np.array_equal(got, want)


def test_bad_offsets_rejected(tiny):
    import paper_1408_6282_amd as sk
    cfg, g, R, S, rt, st = tiny
    off = np.array([0, 5, 3], dtype=np.uint64)
    nodes = np.arange(5, dtype=np.uint32)
    with pytest.raises(sk.SkimError) as ei:
        gpu_query(rt, st, g.n, cfg["k"], cfg["ell"], off, nodes)
    assert ei.value.status == sk.SKIM_EINVAL


def test_graph_plan_replays_match_batches(oracle_lib, tiny):
    """A captured plan, replayed several times with eager work and
    synchronisations in between, equals the batch call every time; sets
    rewritten in place are answered as rewritten; out-of-order offsets get
    status -3 without touching the sets that do not share them."""
    import torch
    import paper_1408_6282_amd as sk
    from gpu_util import to_dev_u64, to_dev_u32
    cfg, g, R, S, rt, st = tiny
    k, ell = cfg["k"], cfg["ell"]
    off, nodes = uniform_query_sets(500, g.n, 23, 1, 300)
    qo, qn = to_dev_u64(off), to_dev_u32(nodes)
    q = len(off) - 1
    for estimator, fn in [(0, oracle_lib.union_query), (1, oracle_lib.ck_query)]:
        est = torch.empty(q, dtype=torch.float64, device="cuda:0")
        status = torch.empty(q, dtype=torch.int32, device="cuda:0")
        plan = sk.QueryPlan(rt, st, g.n, k, ell, qo, qn, est, status, estimator=estimator)
        want, _ = fn(R, S, k, ell, off, nodes)
        for rep in range(4):
            est.fill_(-1.0)
            plan.launch()
            torch.cuda.synchronize()
            assert np.array_equal(est.cpu().numpy(), want), f"replay {rep}"
            assert (status.cpu().numpy() == 0).all()
            x = torch.arange(1 << 16, device="cuda:0").sum()  # eager work between replays
            torch.cuda.synchronize()
            assert int(x) == (1 << 16) * ((1 << 16) - 1) // 2
        # rewrite the sets in place (same offsets, other nodes)
        rng = np.random.default_rng(estimator)
        nodes2 = nodes.copy()
        for j in range(q):
            a, b = int(off[j]), int(off[j + 1])
            nodes2[a:b] = rng.choice(g.n, b - a, replace=False)
        qn.copy_(to_dev_u32(nodes2))
        plan.launch()
        torch.cuda.synchronize()
        want2, _ = fn(R, S, k, ell, off, nodes2)
        assert np.array_equal(est.cpu().numpy(), want2)
        # break the order of one offset in place
        bad = off.copy()
        bad[7] = bad[8] + 1
        qo.copy_(to_dev_u64(bad))
        plan.launch()
        torch.cuda.synchronize()
        stat = status.cpu().numpy()
        got = est.cpu().numpy()
        assert stat[7] == -3 and got[7] == 0.0  # its end now lies before its start
        # set 6 ends at the moved offset: a valid, longer set
        s6 = nodes2[int(off[6]):int(bad[7])]
        w6, _ = fn(R, S, k, ell, np.array([0, s6.size], dtype=np.uint64), s6)
        assert stat[6] == 0 and got[6] == w6[0]
        good = np.ones(q, dtype=bool)
        good[[6, 7]] = False
        assert (stat[good] == 0).all()
        assert np.array_equal(got[good], want2[good])
        qo.copy_(to_dev_u64(off))
        qn.copy_(to_dev_u32(nodes))
        plan.free()


def _pool_tables(rng, n, k, low_bits):
    """Sorted sketches drawn from a shared pool (so sets overlap), some of them
    short.  low_bits > 0: ranks that share their leading bits and differ only
    in the last `low_bits` (neighbours a truncated key would confuse)."""
    pool = rng.integers(1, 2 ** 63, size=max(4 * k, 40), dtype=np.uint64) * np.uint64(2)
    if low_bits:
        base = np.repeat(pool[:max(2, len(pool) // 8)], 8)[:len(pool)]
        pool = (base & ~np.uint64((1 << low_bits) - 1)) + \
            rng.integers(0, 1 << low_bits, size=len(base), dtype=np.uint64)
    pool = np.unique(pool)
    R = np.full((n, k), 2 ** 64 - 1, dtype=np.uint64)
    S = np.zeros(n, dtype=np.uint32)
    for v in range(n):
        c = int(rng.integers(0, k)) if v % 3 == 0 else k
        c = min(c, len(pool))
        R[v, :c] = np.sort(rng.choice(pool, size=c, replace=False))
        S[v] = c
    return R, S


@pytest.mark.parametrize("k", [2, 15, 16, 17, 32, 33, 64, 65])
@pytest.mark.parametrize("low_bits", [0, 10])
def test_set_sizes_at_class_edges(oracle_lib, k, low_bits):
    """Every size class of both estimators at its edges (lane groups of 2 to 64,
    2 and 4 members a lane, the wave), over the register widths of the sorted
    path, with members repeated; bit for bit, hashed and permutation readings.
    Batches below and above the grid (one query a workgroup; runs of 64)."""
    from gpu_util import to_dev_u32, to_dev_u64
    import torch
    import paper_1408_6282_amd as sk
    rng = np.random.default_rng(100 * k + low_bits)
    n, ell = 300, 8
    R, S = _pool_tables(rng, n, k, low_bits)
    rt, st = to_dev_u64(R.reshape(-1)), to_dev_u32(S)
    edges = [0, 1, 2, 3, 4, 5, 8, 9, 16, 17, 31, 32, 33, 63, 64, 65, 256, 257, 1024, 1025]
    few = [rng.integers(0, n, size=s).tolist() for s in edges] + [[n, 1], [1, 2, n + 5]]
    many = [rng.integers(0, n, size=int(rng.choice(edges[:16]))).tolist() for _ in range(20000)]
    for sets in (few, few + many):
        off, nodes = _sets(sets)
        for estimator, fn in [(0, oracle_lib.union_query), (1, oracle_lib.ck_query)]:
            log(f"classes k={k} low={low_bits} q={len(sets)} est={estimator}")
            want, wst = fn(R, S, k, ell, off, nodes)
            over = np.diff(off.astype(np.int64)) > 1024  # the library's limit, not the oracle's
            want, wst = np.where(over, 0.0, want), np.where(over, -2, wst)
            got, status = gpu_query(rt, st, n, k, ell, off, nodes, estimator)
            assert np.array_equal(status, wst)
            assert np.array_equal(got, want)
    # permutation positions: small integers (below 2^32)
    P = np.where(R == np.uint64(2 ** 64 - 1), R, (R >> np.uint64(44)) + np.uint64(2))
    if low_bits == 0 and all(np.all(np.diff(P[v, :S[v]].astype(np.int64)) > 0) for v in range(n)):
        few = [x for x in few if len(x) <= 1024]
        off, nodes = _sets(few)
        pt = to_dev_u64(P.reshape(-1))
        est = torch.empty(len(few), dtype=torch.float64, device="cuda:0")
        for estimator in (0, 1):
            sk.skim_perm_query_batch(pt, st, 1 << 17, k, ell, to_dev_u64(off),
                                     to_dev_u32(np.minimum(nodes, n - 1)), est,
                                     estimator=estimator)
            want, _ = oracle_lib.perm_union_query(P, S, 1 << 17, k, ell, off,
                                                  np.minimum(nodes, n - 1), estimator)
            assert np.array_equal(est.cpu().numpy(), want)


@pytest.mark.parametrize("k,q", [(16, 64), (16, 65), (33, 1024), (33, 1025), (64, 1024), (64, 1025),
                                 (64, 2000)])
def test_batch_sizes_at_kernel_edges(oracle_lib, k, q):
    """Bottom-k batches at the sizes where the kernel for few queries gives way
    to a wave per query, within the grid of the persistent one."""
    from gpu_util import to_dev_u32, to_dev_u64
    n, ell = 300, 16
    rng = np.random.default_rng(k + q)
    R, S = _pool_tables(rng, n, k, 0)
    sets = [rng.integers(0, n, size=int(s)).tolist()
            for s in rng.choice([0, 1, 2, 7, 8, 9, 16, 17, 64, 65, 300], size=q)]
    off, nodes = _sets(sets)
    log(f"batch sizes k={k} q={q}")
    want, wst = oracle_lib.union_query(R, S, k, ell, off, nodes)
    got, status = gpu_query(to_dev_u64(R.reshape(-1)), to_dev_u32(S), n, k, ell, off, nodes, 0)
    assert np.array_equal(status, wst)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("k", [65, 256])
def test_single_nodes_over_long_sketches(oracle_lib, k):
    """Sets of one node, a workgroup each, over sketches of more than 64 ranks: full
    ones, short ones and empty ones, and a bad id."""
    from gpu_util import to_dev_u32, to_dev_u64
    n, ell = 120, 8
    rng = np.random.default_rng(k)
    R, S = _pool_tables(rng, n, k, 0)
    S[5], R[5] = 0, 2 ** 64 - 1
    sets = [[v] for v in range(n)] + [[n], [3, 3]]
    off, nodes = _sets(sets)
    want, wst = oracle_lib.union_query(R, S, k, ell, off, nodes)
    for mode in (0, 1):
        got, status = gpu_query(to_dev_u64(R.reshape(-1)), to_dev_u32(S), n, k, ell, off, nodes, 0,
                                mode)
        assert np.array_equal(status, wst) and np.array_equal(got, want)


def _uneven(kind, q, rng):
    sizes = np.clip(np.floor(np.exp(1.5 + 1.5 * rng.standard_normal(q))), 0, 1024).astype(int)
    if kind == "ascending":
        sizes = np.sort(sizes)
    elif kind == "descending":
        sizes = np.sort(sizes)[::-1]
    elif kind == "front":  # the large sets next to each other
        sizes = np.concatenate([np.full(q // 100, 700), rng.integers(0, 3, size=q - q // 100)])
    elif kind == "one":
        sizes = np.ones(q, dtype=int)
        sizes[q // 2] = 1024
    return sizes


@pytest.mark.parametrize("kind", ["ascending", "descending", "front", "one"])
@pytest.mark.parametrize("k", [16, 33, 64])
def test_uneven_batches(oracle_lib, kind, k):
    """Batches above the grid whose large sets stand together, of both estimators:
    every set is answered, whichever wave's share it falls into."""
    from gpu_util import to_dev_u32, to_dev_u64
    n, ell, q = 300, 16, 4097 if kind == "one" else 7001
    rng = np.random.default_rng(k)
    R, S = _pool_tables(rng, n, k, 0)
    off, nodes = _sets([rng.integers(0, n, size=s).tolist() for s in _uneven(kind, q, rng)])
    rt, st = to_dev_u64(R.reshape(-1)), to_dev_u32(S)
    for estimator, fn in [(0, oracle_lib.union_query), (1, oracle_lib.ck_query)]:
        log(f"uneven {kind} k={k} est={estimator}")
        want, wst = fn(R, S, k, ell, off, nodes)
        got, status = gpu_query(rt, st, n, k, ell, off, nodes, estimator)
        assert np.array_equal(status, wst) and np.array_equal(got, want)


@pytest.mark.parametrize("estimator", [0, 1])
def test_replayed_plan_with_offsets_out_of_order(oracle_lib, estimator):
    """A plan above the grid, replayed after some of its offsets were moved: the sets
    they bound get status -3 and estimate 0, every other set its answer."""
    import torch
    import paper_1408_6282_amd as sk
    from gpu_util import to_dev_u32, to_dev_u64
    n, ell, k, q = 300, 16, 16, 9000
    rng = np.random.default_rng(8)
    R, S = _pool_tables(rng, n, k, 0)
    sizes = rng.integers(0, 6, size=q)
    sizes[::500] = 70
    off, nodes = _sets([rng.integers(0, n, size=s).tolist() for s in sizes])
    rt, st, qo, qn = to_dev_u64(R.reshape(-1)), to_dev_u32(S), to_dev_u64(off), to_dev_u32(nodes)
    est = torch.full((q,), -1.0, dtype=torch.float64, device="cuda:0")
    status = torch.full((q,), 7, dtype=torch.int32, device="cuda:0")
    plan = sk.QueryPlan(rt, st, n, k, ell, qo, qn, est, status, estimator=estimator)
    try:
        for moved in ([], [1, 2000, 2001, 6500], list(range(100, 400, 7)) + [q - 1]):
            o = off.astype(np.int64).copy()
            for x in moved:  # back to the start, or past the end
                o[x] = 0 if x % 2 else int(off[-1]) + 5
            qo.copy_(torch.from_numpy(o).to(qo.device))
            est.fill_(-1.0)
            status.fill_(7)
            log(f"plan est={estimator} with {len(moved)} offsets moved")
            plan.launch()
            torch.cuda.synchronize()
            bad = (o[1:] < o[:-1]) | (o[1:] > o[-1])
            bad[0] |= o[0] != 0
            big = ~bad & (np.diff(o) > 1024)
            good = np.flatnonzero(~bad & ~big)
            o2, n2 = _sets([nodes[o[j]:o[j + 1]].tolist() for j in good])
            fn = oracle_lib.ck_query if estimator else oracle_lib.union_query
            want, _ = fn(R, S, k, ell, o2, n2)
            got, code = est.cpu().numpy(), status.cpu().numpy()
            assert np.all(code[bad] == -3) and np.all(got[bad] == 0.0)
            assert np.all(code[big] == -2) and np.all(got[big] == 0.0)
            assert np.all(code[good] == 0) and np.array_equal(got[good], want)
    finally:
        plan.free()


@pytest.mark.parametrize("k,q,members", [(33, 128, 1024), (33, 129, 1024), (64, 40, 1024),
                                         (64, 700, 190), (16, 60, 900)])
def test_few_large_sets(oracle_lib, k, q, members):
    """Few sets of many members, whose heads are often equal, around the number of
    entries from which they go to the kernel for larger batches, a bad member among
    them."""
    from gpu_util import to_dev_u32, to_dev_u64
    n, ell = 300, 16
    rng = np.random.default_rng(k + q)
    R, S = _pool_tables(rng, n, k, 0)
    sets = [rng.integers(0, n, size=members).tolist() for _ in range(q)]
    sets[3][members // 2] = n
    sets[7] = rng.integers(0, n, size=65).tolist()
    off, nodes = _sets(sets)
    want, wst = oracle_lib.union_query(R, S, k, ell, off, nodes)
    got, status = gpu_query(to_dev_u64(R.reshape(-1)), to_dev_u32(S), n, k, ell, off, nodes, 0)
    assert np.array_equal(status, wst) and np.array_equal(got, want)
