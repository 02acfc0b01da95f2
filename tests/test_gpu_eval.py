"""GPU parity of skim_influence_batch, the exact influence evaluator of the
quality harness (Section 2, eqs. (Inf) and (timedinf)), against the oracle's
forward search per instance: every count bit for bit.

* random graphs over l, with empty sets, duplicate members and invalid nodes;
* SKIM's seed prefixes on the instances SKIM used: the evaluator must
  reproduce the cumulative gains (Section 4.1.1), and on 512 fresh instances
  (8 other seeds) the oracle's counts;
* the Chung-Lu graph at full size (10^6 nodes, 1.6 10^7 edges, l = 64);
* argument errors.
"""
import numpy as np
import pytest

from workloads import from_edges
from workloads.configs import make_config, make_graph
from brute import random_small_graph
from gpu_util import dev, gpu_greedy, log, to_dev_u32, to_dev_u64

pytestmark = pytest.mark.gpu


def gpu_influence(g, ell, seed, sets, G=None, status=True):
    import torch
    import paper_1408_6282_amd as sk
    G = G or sk.DeviceGraph.from_host(g, dev())
    off = np.zeros(len(sets) + 1, dtype=np.uint64)
    off[1:] = np.cumsum([len(s) for s in sets])
    nodes = np.concatenate([np.asarray(s, dtype=np.uint32) for s in sets]) if off[-1] else None
    q = len(sets)
    out = torch.full((max(q, 1),), -5, dtype=torch.int64, device=dev())
    st = torch.full((max(q, 1),), 7, dtype=torch.int32, device=dev()) if status else None
    sk.skim_influence_batch(G, ell, seed, to_dev_u64(off),
                            to_dev_u32(nodes) if nodes is not None else None, out, st)
    torch.cuda.synchronize()
    r = out.cpu().numpy().view(np.uint64)[:q]
    return (r, st.cpu().numpy()[:q]) if status else r


@pytest.mark.parametrize("ell", [1, 5, 64])
def test_random_graphs_and_sets(oracle_lib, ell):
    rng = np.random.default_rng(ell + 40)
    for trial in range(4):
        n = int(rng.integers(2, 120))
        src, dst, thr = random_small_graph(rng, n, int(rng.integers(0, 4 * n)),
                                           [0xFFFFFFFF, 0xFFFFFFFF // 3, 0xFFFFFFFF // 20])
        g = from_edges(n, src, dst, thr)
        seed = int(rng.integers(0, 2 ** 62))
        sets = [[]]
        for _ in range(60):
            sz = int(rng.integers(1, min(n, 12) + 1))
            sets.append(rng.integers(0, n, size=sz).tolist())  # duplicates allowed
        sets.append([0, 0, 0])
        sets.append([n - 1, n])  # invalid: node n
        log(f"influence ell={ell} n={n} m={g.m} q={len(sets)} seed={seed}")
        got, st = gpu_influence(g, ell, seed, sets)
        for j, S in enumerate(sets):
            if max(S, default=-1) >= n:
                assert st[j] == -1 and got[j] == 0
                continue
            assert st[j] == 0
            assert int(got[j]) == oracle_lib.influence(g, seed, ell, sorted(set(S))), (j, S)


def test_skim_prefixes_same_and_fresh_instances(oracle_lib):
    cfg = make_config("served-skim")
    g = make_graph(cfg)
    ell, k, seed = cfg["ell"], cfg["k"], cfg["seed"]
    seeds, gains, _, _ = gpu_greedy(g, ell, k, seed, [200])
    prefixes = [seeds[:j].tolist() for j in (1, 2, 5, 10, 50, 100, 200)]
    log("influence: SKIM prefixes on SKIM's own instances")
    got, st = gpu_influence(g, ell, seed, prefixes)
    assert np.all(st == 0)
    cum = np.cumsum(gains.astype(np.uint64))
    assert [int(x) for x in got] == [int(cum[len(p) - 1]) for p in prefixes]
    for fresh in range(1, 9):  # 8 x 64 = 512 fresh instances
        log(f"influence: SKIM prefixes on fresh instances, seed {seed + 1000 * fresh}")
        got = gpu_influence(g, 64, seed + 1000 * fresh, prefixes, status=False)
        want = [oracle_lib.influence(g, seed + 1000 * fresh, 64, p) for p in prefixes]
        assert [int(x) for x in got] == want


@pytest.mark.slow
def test_chung_lu_1m_sets(oracle_lib):
    cfg = make_config("chung-lu-1m")
    log("generating chung-lu-1m")
    g = make_graph(cfg)
    rng = np.random.default_rng(77)
    outdeg = np.diff(g.row_ptr.astype(np.int64))
    hubs = np.argsort(outdeg)[::-1][:64].tolist()
    sets = [rng.integers(0, g.n, size=sz).tolist() for sz in (1, 1, 8, 64, 1000)]
    sets += [hubs[:1], hubs[:16], hubs]
    log("gpu influence chung-lu-1m")
    got, st = gpu_influence(g, cfg["ell"], cfg["seed"], sets)
    assert np.all(st == 0)
    for j, S in enumerate(sets):
        want = oracle_lib.influence(g, cfg["seed"], cfg["ell"], sorted(set(S)))
        log(f"  set {j} |S|={len(S)}: {int(got[j])} vs {want}")
        assert int(got[j]) == want


def test_errors_and_empty_batches():
    import torch
    import paper_1408_6282_amd as sk
    g = from_edges(6, [0, 1, 2], [1, 2, 3])
    G = sk.DeviceGraph.from_host(g, dev())
    r = torch.empty(2, dtype=torch.int64, device=dev())
    nodes = to_dev_u32([0, 1])
    # every set empty: no node array needed
    got = gpu_influence(g, 4, 1, [[], []], G=G, status=False)
    assert got.tolist() == [0, 0]
    # q = 0
    sk.skim_influence_batch(G, 4, 1, to_dev_u64([0]), None, r)
    for off in ([1, 1, 2], [0, 2, 1]):  # qoff[0] != 0; decreasing
        with pytest.raises(sk.SkimError) as ei:
            sk.skim_influence_batch(G, 4, 1, to_dev_u64(off), nodes, r)
        assert ei.value.status == sk.SKIM_EINVAL
    for ell in (0, 65):
        with pytest.raises(sk.SkimError) as ei:
            sk.skim_influence_batch(G, ell, 1, to_dev_u64([0, 1, 2]), nodes, r)
        assert ei.value.status == sk.SKIM_EINVAL
    with pytest.raises(sk.SkimError) as ei:  # sets hold nodes but no node array
        sk.skim_influence_batch(G, 4, 1, to_dev_u64([0, 1, 2]), None, r)
    assert ei.value.status == sk.SKIM_EINVAL


def gpu_greedy_exact(g, ell, seed, s):
    import torch
    import paper_1408_6282_amd as sk
    G = sk.DeviceGraph.from_host(g, dev())
    a = torch.full((max(s, 1),), -1, dtype=torch.int32, device=dev())
    b = torch.full((max(s, 1),), -1, dtype=torch.int64, device=dev())
    sk.skim_greedy_exact(G, ell, seed, s, a, b)
    torch.cuda.synchronize()
    return a.cpu().numpy().view(np.uint32)[:s], b.cpu().numpy().view(np.uint64)[:s]


@pytest.mark.parametrize("ell", [1, 8, 64])
def test_greedy_exact_matches_oracle(oracle_lib, ell):
    # the oracle's SKIM with k above every |R_u| is exact greedy (pinned
    # against brute force): every seed from the exhaustion rule
    rng = np.random.default_rng(ell + 70)
    for trial in range(3):
        n = int(rng.integers(2, 60))
        src, dst, thr = random_small_graph(rng, n, int(rng.integers(0, 3 * n)),
                                           [0xFFFFFFFF, 0xFFFFFFFF // 2, 0xFFFFFFFF // 10])
        g = from_edges(n, src, dst, thr)
        seed = int(rng.integers(0, 2 ** 62))
        s = n if trial == 0 else int(rng.integers(1, n + 1))
        log(f"greedy exact ell={ell} n={n} m={g.m} s={s}")
        seeds, gains = gpu_greedy_exact(g, ell, seed, s)
        ws, wg, cnt = oracle_lib.skim(g, seed, ell, n * ell + 1, s)
        assert cnt["fallback"] == s
        assert np.array_equal(seeds, ws) and np.array_equal(gains, wg)


def test_greedy_exact_served_config(oracle_lib):
    cfg = make_config("served-skim")
    g = make_graph(cfg)
    log("greedy exact served-skim 50 seeds")
    seeds, gains = gpu_greedy_exact(g, cfg["ell"], cfg["seed"], 50)
    ws, wg, _ = oracle_lib.skim(g, cfg["seed"], cfg["ell"], g.n * cfg["ell"] + 1, 50)
    assert np.array_equal(seeds, ws) and np.array_equal(gains, wg)
    # the prefixes' influence on the same instances is the running sum of gains
    got = gpu_influence(g, cfg["ell"], cfg["seed"], [seeds[:j].tolist() for j in (1, 10, 50)],
                        status=False)
    cum = np.cumsum(gains)
    assert [int(v) for v in got] == [int(cum[0]), int(cum[9]), int(cum[49])]


@pytest.mark.parametrize("n,q", [(1, 1), (64, 31), (4096, 32), (4097, 33), (25999, 65),
                                 (26000, 2), (26001, 40)])
def test_words_of_32_queries_at_state_limits(oracle_lib, n, q):
    """The masks' places (LDS at 256 and at 1024 threads, global memory) and the
    words of 32 queries at their edges: nested prefixes, lone nodes (few pushes:
    counted over the ring), and sets that reach a dense core (counted over all
    nodes)."""
    rng = np.random.default_rng(n + q)
    m = 0 if n == 1 else 3 * n
    e = np.unique(rng.integers(0, n, size=(m, 2)), axis=0)
    e = e[e[:, 0] != e[:, 1]]
    g = from_edges(n, e[:, 0], e[:, 1], 0xFFFFFFFF // 2)
    order = rng.permutation(n)
    sets = []
    for j in range(q):
        kind = j % 3
        if kind == 0:
            sets.append(order[:1 + j].tolist())
        elif kind == 1:
            sets.append([int(rng.integers(n))])
        else:
            sets.append([] if j == 2 else rng.integers(0, n, size=5).tolist())
    if q > 32:
        sets[32] = [0, n]  # a bad member leaves the other queries of its word alone
    for ell in (1, 9):
        log(f"influence words n={n} q={q} ell={ell}")
        got, st = gpu_influence(g, ell, 11, sets)
        for j, S in enumerate(sets):
            if max(S, default=-1) >= n:
                assert st[j] == -1 and got[j] == 0
                continue
            assert st[j] == 0
            assert int(got[j]) == oracle_lib.influence(g, 11, ell, sorted(set(S))), (j, S)


def test_sizes_of_two_threads_do_not_meet(oracle_lib):
    # two threads evaluate graphs of different sizes, each on a stream of its
    # own: the LDS that one needs is not limited by the other's call
    import threading
    import torch
    import paper_1408_6282_amd as sk
    from workloads.graphs import Graph, er_graph
    work = []
    for n in (4200, 26000):
        rp, col = er_graph(n, 2 * n, n)
        g = Graph(n, rp, col, np.full(col.size, 0xFFFFFFFF // 4, dtype=np.uint32))
        sets = [[v] for v in range(8)]
        work.append((sk.DeviceGraph.from_host(g, "cuda:0"), sets,
                     [oracle_lib.influence(g, 9, 2, s) for s in sets]))
    errors = []

    def run(G, sets, want):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                off = torch.arange(len(sets) + 1, dtype=torch.int64, device="cuda:0")
                nodes = torch.tensor([s[0] for s in sets], dtype=torch.int32, device="cuda:0")
                out = torch.empty(len(sets), dtype=torch.int64, device="cuda:0")
                for _ in range(50):
                    sk.skim_influence_batch(G, 2, 9, off, nodes, out, stream=stream)
                    if out.cpu().tolist() != [int(w) for w in want]:
                        errors.append("wrong counts")
        except Exception as e:  # noqa: BLE001 - reported by the test
            errors.append(repr(e))

    threads = [threading.Thread(target=run, args=w) for w in work]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors[:3]


@pytest.mark.parametrize("n", [300, 27000])
def test_few_instances_and_word_widths(oracle_lib, n):
    """Fewer instances than XCDs, and batches at the sizes where a word of queries
    changes its width, on LDS and on global state."""
    rng = np.random.default_rng(n)
    e = np.unique(rng.integers(0, n, size=(4 * n, 2)), axis=0)
    e = e[e[:, 0] != e[:, 1]]
    g = from_edges(n, e[:, 0], e[:, 1], 0xFFFFFFFF // 3)
    for ell, qs in [(1, (1, 64, 65, 129)), (2, (32, 33)), (3, (22,)), (5, (13, 26)), (9, (7, 8, 33))]:
        for q in qs:
            sets = [rng.integers(0, n, size=int(rng.integers(0, 4))).tolist() for _ in range(q)]
            log(f"influence n={n} ell={ell} q={q}")
            got, st = gpu_influence(g, ell, 7, sets)
            assert not st.any()
            for j in rng.permutation(q)[:12]:
                assert int(got[j]) == oracle_lib.influence(g, 7, ell, sorted(set(sets[j]))), (j, ell)


@pytest.mark.parametrize("fan", [1, 7, 8, 9, 33, 63, 64, 65, 200])
def test_out_lists_of_sources_in_one_wave(oracle_lib, fan):
    """Sources of `fan` edges each: waves of one source, of a few and of more than
    are counted from the transposed masks, with a ragged last wave."""
    rng = np.random.default_rng(fan)
    n, hubs = 900, 40
    src = np.repeat(np.arange(hubs), fan)
    dst = np.concatenate([hubs + rng.choice(n - hubs, fan, replace=False) for _ in range(hubs)])
    g = from_edges(n, src, dst, rng.integers(0, 1 << 32, size=src.size, dtype=np.uint32))
    sets = [[h] for h in range(hubs)]
    for ell in (1, 16, 64):
        log(f"out-lists fan={fan} ell={ell}")
        got, _ = gpu_influence(g, ell, 13, sets)
        assert [int(x) for x in got] == [int(oracle_lib.influence(g, 13, ell, s)) for s in sets]
