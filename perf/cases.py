"""What users of this library run, as cases whose time can be measured.

Six kinds of call, each through the package's entry points: sketch builds
(hashed and structured permutation ranks), union queries (one batch call, or
resident sketches), SKIM seed selection, IC-model sketches, the exact
influence evaluator, and the discrepancy tail of the adaptive error estimate.
The graphs are the synthetic kinds of ``workloads`` (Erdos-Renyi with uniform
probabilities, Chung-Lu with the weighted cascade, R-MAT with trivalency),
drawn here with torch on the GPU.
"""
import math

import numpy as np
import torch

import paper_1408_6282_amd as sk

DEV = "cuda"
U32 = 0xFFFFFFFF


def listed():
    return [
        # The smallest build: a 1000-node graph (the tests' and smoke check's
        # graph), where launches and host round trips are the time.
        dict(name="build_er_1k", kind="build", graph="er", n=1000, m=8000, denom=20, ell=16, k=16,
             perm=False),
        # An ordinary build at ragged sizes, no power of two among them.
        dict(name="build_wc_20k", kind="build", graph="wc", n=20011, m=317003, denom=0, ell=50,
             k=48, perm=False),
        # The benchmark's build: 10^6 nodes, 1.6 10^7 edges, weighted cascade.
        dict(name="build_wc_1m", kind="build", graph="wc", n=1_000_000, m=16_000_000, denom=0,
             ell=64, k=64, perm=False),
        # A graph with a dense core and huge reach sets (R-MAT, trivalency).
        dict(name="build_rmat_18", kind="build", graph="rmat", n=1 << 18, m=1 << 22, denom=0,
             ell=64, k=32, perm=False),
        # A handful of sets asked of resident sketches: one enqueued launch,
        # as an interactive oracle or a serving loop makes it.
        dict(name="query_few", kind="query", graph="wc", n=20000, m=320000, denom=0, ell=64, k=64,
             q=16, mean=2.0, sigma=1.0, hi=512, estimator=0, resident=True),
        # The batched workload: 10^6 lognormal sets over a small table.
        dict(name="query_lognormal_1m", kind="query", graph="er", n=1000, m=8000, denom=20, ell=16,
             k=16, q=1_000_000, mean=2.0, sigma=1.0, hi=512, estimator=0, resident=False),
        # Cohen-Kaplan estimates of sets of 50 nodes over the table of the
        # large graph (the sizes of the accuracy table: 1, 50, 1000).
        dict(name="query_ck_50", kind="query", graph="wc", n=1_000_000, m=16_000_000, denom=0,
             ell=64, k=64, q=20_000, mean=math.log(50.0), sigma=0.0, hi=512, estimator=1,
             resident=False),
        # SKIM as it is served: 200 seeds on a 1000-node graph.
        dict(name="greedy_er_1k", kind="greedy", graph="er", n=1000, m=8000, denom=100, ell=64,
             k=64, s=200),
        # SKIM on the large graph: 50 seeds.
        dict(name="greedy_wc_1m", kind="greedy", graph="wc", n=1_000_000, m=16_000_000, denom=0,
             ell=64, k=64, s=50),
        # Sketches for the IC model itself.
        dict(name="ic_wc_20k", kind="ic", graph="wc", n=20000, m=320000, denom=0, k=64),
        # The quality harness: every prefix of a 200-seed sequence scored on
        # 64 fresh instances.
        dict(name="influence_wc_20k", kind="influence", graph="wc", n=20000, m=320000, denom=0,
             ell=64, s=200),
        # The confidence distribution of a 200-seed run on 4096 bins.
        dict(name="tail_200", kind="tail", s=200, bins=4096, k=64, max_rel=0.25),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_graph(rng, lo, hi, kinds=("er", "wc", "wc", "rmat")):
    kind = rng.choice(kinds)
    if kind == "rmat":
        n = 1 << rng.randint(10, max(11, min(17, int(math.log2(hi)))))
        return dict(graph=kind, n=n, m=n * rng.randint(4, 16), denom=0)
    n = _log_int(rng, lo, hi)
    deg = rng.uniform(4.0, 16.0)
    # Erdos-Renyi: live out-degree 0.2 .. 0.8, below the giant component
    denom = max(2, int(deg / rng.uniform(0.2, 0.8))) if kind == "er" else 0
    return dict(graph=kind, n=n, m=int(n * deg), denom=denom)


def draw(rng):
    kind = rng.choice(["build", "build", "build", "query", "query", "query", "greedy", "greedy",
                       "ic", "influence", "tail"])
    if kind == "build":
        return dict(kind=kind, **_draw_graph(rng, 500, 600_000),
                    ell=rng.choice([4, 7, 16, 25, 32, 50, 64, 64]), k=_log_int(rng, 8, 64),
                    perm=rng.random() < 0.25)
    if kind == "query":
        c = dict(kind=kind, **_draw_graph(rng, 700, 300_000, ("er", "wc")),
                 ell=rng.choice([16, 31, 64]), k=rng.choice([16, 24, 32, 64]),
                 estimator=int(rng.random() < 0.4), resident=rng.random() < 0.4)
        # uniform-ish, lognormal or fixed sizes; the entries in all bounded
        c.update(mean=rng.uniform(0.0, 5.0), sigma=rng.choice([0.0, 0.5, 1.0]), hi=512)
        top = 1_000_000 * (0.02 if c["estimator"] else 1.0) * 8.0 / math.exp(c["mean"] + c["sigma"])
        c["q"] = _log_int(rng, 1, max(2.0, min(1_000_000, top)))
        return c
    if kind == "greedy":
        c = dict(kind=kind, **_draw_graph(rng, 700, 300_000, ("er", "wc", "wc")),
                 ell=rng.choice([16, 33, 64]), k=rng.choice([16, 32, 64]))
        c["s"] = rng.randint(5, 50)
        return c
    if kind == "ic":
        return dict(kind=kind, **_draw_graph(rng, 500, 20_000, ("er", "wc")),
                    k=rng.randint(8, 64))
    if kind == "influence":
        return dict(kind=kind, **_draw_graph(rng, 500, 20_000, ("er", "wc")),
                    ell=rng.choice([5, 16, 32, 64]), s=rng.randint(2, 200))
    return dict(kind=kind, s=rng.randint(2, 200), bins=_log_int(rng, 50, 4096),
                k=rng.choice([16, 64]), max_rel=rng.choice([0.1, 0.25, 0.5]))


# ------------------------------------------------------------------- inputs
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * int(seed) + salt)
    return g


def _rand(g, size, dtype=torch.float64):
    return torch.rand(size, generator=g, device=DEV, dtype=dtype)


def _powerlaw(g, n, size):
    """Ranks in [0, n) with weight (j + 1)^(-1 / 1.1) (gamma = 2.1)."""
    one = 1.0 - 1.0 / 1.1
    x = (1.0 + _rand(g, size) * ((n + 1.0) ** one - 1.0)) ** (1.0 / one) - 1.0
    return x.to(torch.int64).clamp_(max=n - 1)


def _sample_edges(kind, g, n, size, perms):
    if kind == "er":
        u = torch.randint(n, (size,), generator=g, device=DEV)
        v = torch.randint(n, (size,), generator=g, device=DEV)
    elif kind == "wc":
        u, v = perms[0][_powerlaw(g, n, size)], perms[1][_powerlaw(g, n, size)]
    else:  # R-MAT quadrants (.57, .19, .19, .05)
        u = torch.zeros(size, dtype=torch.int64, device=DEV)
        v = torch.zeros_like(u)
        for _ in range(n.bit_length() - 1):
            x = _rand(g, size, torch.float32)
            down = x >= 0.76
            right = torch.where(down, x >= 0.95, x >= 0.57)
            u, v = 2 * u + down, 2 * v + right
        u, v = perms[0][u], perms[0][v]
    return (u * n + v)[u != v]


def _graph(case, seed):
    """(row_ptr int64, col int32, thr int32) on the GPU; m distinct edges (R-MAT:
    m samples, duplicates dropped)."""
    kind, n, m = case["graph"], case["n"], case["m"]
    g = _gen(seed, 1)
    perms = [torch.randperm(n, generator=g, device=DEV) for _ in range(2)]
    keys = torch.unique(_sample_edges(kind, g, n, m if kind == "rmat" else int(1.35 * m) + 1024,
                                      perms))
    while kind != "rmat" and keys.numel() < m:
        more = _sample_edges(kind, g, n, 2 * (m - keys.numel()) + 1024, perms)
        keys = torch.unique(torch.cat([keys, more]))
    if kind != "rmat" and keys.numel() > m:
        keep = torch.randperm(keys.numel(), generator=g, device=DEV)[:m]
        keys = keys[keep.sort().values]
    src, dst = keys // n, keys % n
    row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    row_ptr[1:] = torch.bincount(src, minlength=n).cumsum(0)
    if kind == "er":
        thr = torch.full_like(dst, U32 // case["denom"])
    elif kind == "wc":
        thr = U32 // torch.bincount(dst, minlength=n)[dst]
    else:
        p = torch.tensor([U32 // 10, U32 // 100, U32 // 1000], device=DEV)
        thr = p[torch.randint(3, dst.shape, generator=g, device=DEV)]
    return row_ptr, dst.to(torch.int32), thr.to(torch.int32)


def _sets(case, seed):
    """(qoff int64, qnodes int32): lognormal sizes, distinct members (an
    arithmetic walk of a random stride over a random permutation)."""
    n, q = case["n"], case["q"]
    g = _gen(seed, 2)
    z = torch.randn(q, generator=g, device=DEV, dtype=torch.float64)
    size = torch.exp(case["mean"] + case["sigma"] * z).add_(0.5).floor_().to(torch.int64)
    size.clamp_(1, min(case["hi"], n))
    qoff = torch.zeros(q + 1, dtype=torch.int64, device=DEV)
    qoff[1:] = size.cumsum(0)
    total = int(qoff[-1])
    strides = torch.tensor([b for b in range(1, min(n, 4000)) if math.gcd(b, n) == 1], device=DEV)
    b = strides[torch.randint(strides.numel(), (q,), generator=g, device=DEV)]
    a = torch.randint(n, (q,), generator=g, device=DEV)
    j = torch.arange(total, device=DEV) - torch.repeat_interleave(qoff[:-1], size)
    perm = torch.randperm(n, generator=g, device=DEV)
    at = (torch.repeat_interleave(a, size) + torch.repeat_interleave(b, size) * j) % n
    return qoff, perm[at].to(torch.int32)


def _records(case, seed):
    """SKIM records as a run leaves them: falling gains (pairs), the rank that
    filled each sketch (rho about k / gain), the second largest sketch."""
    s, k = case["s"], case["k"]
    rng = np.random.default_rng([int(seed), 3])
    gain = np.maximum(64, 20000.0 * np.arange(1, s + 1) ** -0.6 * rng.uniform(0.9, 1.1, s))
    gain = np.sort(gain.astype(np.int64))[::-1].copy()
    rho = np.minimum(1.0, k / gain * rng.uniform(0.85, 1.15, s))
    tau = (rho * 2.0 ** 53).astype(np.uint64) << np.uint64(11)
    tau[rho >= 1.0] = np.uint64(0xFFFFFFFFFFFFF800)
    second = (k - 1 - np.minimum(k - 1, rng.geometric(0.2, s) - 1)).astype(np.int32)
    return tau, second, gain


def _empty(n, dtype):
    return torch.empty(n, dtype=dtype, device=DEV)


def _tables(G, case, seed):
    """Sketches of the graph, as the caller of a query holds them."""
    n, k = case["n"], case["k"]
    ranks, size = _empty(n * k, torch.int64), _empty(n, torch.int32)
    sk.skim_build_sketches(G, case["ell"], k, _method_seed(seed), ranks, size)
    return ranks, size


def _method_seed(seed):
    return 7919 * int(seed) + 1


def prepare(case, seed):
    st = dict(case=case, seed=_method_seed(seed))
    kind = case["kind"]
    if kind == "tail":
        tau, second, gain = _records(case, seed)
        st.update(tau=torch.from_numpy(tau.view(np.int64)).to(DEV),
                  second=torch.from_numpy(second).to(DEV), gain=torch.from_numpy(gain).to(DEV),
                  tail=_empty(case["bins"] + 1, torch.float64))
        return st
    n = case["n"]
    G = st["G"] = sk.DeviceGraph(n, *_graph(case, seed))
    if kind == "build":
        st.update(ranks=_empty(n * case["k"], torch.int64), size=_empty(n, torch.int32),
                  est=_empty(n, torch.float64))
    elif kind == "query":
        ranks, size = _tables(G, case, seed)
        qoff, qnodes = _sets(case, seed)
        st.update(ranks=ranks, size=size, qoff=qoff, qnodes=qnodes,
                  est=_empty(case["q"], torch.float64), status=_empty(case["q"], torch.int32))
        if case["resident"]:
            st["table"] = sk.Sketches.from_tables(ranks, size, n, case["k"], case["ell"])
        del st["G"]
    elif kind == "greedy":
        s = case["s"]
        st.update(seeds=_empty(s, torch.int32), gain_pairs=_empty(s, torch.int64),
                  gain=_empty(s, torch.float64))
    elif kind == "ic":
        st.update(pos=_empty(n * case["k"], torch.int32), est=_empty(n, torch.float64))
    else:  # influence: the prefixes of the nodes of largest out-degree
        s = case["s"]
        seeds = torch.argsort(G.row_ptr.diff(), descending=True, stable=True)[:s]
        size = torch.arange(1, s + 1, device=DEV)
        qoff = torch.zeros(s + 1, dtype=torch.int64, device=DEV)
        qoff[1:] = size.cumsum(0)
        j = torch.arange(s * (s + 1) // 2, device=DEV)
        at = j - torch.repeat_interleave(qoff[:-1], size)
        st.update(qoff=qoff, qnodes=seeds[at].to(torch.int32), reach=_empty(s, torch.int64))
    return st


def run(st):
    c, kind = st["case"], st["case"]["kind"]
    if kind == "build":
        build = sk.skim_build_sketches_perm if c["perm"] else sk.skim_build_sketches
        build(st["G"], c["ell"], c["k"], st["seed"], st["ranks"], st["size"], st["est"])
        return dict(ranks=st["ranks"], size=st["size"], est=st["est"])
    if kind == "query":
        if c["resident"]:
            st["table"].query(st["qoff"], st["qnodes"], st["est"], st["status"],
                              estimator=c["estimator"])
        else:
            sk.skim_query_batch(st["ranks"], st["size"], c["n"], c["k"], c["ell"], st["qoff"],
                                st["qnodes"], st["est"], st["status"], estimator=c["estimator"])
        return dict(est=st["est"], status=st["status"])
    if kind == "greedy":
        sk.skim_greedy(st["G"], c["ell"], c["k"], st["seed"], c["s"], st["seeds"],
                       st["gain_pairs"], st["gain"])
        return dict(seeds=st["seeds"], gain_pairs=st["gain_pairs"], gain=st["gain"])
    if kind == "ic":
        sk.skim_build_ic_sketches(st["G"], c["k"], st["seed"], st["pos"], st["est"])
        return dict(pos=st["pos"], est=st["est"])
    if kind == "influence":
        sk.skim_influence_batch(st["G"], c["ell"], st["seed"], st["qoff"], st["qnodes"],
                                st["reach"])
        return dict(reach=st["reach"])
    sk.skim_discrepancy_tail(st["tau"], st["second"], st["gain"], c["bins"], c["max_rel"],
                             st["tail"])
    return dict(tail=st["tail"])


def work(case):
    """Bytes: the inputs once and the outputs once (a query: its set, the heads
    of its members' sketches and the k ranks, or 8 (k - 1) |S| bytes for
    Cohen-Kaplan, which reads every rank; never more than the whole table).
    Flops: the multiply-adds of the tail's convolutions; the other paths are
    integer work."""
    kind = case["kind"]
    if kind == "tail":
        s, w = case["s"], case["bins"] + 1
        return {"bytes": 20.0 * s + 8.0 * w, "flops": float(s - 1) * w * (w + 1)}
    n, m = case["n"], case["m"]
    graph = 8.0 * (n + 1) + 8.0 * m
    if kind == "build":
        return {"bytes": graph + n * (8.0 * case["k"] + 12.0), "flops": 0.0}
    if kind == "ic":
        return {"bytes": graph + n * (4.0 * case["k"] + 8.0), "flops": 0.0}
    if kind == "greedy":
        return {"bytes": graph + 20.0 * case["s"], "flops": 0.0}
    if kind == "influence":
        s = case["s"]
        return {"bytes": graph + 16.0 * s + 2.0 * s * (s + 1), "flops": 0.0}
    q, k = case["q"], case["k"]
    members = q * min(case["hi"], n, max(1.0, math.exp(case["mean"] + case["sigma"] ** 2 / 2)))
    read = 8.0 * (k - 1) * members if case["estimator"] else 8.0 * (members + k * q)
    return {"bytes": 20.0 * q + 8 + 8.0 * members + min(read, 8.0 * n * k), "flops": 0.0}


# ---------------------------------------------------------------- in 64 bits
_GOLD = np.uint64(0x9E3779B97F4A7C15)


def _splitmix(seed, c):
    """Output c of the SplitMix64 stream of `seed`."""
    with np.errstate(over="ignore"):
        z = np.uint64(seed) + (c + np.uint64(1)) * _GOLD
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        return z ^ (z >> np.uint64(31))


def _plain_sketches(case, seed):
    """Each node's k smallest ranks (uint64, all ones where there are fewer)
    by transitive closure of every instance; None for large graphs."""
    n, ell, k = case["n"], case["ell"], case["k"]
    if n > 2048 or case["graph"] != "er":
        return None
    ms = _method_seed(seed)
    row_ptr, col, thr = (t.cpu().numpy() for t in _graph(case, seed))
    src = np.repeat(np.arange(n), np.diff(row_ptr)).astype(np.uint64)
    dst = col.astype(np.uint64)
    best = np.full((n, 0), 0, dtype=np.uint64)
    for i in range(ell):
        h = _splitmix(ms, np.uint64(1 << 62) + np.uint64(32) * (src * np.uint64(n) + dst)
                      + np.uint64(i // 2))
        coin = (h >> np.uint64(32)) if i % 2 == 0 else (h & np.uint64(U32))
        live = coin <= thr.view(np.uint32).astype(np.uint64)
        reach = torch.eye(n, device=DEV)
        reach[torch.from_numpy(src[live].astype(np.int64)).to(DEV),
              torch.from_numpy(dst[live].astype(np.int64)).to(DEV)] = 1.0
        while True:
            wider = (reach @ reach > 0.5).float()
            if torch.equal(wider, reach):
                break
            reach = wider
        ranks = _splitmix(ms, np.arange(n, dtype=np.uint64) * np.uint64(64) + np.uint64(i))
        seen = np.where(reach.cpu().numpy() > 0.5, ranks[None, :], np.uint64(2 ** 64 - 1))
        kk = min(k, n) - 1
        low = np.partition(seen, kk, axis=1)[:, :kk + 1]
        best = np.sort(np.concatenate([best, low], axis=1), axis=1)[:, :k]
    out = np.full((n, k), 2 ** 64 - 1, dtype=np.uint64)
    out[:, :best.shape[1]] = best
    return out


def _rho(rank):
    return ((rank >> np.uint64(11)) + np.uint64(1)).astype(np.float64) * 2.0 ** -53


def _bottom_k(count, tau, k, ell):
    full = (k - 1) / _rho(tau) / ell
    return np.where(count < k, count / ell, full)


def _plain_queries(case, seed):
    table = _plain_sketches(case, seed)
    if table is None:
        return None
    k, ell, q = case["k"], case["ell"], case["q"]
    none = np.uint64(2 ** 64 - 1)
    values, index = np.unique(table, return_inverse=True)
    index = torch.from_numpy(index.reshape(table.shape).astype(np.int64)).to(DEV)
    last = values.size - 1 if values[-1] == none else values.size  # index of "no rank"
    qoff, qnodes = _sets(case, seed)
    width = 1 << int(values.size).bit_length()
    est = np.empty(q)
    step = max(1, int(q * 4_000_000 / max(1, qnodes.numel())))
    real = torch.from_numpy(_rho(values)).to(DEV)
    real = torch.cat([real[:last], torch.ones(width - last, dtype=torch.float64, device=DEV)])
    for a in range(0, q, step):
        b = min(q, a + step)
        off = qoff[a:b + 1]
        nodes = qnodes[int(off[0]):int(off[-1])].long()
        sets = torch.repeat_interleave(torch.arange(b - a, device=DEV), off.diff())
        rows = index[nodes]
        full = rows[:, k - 1] < last
        if case["estimator"]:
            held = rows.clone()
            held[full, k - 1] = last  # a full sketch's threshold does not count
        else:
            held = rows
        key = (sets[:, None] * width + held)[held < last]
        uniq, inv = torch.unique(key, return_inverse=True)
        of = uniq // width
        count = torch.bincount(of, minlength=b - a)
        if case["estimator"]:
            tau = torch.where(full, real[rows[:, k - 1]], torch.ones_like(real[rows[:, k - 1]]))
            each = tau[:, None].expand(-1, k)[held < last]
            most = torch.zeros(uniq.numel(), dtype=torch.float64, device=DEV)
            most.scatter_reduce_(0, inv, each, "amax")
            tot = torch.zeros(b - a, dtype=torch.float64, device=DEV)
            tot.index_add_(0, of, 1.0 / most)
            est[a:b] = (tot / ell).cpu().numpy()
        else:
            start = count.cumsum(0) - count
            at = (start + k - 1).clamp(max=uniq.numel() - 1)
            tau = values[(uniq[at] % width).cpu().numpy().clip(max=values.size - 1)]
            est[a:b] = _bottom_k(count.cpu().numpy(), tau, k, ell)
    return est


def _plain_tail(case, seed):
    """The distribution after each seed, one convolution at a time."""
    tau, second, gain = _records(case, seed)
    bins, total = case["bins"], float(gain.sum())
    h = case["max_rel"] * total / bins
    mass = np.zeros(bins + 1)
    mass[0] = 1.0
    for t, z, d in zip(tau, second.astype(np.float64), gain.astype(np.float64)):
        eps = np.arange(bins) * h / d
        mu = float(_rho(np.array([t]))[0]) * d * (1.0 + eps)
        with np.errstate(divide="ignore", invalid="ignore"):
            bound = np.exp(z - mu + (z * np.log(mu / z) if z else 0.0))
        surv = np.concatenate([[1.0], np.where(z >= mu, 1.0, np.minimum(1.0, bound)), [0.0]])
        step = surv[:-1] - surv[1:]
        both = np.convolve(mass, step)
        mass = np.append(both[:bins], both[bins:].sum())
    return mass[::-1].cumsum()[::-1].copy()


def exact(case, seed):
    kind = case["kind"]
    if kind == "build" and not case["perm"]:
        table = _plain_sketches(case, seed)
        if table is None:
            return None
        count = (table != np.uint64(2 ** 64 - 1)).sum(axis=1)
        est = _bottom_k(count, table[:, -1], case["k"], case["ell"])
        return dict(ranks=None, size=None, est=est)
    if kind == "query":
        est = _plain_queries(case, seed)
        return None if est is None else dict(est=est, status=None)
    if kind == "tail":
        return dict(tail=_plain_tail(case, seed))
    return None
