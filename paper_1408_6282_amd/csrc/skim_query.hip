// skim_query.hip -- influence queries from the sketches (Section 5.1).
//
// The member sketches are sorted, so the distinct ranks of their union come
// out in increasing order from a k-way merge: each step takes the minimum head
// over the members, then advances every member whose head equals it.
//  * bottom-k estimator: stop at the k-th distinct value tau (or when the
//    union runs out), estimate as for a single sketch.  A set of up to 64
//    members is merged by a group of 4 to 16 lanes (merge_group), so a wave
//    answers 4 to 16 sets at once; a larger one by the whole wave;
//  * Cohen-Kaplan (eq. unionest): every distinct non-threshold value of the
//    union weighs 1/rho(max tau_u over the members holding it), a non-full
//    member counting as rho = 1; the weights are added in increasing order of
//    the value.  Sets of up to 64 members over sketches of k <= 64 are sorted
//    in registers (ck_sorted); others are merged by the whole wave.
// The batched path is one persistent launch whose waves take shares of the batch or
// pull runs of queries from a device counter (Cohen-Kaplan's large sets of a long
// batch: a second launch); the plain path launches the same device code once per
// query.
#include "skim_internal.h"
#include "skim_wave.h"

#include <atomic>
#include <memory>

namespace skim {

namespace {

constexpr uint32_t kMaxMembers = 1024;  // members per query (LDS state)
constexpr int kQBlock = 64;             // one wave per block
constexpr int kPerLane = kMaxMembers / 64;
constexpr uint32_t kRun = 64;           // most queries a wave takes at once
constexpr uint64_t kTakeMembers = 48;   // mean set size from which the counter balances
constexpr uint64_t kSetWeight = 4;      // a set weighs as much as its members and this many more

using QArgs = QueryArgs;

// Members of a set merged by the whole wave.
struct MergeLds {
    uint32_t mnode[kMaxMembers];
    uint16_t mpos[kMaxMembers];
    uint16_t mlim[kMaxMembers];
};

__device__ __forceinline__ uint64_t shfl_u64(uint64_t x, uint32_t src) {
    const uint32_t lo = __shfl((uint32_t)x, (int)src), hi = __shfl((uint32_t)(x >> 32), (int)src);
    return ((uint64_t)hi << 32) | lo;
}

// The k-way merge over S members (R >= S / 64 register slots per lane).
// Each lane keeps the current head of its members t = lane + 64 r in
// registers; a step reads global memory only for the members that advance.
// Bottom-k stops at the k-th distinct value (d, tau); Cohen-Kaplan adds each
// distinct value's weight in increasing order (sum).
template <int R>
__device__ __forceinline__ void merge_members(const QArgs &Q, uint64_t S, uint32_t k, MergeLds &X,
                                              uint32_t &d, uint64_t &tau, double &sum) {
    const uint32_t lane = lane_id();
    uint64_t head[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t t = lane + 64u * r;
        head[r] = kNone;
        if (t < S && X.mlim[t] > 0) head[r] = Q.ranks[(uint64_t)X.mnode[t] * k];
    }
    for (;;) {
        uint64_t lmin = kNone;
#pragma unroll
        for (int r = 0; r < R; ++r) lmin = head[r] < lmin ? head[r] : lmin;
        const uint64_t g = group_min_u64<64>(lmin);
        if (g == kNone) break;
        // advance the holders of g; for CK also find their largest threshold
        uint64_t tmax = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (head[r] == g) {
                const uint32_t t = lane + 64u * r;
                const uint32_t u = X.mnode[t];
                const uint32_t p = X.mpos[t] + 1u;
                X.mpos[t] = (uint16_t)p;
                head[r] = p < X.mlim[t] ? Q.ranks[(uint64_t)u * k + p] : kNone;
                if (Q.estimator == 1) {
                    const uint64_t tu = Q.size[u] >= k ? Q.ranks[(uint64_t)u * k + k - 1] : kNone;
                    tmax = tu > tmax ? tu : tmax;
                }
            }
        }
        if (Q.estimator == 1) {
            tmax = ~group_min_u64<64>(~tmax);
            // the weight 1/r of the largest holder threshold: r = rho(T) for
            // hashed ranks, (T - 1)/(l n - 1) for permutation positions
            sum += tmax == kNone ? 1.0
                   : Q.perm_d    ? ((double)Q.perm_d - 1.0) / (double)(tmax - 1)
                                 : 1.0 / rank_real(tmax);
        } else {
            ++d;
            if (d == k) {
                tau = g;
                break;
            }
        }
    }
}

__device__ __forceinline__ double union_estimate(const QArgs &Q, uint32_t d, uint64_t tau) {
    return Q.perm_d ? perm_estimate(d, tau, Q.k, Q.ell, Q.perm_d)
                    : bottomk_estimate(d, tau, Q.k, Q.ell);
}

__device__ __forceinline__ void put_answer(const QArgs &Q, uint64_t j, double est, int32_t status) {
    Q.est[j] = est;
    if (Q.qstatus) Q.qstatus[j] = status;
}

// Cohen-Kaplan answer of query j (members qnodes[a .. a + S), S >= 1) by the
// whole wave's merge.
__device__ void ck_wave(const QArgs &Q, uint64_t j, uint64_t a, uint64_t S, MergeLds &X) {
    const uint32_t lane = lane_id();
    const uint32_t k = Q.k;
    // membership checks (node ids are validated per query)
    bool bad = false;
    for (uint64_t t = a + lane; t < a + S; t += 64) bad |= Q.qnodes[t] >= Q.n;
    bad = __ballot(bad) != 0;
    if (bad || S > kMaxMembers) {
        if (lane == 0) put_answer(Q, j, 0.0, bad ? -1 : -2);
        return;
    }
    // member state: node, next position, usable length
    for (uint32_t t = lane; t < S; t += 64) {
        const uint32_t u = Q.qnodes[a + t];
        const uint32_t sz = Q.size[u];
        X.mnode[t] = u;
        X.mpos[t] = 0;
        X.mlim[t] = (uint16_t)(sz >= k ? k - 1 : sz);  // without a full sketch's threshold
    }
    wave_sync();
    uint32_t d = 0;
    uint64_t tau = 0;
    double sum = 0.0;
    if (S <= 64) merge_members<1>(Q, S, k, X, d, tau, sum);
    else if (S <= 256) merge_members<4>(Q, S, k, X, d, tau, sum);
    else merge_members<kPerLane>(Q, S, k, X, d, tau, sum);
    if (lane == 0) put_answer(Q, j, sum / (double)Q.ell, 0);
    wave_sync();  // X is refilled by the next query
}

// --------------------------------------------------- bottom-k, small sets
// One query per aligned group of G lanes, S <= G R members (member t = lane
// in group + G r).  The group's minimum is 2 log2(G) vector-unit steps; each
// member keeps its head and the rank after it in registers, so a member that
// advances does not wait for memory unless it advances twice in a row.
// Groups without a query (S = 0) idle.
template <int G, int R>
__device__ __forceinline__ void merge_group(const QArgs &Q, uint64_t j, const uint32_t *nodes,
                                            uint32_t S) {
    const uint32_t gl = lane_id() & (G - 1), k = Q.k;
    uint32_t node[R];
    bool bad = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t t = gl + G * r;
        node[r] = t < S ? nodes[t] : 0u;
        bad |= t < S && node[r] >= Q.n;
    }
    {
        const unsigned long long m = __ballot(bad);
        const uint32_t g0 = lane_id() & ~(uint32_t)(G - 1);
        bad = ((m >> g0) & (G == 64 ? ~0ull : (1ull << (G & 63)) - 1ull)) != 0;
    }
    const bool mine = S > 0;
    uint64_t head[R], next[R];
    const uint64_t *at[R];  // the rank after `next`
    uint32_t left[R];       // ranks from there on
#pragma unroll
    for (int r = 0; r < R; ++r) {
        head[r] = next[r] = kNone;
        left[r] = 0;
        at[r] = Q.ranks;
        if (gl + G * r < S && !bad) {
            const uint32_t sz = Q.size[node[r]], lim = sz < k ? sz : k;
            const uint64_t *row = Q.ranks + (uint64_t)node[r] * k;
            if (lim > 0) head[r] = row[0];
            if (lim > 1) next[r] = row[1];
            left[r] = lim > 2 ? lim - 2 : 0;
            at[r] = row + 2;
        }
    }
    uint32_t d = 0;
    uint64_t tau = 0;
    bool open = mine && !bad;
    for (;;) {
        uint64_t lmin = head[0];
#pragma unroll
        for (int r = 1; r < R; ++r) lmin = head[r] < lmin ? head[r] : lmin;
        const uint64_t g = group_min_u64<G>(lmin);
        if (open) {
            if (g == kNone) {
                open = false;
            } else if (++d == k) {
                tau = g;
                open = false;
            }
        }
        if (!__any(open)) break;
        if (open) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (head[r] == g) {
                    head[r] = next[r];
                    next[r] = kNone;
                    if (left[r]) {
                        next[r] = *at[r]++;
                        --left[r];
                    }
                }
        }
    }
    if (mine && gl == 0) put_answer(Q, j, bad ? 0.0 : union_estimate(Q, d, tau), bad ? -1 : 0);
}

// One set alone in its workgroup (k_query_each), S <= G members: the
// first ranks of every row go to LDS at once, one memory latency instead of
// one in most steps (a member takes about k / S steps in a row's order, so
// the rest is rarely reached), and lane t merges member t from there.  Bound by
// the chain of k steps: 16 lognormal sets over k = 256 (20,000 nodes), a batch
// call, 159 us with steps in global memory and LDS permutes, 102 so.
constexpr uint32_t kStagedRanks = sizeof(MergeLds) / sizeof(uint64_t);
template <uint32_t G>
__device__ __forceinline__ void merge_staged(const QArgs &Q, uint64_t j, const uint32_t *nodes,
                                             uint32_t S, uint64_t *rows) {
    const uint32_t lane = lane_id(), k = Q.k;
    const uint32_t u = lane < S ? nodes[lane] : 0u;
    if (__any(u >= Q.n)) {
        if (lane == 0) put_answer(Q, j, 0.0, -1);
        return;
    }
    const uint32_t c = min(k, kStagedRanks / S);  // ranks of a row in LDS, >= 16
    uint32_t lim = 0;
    if (lane < S) {
        const uint32_t sz = Q.size[u];
        lim = sz < k ? sz : k;
    }
#pragma unroll 16
    for (uint32_t x0 = 0; x0 < S * c; x0 += 64) {  // every lane takes part in the shuffles
        const uint32_t x = x0 + lane, t = min(x / c, S - 1);
        const uint64_t ur = (uint32_t)__shfl((int)u, (int)t);
        if (x < S * c) rows[x] = Q.ranks[ur * k + (x - t * c)];
    }
    wave_sync();
    const uint64_t *row = rows + lane * c, *all = Q.ranks + (uint64_t)u * k;
    uint64_t head = lim > 0 ? row[0] : kNone, next = lim > 1 ? row[1] : kNone;
    uint32_t at = 2, d = 0;
    uint64_t tau = 0;
    for (;;) {
        uint64_t g = group_min_u64<G>(head);
        if (G < 64) g = shfl_u64(g, 0);  // the other lanes hold no member
        if (g == kNone) break;
        if (++d == k) {
            tau = g;
            break;
        }
        if (head == g) {
            head = next;
            next = at < lim ? (at < c ? row[at] : all[at]) : kNone;
            ++at;
        }
    }
    if (lane == 0) put_answer(Q, j, union_estimate(Q, d, tau), 0);
    wave_sync();  // the rows' LDS is reused
}

// Ascending sort of one key per lane.
__device__ __forceinline__ uint64_t sort_lanes(uint64_t x) {
    const uint32_t lane = lane_id();
    // merge runs of 1, 2, .. 32 lanes: the mirrored partner first, then halves
    x = keep_of(x, lane_xor64<1>(x), !(lane & 1));
    x = keep_of(x, lane_xor64<3>(x), !(lane & 2));
    x = keep_of(x, lane_xor64<1>(x), !(lane & 1));
    x = keep_of(x, lane_xor64<7>(x), !(lane & 4));
    x = keep_of(x, lane_xor64<2>(x), !(lane & 2));
    x = keep_of(x, lane_xor64<1>(x), !(lane & 1));
    x = keep_of(x, lane_xor64<15>(x), !(lane & 8));
    x = keep_of(x, lane_xor64<4>(x), !(lane & 4));
    x = keep_of(x, lane_xor64<2>(x), !(lane & 2));
    x = keep_of(x, lane_xor64<1>(x), !(lane & 1));
    x = keep_of(x, lane_xor64<31>(x), !(lane & 16));
    x = keep_of(x, lane_xor64<8>(x), !(lane & 8));
    x = keep_of(x, lane_xor64<4>(x), !(lane & 4));
    x = keep_of(x, lane_xor64<2>(x), !(lane & 2));
    x = keep_of(x, lane_xor64<1>(x), !(lane & 1));
    x = keep_of(x, lane_xor64<63>(x), !(lane & 32));
    x = keep_of(x, lane_xor64<16>(x), !(lane & 16));
    x = keep_of(x, lane_xor64<8>(x), !(lane & 8));
    x = keep_of(x, lane_xor64<4>(x), !(lane & 4));
    x = keep_of(x, lane_xor64<2>(x), !(lane & 2));
    return keep_of(x, lane_xor64<1>(x), !(lane & 1));
}

// The k-th smallest distinct one of the lanes' values (kNone: none of so many).
__device__ __forceinline__ uint64_t bottomk_bound(uint64_t least, uint32_t k) {
    const uint32_t lane = lane_id();
    const uint64_t x = sort_lanes(least);
    const uint64_t before = shfl_u64(x, lane ? lane - 1 : 0);
    const unsigned long long first = __ballot(x != kNone && (lane == 0 || x != before));
    if ((uint32_t)__popcll(first) < k) return kNone;
    const bool at = ((first >> lane) & 1ull) &&
                    (uint32_t)__popcll(first & ((1ull << lane) - 1ull)) == k - 1;
    return shfl_u64(x, (uint32_t)__ffsll((long long)__ballot(at)) - 1);
}

// Bottom-k of a set of more than 64 members, by the whole wave.  Each lane
// takes the smallest head of its 16 members; the k-th smallest distinct one of
// those 64 is a value of the union with at least k - 1 distinct values below
// it, so members whose head lies above it cannot contribute.  What is left
// (little more than k members) is merged.
__device__ __forceinline__ int bottomk_filter(const QArgs &Q, uint64_t j, uint64_t a, uint64_t S,
                                              MergeLds &X) {
    const uint32_t lane = lane_id(), k = Q.k;
    bool bad = false;
    for (uint64_t t = a + lane; t < a + S; t += 64) bad |= Q.qnodes[t] >= Q.n;
    bad = __ballot(bad) != 0;
    if (bad || S > kMaxMembers) {
        if (lane == 0) put_answer(Q, j, 0.0, bad ? -1 : -2);
        return -1;
    }
    uint64_t head[kPerLane], least = kNone;
#pragma unroll
    for (int r = 0; r < kPerLane; ++r) {
        const uint32_t t = lane + 64u * r;
        head[r] = kNone;
        if (t < S) {
            const uint32_t u = Q.qnodes[a + t];
            if (Q.size[u]) head[r] = Q.ranks[(uint64_t)u * k];
        }
        least = head[r] < least ? head[r] : least;
    }
    const uint64_t bound = bottomk_bound(least, k);
    uint32_t kept = 0;
#pragma unroll
    for (int r = 0; r < kPerLane; ++r) {
        const bool keep = head[r] != kNone && head[r] <= bound;
        const unsigned long long m = __ballot(keep);
        if (keep)
            X.mnode[kept + __popcll(m & ((1ull << lane) - 1ull))] = Q.qnodes[a + lane + 64u * r];
        kept += (uint32_t)__popcll(m);
    }
    wave_sync();
    return (int)kept;
}
__device__ __forceinline__ void bottomk_kept(const QArgs &Q, uint64_t j, uint32_t kept, MergeLds &X) {
    const uint32_t lane = lane_id(), k = Q.k;
    if (kept <= 64) {
        if (kept) merge_group<64, 1>(Q, j, X.mnode, kept);
        else if (lane == 0) put_answer(Q, j, union_estimate(Q, 0, 0), 0);
    } else {
        for (uint32_t t = lane; t < kept; t += 64) {
            const uint32_t sz = Q.size[X.mnode[t]];
            X.mpos[t] = 0;
            X.mlim[t] = (uint16_t)(sz < k ? sz : k);
        }
        wave_sync();
        uint32_t d = 0;
        uint64_t tau = 0;
        double sum = 0.0;
        if (kept <= 256) merge_members<4>(Q, kept, k, X, d, tau, sum);
        else merge_members<kPerLane>(Q, kept, k, X, d, tau, sum);
        if (lane == 0) put_answer(Q, j, union_estimate(Q, d, tau), 0);
    }
    wave_sync();  // X is refilled by the next query
}
__device__ __forceinline__ void bottomk_wave(const QArgs &Q, uint64_t j, uint64_t a, uint64_t S,
                                             MergeLds &X) {
    const int kept = bottomk_filter(Q, j, a, S, X);
    if (kept >= 0) bottomk_kept(Q, j, (uint32_t)kept, X);
}

// A run of queries' offsets, one per lane, and the lanes of one size class.
struct Run {
    uint64_t j0, a, S;  // first query; this lane's set
    uint8_t *list;      // [64] LDS
};

// The lanes with `in` set, in order, into the list; their number.
__device__ __forceinline__ uint32_t list_class(const Run &run, bool in) {
    const uint32_t lane = lane_id();
    const unsigned long long m = __ballot(in);
    wave_sync();  // the previous class has been read
    if (in) run.list[__popcll(m & ((1ull << lane) - 1ull))] = (uint8_t)lane;
    wave_sync();
    return (uint32_t)__popcll(m);
}

template <int G, int R>
__device__ __forceinline__ void run_class(const QArgs &Q, const Run &run, bool in) {
    const uint32_t total = list_class(run, in);
    for (uint32_t base = 0; base < total; base += 64 / G) {
        const uint32_t x = base + lane_id() / G;
        const uint32_t src = x < total ? run.list[x] : 0u;
        const uint64_t a = shfl_u64(run.a, src);
        const uint32_t S = (uint32_t)__shfl((int)(uint32_t)run.S, (int)src);
        merge_group<G, R>(Q, run.j0 + src, Q.qnodes + a, x < total ? S : 0u);
    }
}

// Offsets of set j.  They are validated before a batch; a replayed plan
// re-checks its own sets here (non-decreasing, within qoff[q]) and never reads
// outside.
__device__ __forceinline__ bool set_bounds(const QArgs &Q, uint64_t j, uint64_t &a, uint64_t &b) {
    a = Q.qoff[j];
    b = Q.qoff[j + 1];
    return !(b < a || b > Q.qoff[Q.q] || b > Q.nodes_cap || (j == 0 && a != 0));
}

// Offsets of query j0 + lane (lane < cnt).  Empty sets and bad offsets are
// answered; returns whether a set with members is left.
__device__ __forceinline__ bool load_run(const QArgs &Q, uint32_t cnt, Run &run) {
    const uint32_t lane = lane_id();
    run.a = run.S = 0;
    if (lane >= cnt) return false;
    const uint64_t j = run.j0 + lane;
    uint64_t a, b;
    if (!set_bounds(Q, j, a, b)) {
        put_answer(Q, j, 0.0, -3);
        return false;
    }
    if (a == b) {
        put_answer(Q, j, 0.0, 0);
        return false;
    }
    run.a = a;
    run.S = b - a;
    return true;
}

// Bottom-k answer of query j, one node, by the calling lane.
__device__ __forceinline__ void single_node(const QArgs &Q, uint64_t j, uint32_t u) {
    if (u >= Q.n) {
        put_answer(Q, j, 0.0, -1);
        return;
    }
    const uint32_t sz = Q.size[u];
    const uint64_t T = sz >= Q.k ? Q.ranks[(uint64_t)u * Q.k + Q.k - 1] : 0;
    put_answer(Q, j, union_estimate(Q, sz, T), 0);
}

// Bottom-k answers of queries j0 .. j0 + cnt (cnt <= 64), by set size: one
// lane for a single node, groups of 4, 8 and 16 lanes up to 64 members (16
// lanes with 2 or 4 members each measured faster than a wave with one each),
// the wave above.
__device__ __forceinline__ void answer_bottomk(const QArgs &Q, uint64_t j0, uint32_t cnt,
                                               MergeLds &X, uint8_t *list) {
    Run run{j0, 0, 0, list};
    const bool set = load_run(Q, cnt, run);
    if (set && run.S == 1) single_node(Q, j0 + lane_id(), Q.qnodes[run.a]);
    run_class<4, 1>(Q, run, set && run.S >= 2 && run.S <= 4);
    run_class<8, 1>(Q, run, set && run.S >= 5 && run.S <= 8);
    run_class<16, 1>(Q, run, set && run.S >= 9 && run.S <= 16);
    run_class<16, 2>(Q, run, set && run.S >= 17 && run.S <= 32);
    run_class<16, 4>(Q, run, set && run.S >= 33 && run.S <= 64);
    unsigned long long rest = __ballot(set && run.S > 64);
    while (rest) {
        const uint32_t src = (uint32_t)__ffsll((long long)rest) - 1;
        rest &= rest - 1;
        bottomk_wave(Q, j0 + src, shfl_u64(run.a, src), shfl_u64(run.S, src), X);
    }
}

// ------------------------------------------- Cohen-Kaplan, sorted in registers
// A set of S <= 2^LG <= 64 members over sketches of k <= R ranks: one lane per
// member holds its R ranks (ascending) in registers; 2^LG lanes merge theirs
// by LG levels of a bitonic network (the first step of a level meets the
// mirrored partner, the steps inside a lane need no cross-lane move), after
// which lane t of the group holds the group's ranks R t .. R t + R - 1 in
// order.  A wave sorts 64 >> LG sets at once.
//
// The keys are the ranks' leading 52 bits (after dropping the zeros common to
// the group) over a 12-bit index (member lane, place), which finds the
// holder's weight afterwards.  Two ranks that agree in those 52 bits and
// differ below could come out in the wrong order: the dropped bits, kept in
// LDS, are compared for every pair of neighbours, and such a set (about one
// in 10^9 for hashed ranks) is answered by the merge instead.
//
// What bounds it: vector-unit instructions (24,000 per set of 50 over k = 64)
// at two waves per SIMD; with 64 ranks a lane part of the keys is in scratch (300
// to 372 bytes a lane), with up to 32 none.  The merge it replaces made one serial step of two
// wave-wide reductions and three dependent loads per distinct value: 20,000
// sets of 50 over a 10^6-node table, 23.9 -> 1.16 ms.
struct CkLds {
    uint64_t stage[64 * 17];  // 16 ranks of every lane, rows padded to 17
    double w[64];             // 1/r of each lane's member threshold
};

template <int R, int kMask> __device__ __forceinline__ void ck_flip(uint64_t (&x)[R], bool low) {
#pragma unroll
    for (int r = 0; r < R / 2; ++r) {
        const uint64_t a = x[r], b = x[R - 1 - r];
        const uint64_t pa = lane_xor64<kMask>(b), pb = lane_xor64<kMask>(a);
        x[r] = keep_of(a, pa, low);
        x[R - 1 - r] = keep_of(b, pb, low);
    }
}
template <int R, int kMask> __device__ __forceinline__ void ck_step(uint64_t (&x)[R], bool low) {
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = keep_of(x[r], lane_xor64<kMask>(x[r]), low);
}
template <int R> __device__ __forceinline__ void ck_inside(uint64_t (&x)[R]) {
#pragma unroll
    for (int s = R / 2; s > 0; s >>= 1)
#pragma unroll
        for (int r = 0; r < R; ++r)
            if ((r & s) == 0) {
                const uint64_t a = x[r], b = x[r | s];
                const bool c = a < b;
                x[r] = c ? a : b;
                x[r | s] = c ? b : a;
            }
}

// Lanes of a group of 2^LG: node u (S valid lanes from the group's first; S =
// 0: no query), all ids valid.  Returns the group's weight sum in every lane
// and whether it must be merged instead.
template <int R>
__device__ __forceinline__ double ck_sorted(const QArgs &Q, uint32_t LG, uint32_t u, bool member,
                                            CkLds &L, bool &redo) {
    const uint32_t lane = lane_id(), k = Q.k, G = 1u << LG;
    uint32_t lim = 0;
    uint64_t last = 0;  // the member's largest usable rank
    {
        double w = 0.0;
        if (member) {
            const uint32_t sz = Q.size[u];
            const uint64_t *row = Q.ranks + (uint64_t)u * k;
            lim = sz >= k ? k - 1 : sz;  // a full sketch's threshold does not count
            if (lim) last = row[lim - 1];
            w = 1.0;
            if (sz >= k) {
                const uint64_t t = row[k - 1];
                w = Q.perm_d ? ((double)Q.perm_d - 1.0) / (double)(t - 1) : 1.0 / rank_real(t);
            }
        }
        L.w[lane] = w;
    }
    // 16 places of every lane's row at a time through LDS, so that the loads
    // take whole lines
    uint64_t x[R];
#pragma unroll
    for (int c = 0; c < R / 16; ++c) {
        uint64_t v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint32_t src = 4 * i + (lane >> 4), p = 16 * c + (lane & 15);
            const uint32_t ur = (uint32_t)__shfl((int)u, (int)src);
            const uint32_t lr = (uint32_t)__shfl((int)lim, (int)src);
            v[i] = p < lr ? Q.ranks[(uint64_t)ur * k + p] : kNone;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) L.stage[(4 * i + (lane >> 4)) * 17 + (lane & 15)] = v[i];
        wave_sync();
#pragma unroll
        for (int q = 0; q < 16; ++q) x[16 * c + q] = L.stage[lane * 17 + q];
        wave_sync();
    }
    uint32_t total = lim;
    for (uint32_t off = 1; off < G; off <<= 1) {
        last |= ((uint64_t)__shfl_xor((uint32_t)(last >> 32), (int)off) << 32) |
                __shfl_xor((uint32_t)last, (int)off);
        total += __shfl_xor(total, (int)off);
    }
    const uint32_t sh = last ? (uint32_t)__clzll((long long)last) : 0u;
    uint16_t *low12 = (uint16_t *)L.stage;  // [64][64] by index
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint64_t z = x[r] << sh;
        low12[lane * 64 + r] = (uint16_t)(z & 0xFFFu);
        // a valid key is never all ones: place 63 is never usable
        x[r] = r < (int)lim ? (z & ~0xFFFull) | (lane << 6) | r : kNone;
    }
    wave_sync();
    for (uint32_t lv = 1; lv <= LG; ++lv) {  // uniform
        const bool lowhalf = (lane & (1u << (lv - 1))) == 0;
        if (lv == 1) ck_flip<R, 1>(x, lowhalf);
        else if (lv == 2) ck_flip<R, 3>(x, lowhalf);
        else if (lv == 3) ck_flip<R, 7>(x, lowhalf);
        else if (lv == 4) ck_flip<R, 15>(x, lowhalf);
        else if (lv == 5) ck_flip<R, 31>(x, lowhalf);
        else ck_flip<R, 63>(x, lowhalf);
        for (int st = (int)lv - 2; st >= 0; --st) {
            const bool low = (lane & (1u << st)) == 0;
            if (st == 4) ck_step<R, 16>(x, low);
            else if (st == 3) ck_step<R, 8>(x, low);
            else if (st == 2) ck_step<R, 4>(x, low);
            else if (st == 1) ck_step<R, 2>(x, low);
            else ck_step<R, 1>(x, low);
        }
        ck_inside<R>(x);
    }
    // eq bit r: place r holds the same rank as the place before it
    uint64_t eq = 0;
    redo = false;
    {
        uint64_t prev = shfl_u64(x[R - 1], lane ? lane - 1 : 0);
        if ((lane & (G - 1)) == 0) prev = kNone;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint64_t cur = x[r];
            if (((cur ^ prev) >> 12) == 0 && cur != kNone && prev != kNone) {
                if (low12[cur & 0xFFFu] == low12[prev & 0xFFFu]) eq |= 1ull << r;
                else redo = true;
            }
            prev = cur;
        }
    }
    // weights; the smallest of a run of equal ranks (the largest threshold
    // among its holders) counts, at the run's last place
    double run = __builtin_huge_val();  // of a run that began in an earlier lane
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const double w = x[r] == kNone ? 0.0 : L.w[(x[r] >> 6) & 63u];
        x[r] = (uint64_t)__double_as_longlong(w);
        run = ((eq >> r) & 1ull) ? fmin(run, w) : w;
    }
    {   // runs that continue from earlier lanes: segmented minimum over lanes
        const uint64_t all = R == 64 ? ~0ull : (1ull << R) - 1ull;
        double v = run;                      // of the lane's last run
        uint32_t open = (eq & all) == all;   // which began in an earlier lane
        for (uint32_t off = 1; off < G; off <<= 1) {
            const uint64_t vu = shfl_u64((uint64_t)__double_as_longlong(v), lane >= off ? lane - off : 0);
            const uint32_t ou = (uint32_t)__shfl((int)open, (int)(lane >= off ? lane - off : 0));
            if (open && (lane & (G - 1)) >= off) {
                v = fmin(v, __longlong_as_double((long long)vu));
                open = ou;
            }
        }
        run = __longlong_as_double(
            (long long)shfl_u64((uint64_t)__double_as_longlong(v), lane ? lane - 1 : 0));
    }
    const uint32_t eq_next = (uint32_t)__shfl((int)((uint32_t)eq & 1u), (int)((lane + 1) & 63u));
    const bool goes_on = eq_next && ((lane + 1) & (G - 1)) != 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const double w = __longlong_as_double((long long)x[r]);
        run = ((eq >> r) & 1ull) ? fmin(run, w) : w;
        const bool ends = r < R - 1 ? !((eq >> (r + 1)) & 1ull) : !goes_on;
        x[r] = (uint64_t)__double_as_longlong(ends ? run : 0.0);
    }
    // the sum in increasing order of the ranks, lane after lane (a place
    // inside a run adds 0.0, which changes nothing)
    double sum = 0.0;
    for (uint32_t t = 0; t < G; ++t) {
        if (!__any(t * R < total)) break;
        double s = sum;
#pragma unroll
        for (int r = 0; r < R; ++r) s += __longlong_as_double((long long)x[r]);
        sum = __longlong_as_double((long long)shfl_u64((uint64_t)__double_as_longlong(s),
                                                       (lane & ~(G - 1)) + t));
    }
    wave_sync();  // L is refilled by the next sets
    return sum;
}

// small_only: sets of more than 64 members are left to k_ck_large.
template <int R>
__device__ __forceinline__ void answer_ck(const QArgs &Q, uint64_t j0, uint32_t cnt, MergeLds &X,
                                          CkLds &L, uint8_t *list, bool small_only) {
    const uint32_t lane = lane_id();
    Run run{j0, 0, 0, list};
    const bool set = load_run(Q, cnt, run);
    unsigned long long rest = __ballot(set && (R == 0 || (run.S > 64 && !small_only)));
    if constexpr (R > 0) {
        for (uint32_t LG = 0; LG <= 6; ++LG) {
            const uint32_t G = 1u << LG;
            const uint32_t total =
                list_class(run, set && run.S <= G && (LG == 0 || run.S > G / 2));
            for (uint32_t base = 0; base < total; base += 64 >> LG) {
                const uint32_t x = base + (lane >> LG), gl = lane & (G - 1);
                const bool mine = x < total;
                const uint32_t src = mine ? list[x] : 0u;
                const uint64_t a = shfl_u64(run.a, src);
                const uint32_t S = (uint32_t)__shfl((int)(uint32_t)run.S, (int)src);
                const bool member = mine && gl < S;
                uint32_t u = member ? Q.qnodes[a + gl] : 0u;
                const unsigned long long gm = (LG == 6 ? ~0ull : (1ull << G) - 1ull)
                                              << (lane & ~(G - 1));
                const bool bad = (__ballot(member && u >= Q.n) & gm) != 0;
                if (bad) u = 0;
                bool redo = false;
                const double sum = ck_sorted<R>(Q, LG, u, member && !bad, L, redo);
                redo = (__ballot(redo) & gm) != 0;
                if (mine && gl == 0 && !redo)
                    put_answer(Q, j0 + src, bad ? 0.0 : sum / (double)Q.ell, bad ? -1 : 0);
                for (unsigned long long m = __ballot(mine && gl == 0 && redo); m; m &= m - 1)
                    rest |= 1ull << list[base + ((uint32_t)(__ffsll((long long)m) - 1) >> LG)];
            }
        }
    }
    while (rest) {
        const uint32_t src = (uint32_t)__ffsll((long long)rest) - 1;
        rest &= rest - 1;
        ck_wave(Q, j0 + src, shfl_u64(run.a, src), shfl_u64(run.S, src), X);
    }
}

// kCk: -1 bottom-k, else Cohen-Kaplan with kCk registers per lane (0: only
// the merge, for k > 64).
template <int kCk> struct QueryLds {
    union {
        MergeLds merge;
        CkLds ck;
    };
    uint8_t list[64];
};
template <int kCk>
__device__ __forceinline__ void answer_run(const QArgs &Q, uint64_t j0, uint32_t cnt,
                                           QueryLds<kCk> &X, bool small_only) {
    if constexpr (kCk < 0) answer_bottomk(Q, j0, cnt, X.merge, X.list);
    else answer_ck<kCk>(Q, j0, cnt, X.merge, X.ck, X.list, small_only);
}

// The sets [j0, j1) of this wave where every wave of the grid takes a contiguous
// share of equal weight: set j begins at weight qoff[j] + kSetWeight j, and wave w
// takes those that begin in [w, w + 1) times the w-th part of the whole.  Both
// ends are searched for together, 32 places of the offsets at a time.  (Offsets
// out of order, which only a replayed plan can meet, give some share or other; the
// shares begin at 0, end at q and follow each other, so no set is left out.)
__device__ __forceinline__ void wave_share(const QArgs &Q, uint64_t q, uint64_t &j0, uint64_t &j1) {
    const uint32_t lane = lane_id(), half = lane >> 5, hl = lane & 31u;
    const uint64_t target = (Q.qoff[q] + kSetWeight * q) * (blockIdx.x + half) / gridDim.x;
    uint64_t lo = 0, hi = q;  // the first place of weight `target` or more lies in [lo, hi]
    while (__any(lo < hi)) {
        const uint64_t step = (hi - lo + 31) / 32, x = lo + step * (hl + 1) - 1;
        const bool in = lo < hi && x < hi;
        const bool below = in && Q.qoff[x] + kSetWeight * x < target;
        const uint32_t m = (uint32_t)(__ballot(below) >> (32 * half));
        const uint32_t c = ~m ? (uint32_t)__ffs((int)~m) - 1u : 32u;  // places below the target
        if (lo < hi) {
            lo += step * c;
            if (c < 32 && lo + step - 1 < hi) hi = lo + step - 1;  // that place is not below it
            lo = lo < hi ? lo : hi;
        }
    }
    j0 = shfl_u64(lo, 0);
    j1 = blockIdx.x + 1 == gridDim.x ? q : shfl_u64(lo, 32);
}

// Whether the sets' weight is spread over the batch: no 64th part of it holds half
// as much again as its share.
__device__ __forceinline__ bool balanced(const QArgs &Q, uint64_t q) {
    const uint64_t x0 = q * lane_id() / 64, x1 = q * (lane_id() + 1) / 64;
    const uint64_t w = Q.qoff[x1] - Q.qoff[x0] + kSetWeight * (x1 - x0);
    return !__any(128 * w > 3 * (Q.qoff[q] + kSetWeight * q));
}

template <int kCk>
__global__ void __launch_bounds__(kQBlock, kCk < 0 ? 4 : kCk == 16 ? 3 : 2) k_query_persistent(
    QArgs Q, uint64_t q, unsigned long long *next, bool small_only) {
    __shared__ QueryLds<kCk> X;
    // Takes from different waves on the one counter are serialised by the
    // hardware (about 12 ns each).  Sets of less than kTakeMembers members on
    // average cost less than that.  They go in equal runs, every wave the same
    // number of them, spread over the batch, if that is balanced (see there), and
    // else, or if a large set costs far more than its members' share (Cohen-Kaplan),
    // each wave takes a share of equal weight.  10^6 lognormal sets, mean 12, a call:
    // 0.51 ms in runs, 0.61 in shares (a share's ends are looked for in cold lines);
    // sorted by size 0.85 and 0.54; 1000 sets of 1024 nodes before 99,000 of one, k =
    // 64: 1.73 and 0.15.  Batches of larger sets are taken from the counter, in runs
    // that shrink as it drains (at most kRun, about a quarter of an even share of
    // what is left).
    const uint64_t part = 4ull * gridDim.x;
    const bool counter = Q.qoff[q] >= kTakeMembers * q;
    uint64_t g = q / part, j0 = 0, end = q, step = 0;
    g = g < 1 ? 1 : g > kRun ? kRun : g;
    if (!counter) {
        if (kCk < 0 && balanced(Q, q)) {
            const uint64_t rounds = (q + (uint64_t)gridDim.x * kRun - 1) / ((uint64_t)gridDim.x * kRun);
            g = (q + gridDim.x * rounds - 1) / (gridDim.x * rounds);  // <= kRun
            step = gridDim.x * g;
            j0 = blockIdx.x * g;
        } else {
            step = g = kRun;
            wave_share(Q, q, j0, end);
        }
    }
    for (;; j0 += step) {  // one call site: the answering code is large
        if (counter) {
            unsigned long long at = 0;
            if (threadIdx.x == 0) at = atomicAdd(next, (unsigned long long)g);
            j0 = shfl_u64(at, 0);
        }
        if (j0 >= end) break;
        const uint64_t j1 = j0 + g < end ? j0 + g : end;
        answer_run<kCk>(Q, j0, (uint32_t)(j1 - j0), X, small_only);
        if (counter) {
            g = (q - j1) / part;
            g = g < 1 ? 1 : g > kRun ? kRun : g;
        }
    }
}

// One query per workgroup, queries j0 on: a batch within the grid (no counter
// to reset), or the plain path's launch for one query.
template <int kCk>
__global__ void __launch_bounds__(kQBlock, 2) k_query_each(QArgs Q, uint64_t j0, bool small_only) {
    __shared__ QueryLds<kCk> X;
    const uint64_t j = j0 + blockIdx.x;
    if constexpr (kCk < 0) {
        Run run{j, 0, 0, X.list};
        load_run(Q, 1, run);
        const uint64_t a = shfl_u64(run.a, 0), S = shfl_u64(run.S, 0);
        uint64_t *rows = (uint64_t *)&X.merge;
        if (S == 0) return;
        if (S == 1) {  // (stepping to the k-th rank of the one row, k = 256: 97 us a call for 39)
            if (threadIdx.x == 0) single_node(Q, j, Q.qnodes[a]);
        } else if (S <= 16) merge_staged<16>(Q, j, Q.qnodes + a, (uint32_t)S, rows);
        else if (S <= 64) merge_staged<64>(Q, j, Q.qnodes + a, (uint32_t)S, rows);
        else bottomk_wave(Q, j, a, S, X.merge);
    } else {
        answer_run<kCk>(Q, j, 1, X, small_only);
    }
}

// The Cohen-Kaplan answers of a batch's sets of more than 64 members, in a launch
// of their own: their merge is a chain of dependent accesses (S (k - 1) steps at
// most), which wants as many waves as fit, and the kernels that sort the small
// sets in registers hold two per SIMD.  A set per wave, or shares of equal
// weight.  20,000 sets of 200 over k = 64: 74 ms; among the sorted sets 132, and 103
// with a wave-wide reduction by LDS permutes in each step.
__global__ void __launch_bounds__(kQBlock, 4) k_ck_large(QArgs Q, uint64_t q) {
    __shared__ MergeLds X;
    const uint32_t lane = lane_id();
    uint64_t j0 = blockIdx.x, end = j0 + 1;
    if (q > gridDim.x) wave_share(Q, q, j0, end);
    for (; j0 < end; j0 += 64) {
        uint64_t a = 0, b = 0;
        const bool big = j0 + lane < end && set_bounds(Q, j0 + lane, a, b) && b - a > 64;
        for (unsigned long long rest = __ballot(big); rest; rest &= rest - 1) {
            const uint32_t src = (uint32_t)__ffsll((long long)rest) - 1;
            ck_wave(Q, j0 + src, shfl_u64(a, src), shfl_u64(b - a, src), X);
        }
    }
}

// The 64 smallest distinct keys of two ascending lists without repeats, a key
// per lane (kNone: none): x, and the other list read in descending order.
__device__ __forceinline__ uint64_t bitonic_merge(uint64_t x) {
    const uint32_t lane = lane_id();
    x = keep_of(x, lane_xor64<32>(x), !(lane & 32));
    x = keep_of(x, lane_xor64<16>(x), !(lane & 16));
    x = keep_of(x, lane_xor64<8>(x), !(lane & 8));
    x = keep_of(x, lane_xor64<4>(x), !(lane & 4));
    x = keep_of(x, lane_xor64<2>(x), !(lane & 2));
    return keep_of(x, lane_xor64<1>(x), !(lane & 1));
}
__device__ __forceinline__ uint64_t merge_rows(uint64_t x, uint64_t down, uint64_t *slot) {
    const uint32_t lane = lane_id();
    const uint64_t lo = bitonic_merge(x < down ? x : down);
    const uint64_t before = shfl_u64(lo, lane ? lane - 1 : 0);
    const unsigned long long rep = __ballot(lane && lo == before && lo != kNone);
    if (!rep) return lo;
    // what repeats leave free is filled from the upper half
    const uint64_t hi = bitonic_merge(x < down ? down : x);
    const uint64_t hb = shfl_u64(hi, lane ? lane - 1 : 0), last = shfl_u64(lo, 63);
    const unsigned long long hrep = __ballot(hi == (lane ? hb : last) && hi != kNone);
    const unsigned long long below = (1ull << lane) - 1ull;
    if (!((rep >> lane) & 1)) slot[__popcll(~rep & below)] = lo;
    const uint32_t at = 64 - (uint32_t)__popcll(rep) + (uint32_t)__popcll(~hrep & below);
    if (!((hrep >> lane) & 1) && at < 64) slot[at] = hi;
    wave_sync();
    x = slot[lane];
    wave_sync();
    return x;
}

// Few bottom-k queries over sketches of k <= 64, a workgroup each: its waves
// merge the members' rows (of more than 64 members those that can matter) two
// at a time, a rank per lane, and then each other's results, so the chain is
// S / kFewWaves + 3 merges of about 0.4 us where stepping through the union is k
// steps of 0.2 us.  Lognormal sets (20,000 nodes, mean 12), k = 64: 16 of them 22.7
// us a call by the kernel for larger batches, 7.6 to 8.4 so.  Batches whose largest
// set has 50 to 500 members: 64 sets 27.5 and 15.7, 1024 30.3 and 22.7, 2048 31.0
// and 29.8.  With k = 16 the steps are few: 64 sets 8.9 and 8.6 us, 256 sets 9.5 and
// 9.7.
constexpr int kFewWaves = 8;

// Where the entries of all sets are known and more than kFewMembers, most sets are
// far above 64 members: if many of those begin with the same rank (20,000 nodes)
// little is filtered, and the workgroups merge whole rows of which the steps read a
// part.  k = 64, a call: 1024 sets of 1024 entries 205 us and 117 by the kernel for
// larger batches, 1024 of 400 110 and 99; 64 of 1024 108, 300 of 400 79.
constexpr uint64_t kFewMembers = 1u << 17;
__host__ inline bool few_queries(uint32_t k, uint64_t q, uint64_t members) {
    return k <= 64 && q <= (k > 32 ? 1024u : 64u) && members <= kFewMembers;
}
static_assert(kMaxMembers == 2 * 64 * kFewWaves, "two members a lane");
__global__ void __launch_bounds__(64 * kFewWaves, 8) k_query_few(QArgs Q, uint64_t j0) {
    // 40 KiB: four workgroups per CU
    __shared__ uint64_t rows[8 * kFewWaves][64], slot[kFewWaves][64];
    __shared__ uint32_t mnode[kMaxMembers];
    const uint32_t lane = lane_id(), wave = threadIdx.x >> 6, k = Q.k;
    const uint64_t j = j0 + blockIdx.x;
    Run run{j, 0, 0, nullptr};
    if (wave == 0) load_run(Q, 1, run);  // answers empty sets and bad offsets
    uint64_t a, b;
    if (!set_bounds(Q, j, a, b) || a == b) return;
    uint32_t S = (uint32_t)(b - a), u;
    if (b - a <= 64) {
        u = lane < S ? Q.qnodes[a + lane] : 0u;
        if (__any(u >= Q.n)) {  // alike in all waves
            if (threadIdx.x == 0) put_answer(Q, j, 0.0, -1);
            return;
        }
    } else {
        // the members that can matter (see bottomk_bound), at most k if no heads
        // are equal: two members a lane over all waves
        bool bad = false;
        for (uint64_t t = a + threadIdx.x; t < b; t += 64 * kFewWaves) bad |= Q.qnodes[t] >= Q.n;
        const bool any = __any(bad);
        if (lane == 0) rows[1][wave] = any;
        __syncthreads();
        bad = __any(lane < kFewWaves && rows[1][lane]);
        if (bad || b - a > kMaxMembers) {
            if (threadIdx.x == 0) put_answer(Q, j, 0.0, bad ? -1 : -2);
            return;
        }
        uint32_t node[2];
        uint64_t head[2];
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const uint32_t t = threadIdx.x + 64 * kFewWaves * r;
            head[r] = kNone;
            node[r] = t < S ? Q.qnodes[a + t] : 0u;
            if (t < S && Q.size[node[r]]) head[r] = Q.ranks[(uint64_t)node[r] * k];
        }
        slot[wave][lane] = head[0] < head[1] ? head[0] : head[1];
        __syncthreads();
        uint64_t least = slot[0][lane];
#pragma unroll
        for (int w = 1; w < kFewWaves; ++w) least = slot[w][lane] < least ? slot[w][lane] : least;
        const uint64_t bound = bottomk_bound(least, k);  // alike in all waves
        const bool k0 = head[0] != kNone && head[0] <= bound, k1 = head[1] != kNone && head[1] <= bound;
        const unsigned long long m0 = __ballot(k0), m1 = __ballot(k1), below = (1ull << lane) - 1ull;
        if (lane == 0) rows[0][wave] = (uint64_t)(__popcll(m0) + __popcll(m1));
        __syncthreads();
        uint32_t at = 0;
        S = 0;
#pragma unroll
        for (uint32_t w = 0; w < kFewWaves; ++w) {
            at += w < wave ? (uint32_t)rows[0][w] : 0u;
            S += (uint32_t)rows[0][w];
        }
        if (k0) mnode[at + __popcll(m0 & below)] = node[0];
        if (k1) mnode[at + __popcll(m0) + __popcll(m1 & below)] = node[1];
        __syncthreads();  // (and rows and slot are used again)
        u = lane < S ? mnode[lane] : 0u;
    }
    // 64 members at a time, of them this wave's wave, wave + 8, ..: all their
    // rows on the way at once
    uint64_t x = kNone;
    for (uint32_t base = 0; base < S; base += 64) {
        if (base) u = base + lane < S ? mnode[base + lane] : 0u;
        const uint32_t cnt = min(S - base, 64u);
        const uint32_t sz = lane < cnt ? Q.size[u] : 0u, lim = sz < k ? sz : k;
        uint64_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t t = wave + kFewWaves * i;
            v[i] = kNone;
            if (t < cnt) {
                const uint64_t ut = (uint32_t)__builtin_amdgcn_readlane((int)u, (int)t);
                if (lane < k) v[i] = Q.ranks[ut * k + lane];
            }
        }
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const uint32_t t = wave + kFewWaves * i;
            const uint32_t lt = (uint32_t)__builtin_amdgcn_readlane((int)lim, (int)t);
            if (lane >= lt) v[i] = kNone;
            rows[8 * wave + i][lane] = v[i];
        }
        wave_sync();
        const uint32_t i0 = base ? 0u : 1u;
        if (!base) x = v[0];
        for (uint32_t i = i0; wave + kFewWaves * i < cnt; ++i)
            x = merge_rows(x, rows[8 * wave + i][63 - lane], slot[wave]);
    }
    for (uint32_t step = kFewWaves / 2; step > 0; step /= 2) {
        if (step >= S) continue;  // uniform
        rows[8 * wave][lane] = x;
        __syncthreads();
        if (wave < step && wave + step < S)
            x = merge_rows(x, rows[8 * (wave + step)][63 - lane], slot[wave]);
    }
    if (wave == 0) {
        const uint32_t d = (uint32_t)__popcll(__ballot(lane < k && x != kNone));
        const uint64_t tau = d >= k ? shfl_u64(x, k - 1) : 0ull;
        if (lane == 0) put_answer(Q, j, union_estimate(Q, d, tau), 0);
    }
}

template <int kCk> void launch_each(const QArgs &Q, uint64_t j0, unsigned grid, bool small_only,
                                    hipStream_t s) {
    k_query_each<kCk><<<grid, kQBlock, 0, s>>>(Q, j0, small_only);
}
void launch_each(const QArgs &Q, uint64_t j0, unsigned grid, bool small_only, hipStream_t s) {
    if (Q.estimator == 0 && few_queries(Q.k, grid, Q.members))
        k_query_few<<<grid, 64 * kFewWaves, 0, s>>>(Q, j0);
    else if (Q.estimator == 0) launch_each<-1>(Q, j0, grid, false, s);
    else if (Q.k <= 16) launch_each<16>(Q, j0, grid, small_only, s);
    else if (Q.k <= 32) launch_each<32>(Q, j0, grid, small_only, s);
    else if (Q.k <= 64) launch_each<64>(Q, j0, grid, small_only, s);
    else launch_each<0>(Q, j0, grid, false, s);
    SKIM_LAUNCH_CHECK();
}

// err: 1 and 2 for bad offsets, 4 if some set has more than 64 entries.
constexpr uint32_t kBadOffsets = 3u, kLargeSets = 4u;
__global__ void k_check_offsets(const uint64_t *qoff, uint64_t q, uint32_t *err) {
    uint32_t seen = 0;
    for (uint64_t j = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; j <= q;
         j += (uint64_t)gridDim.x * blockDim.x) {
        if (j == 0 && qoff[0] != 0) atomicOr(err, 1u);
        if (j < q && qoff[j + 1] < qoff[j]) atomicOr(err, 2u);
        if (__any(j < q && qoff[j + 1] - qoff[j] > 64) && !(seen & 4u)) {
            if (lane_id() == 0) atomicOr(err, 4u);
            seen = 4u;
        }
    }
}

}  // namespace

unsigned query_grid(uint64_t q) {
    static int cus = 0;
    if (!cus) {
        int dev = 0;
        cus = 256;
        if (hipGetDevice(&dev) == hipSuccess)
            (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        (void)hipGetLastError();
    }
    const uint64_t want = (uint64_t)cus * 16;
    return (unsigned)(q < want ? (q ? q : 1) : want);
}

void launch_queries_async(const QueryArgs &Q, uint64_t q, unsigned long long *next, hipStream_t s) {
    const unsigned grid = query_grid(q);
    // Cohen-Kaplan: large sets apart once the waves are more than fit on the
    // chip at two per SIMD (half the grid of a long batch)
    const bool apart = Q.estimator == 1 && Q.k <= 64 && Q.large && q > query_grid(~0ull) / 2;
    if (q <= grid) {
        launch_each(Q, 0, (unsigned)q, apart, s);
    } else {
        fill_u64((uint64_t *)next, 0, 1, s);
        if (Q.estimator == 0) k_query_persistent<-1><<<grid, kQBlock, 0, s>>>(Q, q, next, false);
        else if (Q.k <= 16) k_query_persistent<16><<<grid, kQBlock, 0, s>>>(Q, q, next, apart);
        else if (Q.k <= 32) k_query_persistent<32><<<grid, kQBlock, 0, s>>>(Q, q, next, apart);
        else if (Q.k <= 64) k_query_persistent<64><<<grid, kQBlock, 0, s>>>(Q, q, next, apart);
        else k_query_persistent<0><<<grid, kQBlock, 0, s>>>(Q, q, next, false);
        SKIM_LAUNCH_CHECK();
    }
    if (apart) {
        k_ck_large<<<grid, kQBlock, 0, s>>>(Q, q);
        SKIM_LAUNCH_CHECK();
    }
}

static void query_batch(const uint64_t *ranks, const uint32_t *size, uint32_t n, uint32_t k,
                        uint32_t ell, uint64_t q, const uint64_t *qoff, const uint32_t *qnodes,
                        uint32_t estimator, uint32_t mode, double *est, int32_t *qstatus,
                        hipStream_t s, bool permutation = false) {
    SKIM_REQUIRE(ranks && size, "sketches are NULL");
    SKIM_REQUIRE(n >= 1 && k >= 2 && k <= 256 && ell >= 1 && ell <= 64,
                 "need n >= 1, 2 <= k <= 256, 1 <= l <= 64");
    SKIM_REQUIRE(estimator <= 1, "estimator must be 0 (bottom-k) or 1 (Cohen-Kaplan)");
    SKIM_REQUIRE(mode <= 1, "mode must be 0 (batched) or 1 (one launch per query)");
    if (q == 0) return;
    SKIM_REQUIRE(qoff && est, "qoff/est is NULL");
    Arena A(s);
    uint32_t *err = A.alloc<uint32_t>(1);
    fill_u32(err, 0, 1, s);
    k_check_offsets<<<grid_for(q + 1, 256, 4096), 256, 0, s>>>(qoff, q, err);
    SKIM_LAUNCH_CHECK();
    uint32_t herr = 0;
    read_back(&herr, err, sizeof herr, s);
    SKIM_REQUIRE(!(herr & kBadOffsets), "qoff must start at 0 and be non-decreasing");
    uint64_t total = 0;
    read_back(&total, qoff + q, sizeof total, s);
    SKIM_REQUIRE(total == 0 || qnodes, "qnodes is NULL");
    QArgs Q{ranks, size, n, k, ell, q, qoff, qnodes, est, qstatus, estimator};
    if (permutation) Q.perm_d = (uint64_t)n * ell;
    Q.large = herr & kLargeSets;
    if (mode == 0) {
        unsigned long long *next = A.alloc<unsigned long long>(1);
        Q.members = total;
        LaunchTimer t("k_query_persistent", s);
        launch_queries_async(Q, q, next, s);
    } else {
        for (uint64_t j = 0; j < q; ++j) {
            launch_each(Q, j, 1, false, s);
        }
    }
    SKIM_HIP(hipStreamSynchronize(s));
    timing_resolve();
}

}  // namespace skim

extern "C" skim_status skim_query_batch(const uint64_t *ranks, const uint32_t *size, uint32_t n,
                                        uint32_t k, uint32_t ell, uint64_t q, const uint64_t *qoff,
                                        const uint32_t *qnodes, uint32_t estimator, uint32_t mode,
                                        double *est, int32_t *qstatus, void *stream) {
    skim::clear_error();
    try {
        skim::query_batch(ranks, size, n, k, ell, q, qoff, qnodes, estimator, mode, est, qstatus,
                          (hipStream_t)stream);
        return SKIM_OK;
    } catch (const skim::Fail &f) {
        return f.st;
    }
}

extern "C" skim_status skim_perm_query_batch(const uint64_t *ranks, const uint32_t *size,
                                             uint32_t n, uint32_t k, uint32_t ell, uint64_t q,
                                             const uint64_t *qoff, const uint32_t *qnodes,
                                             uint32_t estimator, double *est, int32_t *qstatus,
                                             void *stream) {
    skim::clear_error();
    try {
        skim::query_batch(ranks, size, n, k, ell, q, qoff, qnodes, estimator, 0, est, qstatus,
                          (hipStream_t)stream, true);
        return SKIM_OK;
    } catch (const skim::Fail &f) {
        return f.st;
    }
}

// ------------------------------------------------------------ query plans
// A plan is the batched launch (counter reset by a fill kernel, then the
// persistent query kernel) captured once into a HIP graph; launching the plan
// replays the graph on the caller's stream.
struct skim_query_plan {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    unsigned long long *next = nullptr;
    uint64_t q = 0;
    int device = 0;
};

namespace skim {

static void plan_free(skim_query_plan *p) {
    if (!p) return;
    int cur = 0;
    const bool have = hipGetDevice(&cur) == hipSuccess;
    if (have) (void)hipSetDevice(p->device);
    if (p->exec) (void)hipGraphExecDestroy(p->exec);
    if (p->graph) (void)hipGraphDestroy(p->graph);
    if (p->next) (void)hipFree(p->next);
    if (have) (void)hipSetDevice(cur);
    (void)hipGetLastError();
    delete p;
}

static skim_query_plan *plan_create(const uint64_t *ranks, const uint32_t *size, uint32_t n,
                                    uint32_t k, uint32_t ell, uint64_t q, const uint64_t *qoff,
                                    const uint32_t *qnodes, uint32_t estimator, double *est,
                                    int32_t *qstatus, hipStream_t s) {
    SKIM_REQUIRE(ranks && size, "sketches are NULL");
    SKIM_REQUIRE(n >= 1 && k >= 2 && k <= 256 && ell >= 1 && ell <= 64,
                 "need n >= 1, 2 <= k <= 256, 1 <= l <= 64");
    SKIM_REQUIRE(estimator <= 1, "estimator must be 0 (bottom-k) or 1 (Cohen-Kaplan)");
    SKIM_REQUIRE(q >= 1, "a plan needs q >= 1 sets");
    SKIM_REQUIRE(qoff && est, "qoff/est is NULL");
    {   // the offsets as they are now
        Arena A(s);
        uint32_t *err = A.alloc<uint32_t>(1);
        fill_u32(err, 0, 1, s);
        k_check_offsets<<<grid_for(q + 1, 256, 4096), 256, 0, s>>>(qoff, q, err);
        SKIM_LAUNCH_CHECK();
        uint32_t herr = 0;
        read_back(&herr, err, sizeof herr, s);
        SKIM_REQUIRE(!(herr & kBadOffsets), "qoff must start at 0 and be non-decreasing");
        uint64_t total = 0;
        read_back(&total, qoff + q, sizeof total, s);
        SKIM_REQUIRE(total == 0 || qnodes, "qnodes is NULL");
    }
    std::unique_ptr<skim_query_plan, void (*)(skim_query_plan *)> p(new skim_query_plan,
                                                                   plan_free);
    SKIM_HIP(hipGetDevice(&p->device));
    p->q = q;
    SKIM_HIP(hipMalloc(&p->next, sizeof(unsigned long long)));
    hipStream_t cs = nullptr;
    SKIM_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
    QArgs Q{ranks, size, n, k, ell, q, qoff, qnodes, est, qstatus, estimator};
    hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
        try {
            launch_queries_async(Q, q, p->next, cs);
        } catch (const Fail &) {
            hipGraph_t g = nullptr;
            (void)hipStreamEndCapture(cs, &g);
            if (g) (void)hipGraphDestroy(g);
            (void)hipStreamDestroy(cs);
            throw;
        }
        e = hipStreamEndCapture(cs, &p->graph);
    }
    (void)hipStreamDestroy(cs);
    SKIM_HIP(e);
    SKIM_HIP(hipGraphInstantiate(&p->exec, p->graph, nullptr, nullptr, 0));
    return p.release();
}

}  // namespace skim

extern "C" skim_status skim_query_plan_create(const uint64_t *ranks, const uint32_t *size,
                                              uint32_t n, uint32_t k, uint32_t ell, uint64_t q,
                                              const uint64_t *qoff, const uint32_t *qnodes,
                                              uint32_t estimator, double *est, int32_t *qstatus,
                                              void *stream, skim_query_plan **plan) {
    skim::clear_error();
    if (!plan) {
        skim::set_error("plan is NULL");
        return SKIM_EINVAL;
    }
    *plan = nullptr;
    try {
        *plan = skim::plan_create(ranks, size, n, k, ell, q, qoff, qnodes, estimator, est, qstatus,
                                  (hipStream_t)stream);
        return SKIM_OK;
    } catch (const skim::Fail &f) {
        return f.st;
    }
}

extern "C" skim_status skim_query_plan_launch(skim_query_plan *plan, void *stream) {
    skim::clear_error();
    if (!plan) {
        skim::set_error("plan is NULL");
        return SKIM_EINVAL;
    }
    try {
        skim::LaunchTimer t("k_query_persistent", (hipStream_t)stream);
        SKIM_HIP(hipGraphLaunch(plan->exec, (hipStream_t)stream));
        return SKIM_OK;
    } catch (const skim::Fail &f) {
        return f.st;
    }
}

extern "C" void skim_query_plan_free(skim_query_plan *plan) { skim::plan_free(plan); }

// -------------------------------------------------------- resident sketches
// A library-owned copy of a sketch table (ranks, sizes, per-node estimates)
// answering union queries by launches that are only enqueued: no host check of the
// offsets (the query kernel checks every set on the device, status -3) and
// no wait, so the call can be captured into a HIP graph.  The persistent
// kernel's work counter is reset by a fill kernel on the stream (no memset
// node) and comes from a ring of per-handle counters, or from a workspace the
// caller passes.
struct skim_sketches {
    int device = 0;
    uint32_t n = 0, k = 0, ell = 0;
    uint64_t *ranks = nullptr;
    uint32_t *size = nullptr;
    double *est = nullptr;
    unsigned long long *counters = nullptr;  // kRing counters, one 128-byte line each
    std::atomic<uint32_t> turn{0};
};

namespace skim {

constexpr uint32_t kRing = 64;

static void sketches_free(skim_sketches *h) {
    if (!h) return;
    int cur = 0;
    const bool have = hipGetDevice(&cur) == hipSuccess;
    if (have) (void)hipSetDevice(h->device);
    (void)hipDeviceSynchronize();  // no queued work may still use the buffers
    (void)hipFree(h->ranks);
    (void)hipFree(h->size);
    (void)hipFree(h->est);
    (void)hipFree(h->counters);
    if (have) (void)hipSetDevice(cur);
    (void)hipGetLastError();
    delete h;
}

static skim_sketches *sketches_alloc(uint32_t n, uint32_t k, uint32_t ell) {
    SKIM_REQUIRE(n >= 1 && k >= 2 && k <= 256 && ell >= 1 && ell <= 64,
                 "need n >= 1, 2 <= k <= 256, 1 <= l <= 64");
    if (alloc_fault()) {
        set_error("device allocation for resident sketches failed: injected failure");
        throw Fail{SKIM_ENOMEM};
    }
    std::unique_ptr<skim_sketches, void (*)(skim_sketches *)> h(new skim_sketches,
                                                                sketches_free);
    SKIM_HIP(hipGetDevice(&h->device));
    h->n = n;
    h->k = k;
    h->ell = ell;
    SKIM_HIP(hipMalloc(&h->ranks, (size_t)n * k * sizeof(uint64_t)));
    SKIM_HIP(hipMalloc(&h->size, (size_t)n * sizeof(uint32_t)));
    SKIM_HIP(hipMalloc(&h->est, (size_t)n * sizeof(double)));
    SKIM_HIP(hipMalloc(&h->counters, (size_t)kRing * 128));
    return h.release();
}

}  // namespace skim

extern "C" skim_status skim_sketches_create(const uint64_t *ranks, const uint32_t *size,
                                            uint32_t n, uint32_t k, uint32_t ell, void *stream,
                                            skim_sketches **out) {
    skim::clear_error();
    if (!out) {
        skim::set_error("out is NULL");
        return SKIM_EINVAL;
    }
    *out = nullptr;
    try {
        SKIM_REQUIRE(ranks && size, "sketches are NULL");
        skim_sketches *h = skim::sketches_alloc(n, k, ell);
        hipStream_t s = (hipStream_t)stream;
        try {
            SKIM_HIP(hipMemcpyAsync(h->ranks, ranks, (size_t)n * k * 8, hipMemcpyDeviceToDevice, s));
            SKIM_HIP(hipMemcpyAsync(h->size, size, (size_t)n * 4, hipMemcpyDeviceToDevice, s));
            skim::launch_estimates(h->ranks, h->size, n, k, ell, h->est, s);
        } catch (const skim::Fail &) {
            skim::sketches_free(h);
            throw;
        }
        *out = h;
        return SKIM_OK;
    } catch (const skim::Fail &f) {
        return f.st;
    }
}

extern "C" skim_status skim_build_sketches_resident(const skim_graph *g, uint32_t ell, uint32_t k,
                                                    uint64_t seed, uint64_t *work, void *stream,
                                                    skim_sketches **out) {
    skim::clear_error();
    if (!out || !g) {
        skim::set_error("NULL argument");
        return SKIM_EINVAL;
    }
    *out = nullptr;
    skim_sketches *h = nullptr;
    try {
        h = skim::sketches_alloc(g->n, k, ell);
    } catch (const skim::Fail &f) {
        return f.st;
    }
    const skim_status st =
        skim_build_sketches(g, ell, k, seed, h->ranks, h->size, h->est, work, stream);
    if (st != SKIM_OK) {
        skim::sketches_free(h);
        return st;
    }
    *out = h;
    return SKIM_OK;
}

extern "C" skim_status skim_sketches_data(const skim_sketches *h, const uint64_t **ranks,
                                          const uint32_t **size, const double **est, uint32_t *n,
                                          uint32_t *k, uint32_t *ell) {
    skim::clear_error();
    if (!h) {
        skim::set_error("handle is NULL");
        return SKIM_EINVAL;
    }
    if (ranks) *ranks = h->ranks;
    if (size) *size = h->size;
    if (est) *est = h->est;
    if (n) *n = h->n;
    if (k) *k = h->k;
    if (ell) *ell = h->ell;
    return SKIM_OK;
}

extern "C" skim_status skim_sketches_query(const skim_sketches *hc, uint64_t q, const uint64_t *qoff,
                                           const uint32_t *qnodes, uint64_t nnodes,
                                           uint32_t estimator, double *est, int32_t *qstatus,
                                           void *workspace, void *stream) {
    skim::clear_error();
    skim_sketches *h = const_cast<skim_sketches *>(hc);
    if (!h) {
        skim::set_error("handle is NULL");
        return SKIM_EINVAL;
    }
    try {
        SKIM_REQUIRE(estimator <= 1, "estimator must be 0 (bottom-k) or 1 (Cohen-Kaplan)");
        if (q == 0) return SKIM_OK;
        SKIM_REQUIRE(qoff && est, "qoff/est is NULL");
        SKIM_REQUIRE(nnodes == 0 || qnodes, "qnodes is NULL");
        skim::QueryArgs Q{h->ranks, h->size, h->n, h->k, h->ell, q, qoff, qnodes, est, qstatus,
                          estimator, nnodes};
        unsigned long long *next =
            workspace ? (unsigned long long *)workspace
                      : h->counters + 16 * (h->turn.fetch_add(1) % skim::kRing);
        skim::launch_queries_async(Q, q, next, (hipStream_t)stream);
        return SKIM_OK;
    } catch (const skim::Fail &f) {
        return f.st;
    }
}

extern "C" void skim_sketches_free(skim_sketches *h) { skim::sketches_free(h); }
