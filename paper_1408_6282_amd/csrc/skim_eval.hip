// skim_eval.hip -- exact influence of seed sets over l live-edge instances
// (Section 2, eqs. (Inf) and (timedinf): l Inf({G^(i)}, S) = sum_i |reach_i(S)|).
//
// This is the evaluator of a quality harness: it scores seed sets (SKIM's,
// or any other) on the instances of a given seed, typically fresh ones that
// the sketches never saw.
//
// One coin pass builds the live out-lists, so the searches never evaluate a
// coin.  A batch (skim_influence_batch) is cut into units of one instance and
// 32 queries, each searched by one workgroup for its 32 queries at once
// (k_eval_sets, see there); the lists are laid out instance by instance, so
// the units of an instance read the same few hundred kilobytes.
//
// Exact greedy (skim_greedy_exact, the reference of a quality harness) scores
// one node per workgroup (k_eval): a breadth-first search over all instances'
// pairs with a visited bitmap of 64 bits per node and an append-only queue of
// pair ids (every pair enters at most once, so the queue never overflows),
// consumed in chunks of one pair per thread.  The workgroup then clears the
// words its pairs set.  The search skips the pairs the seeds so far reach, a
// bitmap of covered pairs.  That set is closed under reachability, so a search
// that skips covered pairs counts exactly a node's marginal gain.  Each step
// scores every node this way (n singleton queries), takes the largest gain on
// the device (smallest id on ties, among unselected nodes), searches once more
// from the winner and adds the pairs it reached to the covered bitmap.
#include "skim_internal.h"

#include <algorithm>
#include <atomic>
#include <type_traits>

namespace skim {

namespace {

constexpr int kEvalBlock = 1024;
constexpr uint64_t kEvalSlotBudget = 2ull << 30;  // bytes of bitmaps + queues
constexpr uint32_t kEvalMaxSlots = 1024;

struct EvalArgs {
    uint32_t n, ell;
    const uint64_t *fptr;  // [64 n + 1] live out-lists per pair
    const uint32_t *fadj;
    uint64_t q;
    const uint64_t *qoff;
    const uint32_t *qnodes;
    uint64_t *reach;       // [q] out
    uint32_t *bitmaps;     // [slots][2 n]
    uint32_t *queues;      // [slots][qcap]
    uint64_t qcap;         // l n
    const uint32_t *covered;  // [2 n] pairs not to enter
};

template <class T> __device__ __forceinline__ T ld(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T> __device__ __forceinline__ void st(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// err = 1 unless qoff[0] = 0 and qoff is non-decreasing.
__global__ void k_eval_offsets(const uint64_t *qoff, uint64_t q, uint32_t *err) {
    for (uint64_t j = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; j <= q;
         j += (uint64_t)gridDim.x * blockDim.x) {
        const bool bad = j == 0 ? qoff[0] != 0 : qoff[j - 1] > qoff[j];
        if (bad) atomicOr(err, 1u);
    }
}

// Marks pair p visited; true if this call set its bit.
__device__ __forceinline__ bool mark(uint32_t *bm, uint64_t p) {
    const uint32_t bit = 1u << (p & 31);
    return (atomicOr(bm + (p >> 5), bit) & bit) == 0;
}

__device__ __forceinline__ bool is_covered(const uint32_t *cov, uint64_t p) {
    return ((cov[p >> 5] >> (p & 31)) & 1u) != 0;
}

__global__ void __launch_bounds__(kEvalBlock) k_eval(EvalArgs A) {
    __shared__ unsigned long long s_tail;
    const uint32_t tid = threadIdx.x;
    uint32_t *bm = A.bitmaps + (uint64_t)blockIdx.x * 2 * A.n;
    uint32_t *Q = A.queues + (uint64_t)blockIdx.x * A.qcap;
    for (uint64_t j = blockIdx.x; j < A.q; j += gridDim.x) {
        const uint64_t b = A.qoff[j], e = A.qoff[j + 1];
        if (tid == 0) s_tail = 0;
        __syncthreads();
        // seeds: every (s, i) with s in S, i < l (duplicates in S act once)
        const uint64_t seeds = (e - b) * A.ell;
        for (uint64_t t0 = 0; t0 < seeds; t0 += kEvalBlock) {
            const uint64_t t = t0 + tid;
            bool add = false;
            uint64_t p = 0;
            if (t < seeds) {
                p = (uint64_t)A.qnodes[b + t / A.ell] * kPairStride + t % A.ell;
                add = !is_covered(A.covered, p) && mark(bm, p);
            }
            const uint64_t slot = wave_reserve(&s_tail, add);
            if (add) st(Q + slot, (uint32_t)p);
        }
        __syncthreads();
        // breadth-first over pairs; the queue only grows
        uint64_t head = 0;
        for (;;) {
            const uint64_t tail = s_tail;
            __syncthreads();  // every thread has the same tail before any append
            if (head >= tail) break;
            const uint64_t chunk = tail - head < (uint64_t)kEvalBlock ? tail - head : kEvalBlock;
            if (tid < chunk) {
                const uint32_t p = ld(Q + head + tid);
                const uint32_t i = p % kPairStride;
                const uint64_t e0 = A.fptr[p], e1 = A.fptr[p + 1];
                for (uint64_t x = e0; x < e1; ++x) {
                    const uint64_t pw = (uint64_t)A.fadj[x] * kPairStride + i;
                    const bool add = !is_covered(A.covered, pw) && mark(bm, pw);
                    const unsigned long long mask = __ballot(add);
                    if (mask) {
                        const int leader = __ffsll((long long)mask) - 1;
                        unsigned long long base = 0;
                        if ((int)lane_id() == leader)
                            base = atomicAdd(&s_tail, (unsigned long long)__popcll(mask));
                        base = ((unsigned long long)__shfl((uint32_t)(base >> 32), leader) << 32) |
                               __shfl((uint32_t)base, leader);
                        if (add)
                            st(Q + base + __popcll(mask & ((1ull << lane_id()) - 1ull)),
                               (uint32_t)pw);
                    }
                }
            }
            head += chunk;
            __syncthreads();  // appends of this chunk are in the queue and s_tail
        }
        const uint64_t total = s_tail;
        if (tid == 0) A.reach[j] = total;
        // clean the bitmap words this query set
        for (uint64_t t = tid; t < total; t += kEvalBlock) st(bm + (ld(Q + t) >> 5), 0u);
        __syncthreads();
    }
}

// --------------------------------------------- batches: 32 queries at once
// A unit is one instance i and one word of up to 32 queries.  Its workgroup keeps a
// 32-bit mask per node, the queries of the word that reach the node, and a
// queue of the nodes whose mask grew since they were last expanded (a node is
// in the queue at most once: its `dirty` bit).  Expanding v sends its mask
// along its live out-edges; a head whose mask grows is queued again.  Queries
// whose searches meet in a node (the prefixes of one seed sequence, any sets
// that reach the same component) go on as one from there, where a search per
// query walks the shared part once for each.
//
// What bounds it: LDS atomics and dependent list reads, with a workgroup per
// unit.  Masks, dirty bits and a ring of 16-bit node ids take 6.125 n bytes of
// LDS, which fits up to kSetsLdsNodes nodes; above that they are in global
// memory (device atomics, 32-bit ids, slots within kEvalSlotBudget).  The 200
// prefixes of a seed sequence on a 20,000-node weighted-cascade graph
// (l = 64): one workgroup per query over all pairs 34.9 ms a call, this 0.52 ms,
// most of it the lists.
constexpr uint32_t kSetsLdsNodes = 26000;   // 6.125 n + 2 KiB of LDS
constexpr uint32_t kSetsSmallNodes = 4096;  // up to here 256 threads: several units per CU
constexpr size_t sets_lds(uint64_t n, uint64_t threads) {
    return 4 * n + 4 * ((n + 31) / 32) + 2 * (n + threads);
}

struct SetsArgs {
    uint32_t n, ell;
    const uint64_t *fptr;  // [l n + 1] live out-lists, instance-major
    const uint32_t *fadj;
    uint64_t q, words;     // queries, words of `width` of them
    uint32_t width;        // queries of a word (<= 32)
    uint32_t shift;        // instances side by side: 8, or with fewer instances 4, 2 or 1
    const uint64_t *qoff;
    const uint32_t *qnodes;
    const uint8_t *bad;    // [q] the query names a node >= n
    uint64_t *reach;       // [q] added to
    uint32_t *masks;       // [slots][n], zero between units (global state)
    uint32_t *dirty;       // [slots][(n + 31) / 32], zero between units
    uint32_t *ring;        // [slots][n + NT]
};

__host__ __device__ inline uint64_t sets_units(uint32_t ell, uint32_t shift, uint64_t words) {
    return ((((uint64_t)ell - 1) >> shift) + 1) * words << shift;
}

// Queries of a word: as few as make no more than kSetsUnits units, where queries
// that meet are walked more than once but side by side; 32 when there are more units
// anyway.  100 pairs of nodes on a giant component (20,000 nodes, l = 1), a call:
// words of 32 0.49 ms, so 0.19; with 256 units the 30 sets of an R-MAT graph of 2^17
// nodes, l = 64, took 1.7 ms for 1.35 (device atomics).
constexpr uint64_t kSetsUnits = 64;
inline uint32_t sets_width(uint32_t ell, uint64_t q) {
    uint32_t w = 32;
    while (w > 1 && ell * ((q + w / 2 - 1) / (w / 2)) <= kSetsUnits) w /= 2;
    return w;
}

// Per query: the status and a zero count (one wave each).
__global__ void __launch_bounds__(256) k_sets_begin(uint32_t n, uint64_t q, const uint64_t *qoff,
                                                    const uint32_t *qnodes, uint8_t *bad,
                                                    uint64_t *reach, int32_t *status) {
    const uint32_t lane = lane_id();
    const uint64_t waves = (uint64_t)gridDim.x * (blockDim.x / 64);
    for (uint64_t j = blockIdx.x * (uint64_t)(blockDim.x / 64) + threadIdx.x / 64; j < q;
         j += waves) {
        bool b = false;
        for (uint64_t t = qoff[j] + lane; t < qoff[j + 1]; t += 64) b |= qnodes[t] >= n;
        const bool any = __ballot(b) != 0;
        if (lane == 0) {
            bad[j] = any;
            reach[j] = 0;
            if (status) status[j] = any ? -1 : 0;
        }
    }
}

// State words: LDS at workgroup scope, global memory at agent scope (as the
// rest of this file, so no stale line of the L1 is read).
template <bool kLds> struct SetWord {
    static constexpr int kScope = kLds ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT;
    static __device__ __forceinline__ uint32_t get(const uint32_t *p) {
        return __hip_atomic_load(p, __ATOMIC_RELAXED, kScope);
    }
    static __device__ __forceinline__ uint32_t set_bits(uint32_t *p, uint32_t v) {
        return __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, kScope);
    }
    static __device__ __forceinline__ uint32_t keep_bits(uint32_t *p, uint32_t v) {
        return __hip_atomic_fetch_and(p, v, __ATOMIC_RELAXED, kScope);
    }
    static __device__ __forceinline__ uint32_t take(uint32_t *p) {
        return __hip_atomic_exchange(p, 0u, __ATOMIC_RELAXED, kScope);
    }
};

// What came before (in program order) has reached the state words before
// anything after is issued.
__device__ __forceinline__ void sets_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
}

// Adds the wave's counts of the 32 mask bits to out[0..32): c[j] holds the
// bytes of bits j, j + 8, j + 16, j + 24 (at most 255 masks per lane).
__device__ __forceinline__ void sets_flush(uint32_t (&c)[8], uint32_t *out) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        uint32_t lo = c[j] & 0x00FF00FFu, hi = (c[j] >> 8) & 0x00FF00FFu;  // sums < 2^14
        for (int off = 32; off > 0; off >>= 1) {
            lo += __shfl_xor(lo, off);
            hi += __shfl_xor(hi, off);
        }
        if (lane_id() == 0) {
            if (lo & 0xFFFFu) atomicAdd(out + j, lo & 0xFFFFu);
            if (hi & 0xFFFFu) atomicAdd(out + j + 8, hi & 0xFFFFu);
            if (lo >> 16) atomicAdd(out + j + 16, lo >> 16);
            if (hi >> 16) atomicAdd(out + j + 24, hi >> 16);
        }
        c[j] = 0;
    }
}

template <bool kLds, int NT>
__global__ void __launch_bounds__(NT) k_eval_sets(SetsArgs A) {
    using W = SetWord<kLds>;
    using Id = typename std::conditional<kLds, uint16_t, uint32_t>::type;
    extern __shared__ uint32_t s_mem[];
    __shared__ uint64_t s_off[33];
    __shared__ uint32_t s_cnt[32];
    __shared__ uint32_t s_tail, s_bad;
    const uint32_t tid = threadIdx.x, lane = lane_id(), n = A.n;
    const uint32_t dwords = (n + 31) / 32, cap = n + NT;
    uint32_t *M = kLds ? s_mem : A.masks + (uint64_t)blockIdx.x * n;
    uint32_t *D = kLds ? s_mem + n : A.dirty + (uint64_t)blockIdx.x * dwords;
    Id *R = kLds ? (Id *)(s_mem + n + dwords) : (Id *)(A.ring + (uint64_t)blockIdx.x * cap);
    if (kLds)
        for (uint32_t v = tid; v < n + dwords; v += NT) s_mem[v] = 0;
    // Workgroups go to the 8 XCDs in turn: with 8 instances or more every unit of
    // instance i runs on XCD i mod 8, whose L2 then holds that instance's lists;
    // with fewer an instance's units go to all XCDs.
    const uint64_t units = sets_units(A.ell, A.shift, A.words);
    for (uint64_t u = blockIdx.x; u < units; u += gridDim.x) {
        const uint64_t r = u >> A.shift;
        const uint32_t inst = (uint32_t)((u & ((1u << A.shift) - 1u)) + ((r / A.words) << A.shift));
        if (inst >= A.ell) continue;  // uniform
        const uint64_t j0 = A.width * (r % A.words);
        const uint32_t nq = A.q - j0 < A.width ? (uint32_t)(A.q - j0) : A.width;
        const uint64_t *ptr = A.fptr + (uint64_t)inst * n;
        __syncthreads();  // the previous unit is done (and the first one's state is clear)
        if (tid <= 32) s_off[tid] = A.qoff[j0 + (tid < nq ? tid : nq)];
        if (tid < 32) s_cnt[tid] = 0;
        if (tid == 0) {
            s_tail = 0;
            s_bad = 0;
        }
        __syncthreads();
        if (tid < nq && A.bad[j0 + tid]) atomicOr(&s_bad, 1u << tid);
        __syncthreads();
        // new bits m for node w; true if w has to be queued (called by lanes
        // with something to send; the queueing itself is wave-wide)
        auto send = [&](uint32_t w, uint32_t m) {
            if ((m & ~W::get(M + w)) == 0) return false;
            if ((m & ~W::set_bits(M + w, m)) == 0) return false;
            sets_order();  // the mask before the dirty bit
            const uint32_t bit = 1u << (w & 31);
            return (W::set_bits(D + (w >> 5), bit) & bit) == 0;
        };
        auto queue = [&](bool add, uint32_t w) {
            const unsigned long long b = __ballot(add);
            if (!b) return;
            const int leader = __ffsll((long long)b) - 1;
            uint32_t base = 0;
            if ((int)lane == leader) base = atomicAdd(&s_tail, (uint32_t)__popcll(b));
            base = (uint32_t)__shfl((int)base, leader);
            if (add) {
                Id *slot = R + (base + (uint32_t)__popcll(b & ((1ull << lane) - 1ull))) % cap;
                if (kLds) *slot = (Id)w;
                else st((uint32_t *)slot, w);
            }
        };
        // the members of the word's sets
        const uint64_t b0 = s_off[0], b1 = s_off[32];
        for (uint64_t t0 = b0; t0 < b1; t0 += NT) {
            const uint64_t t = t0 + tid;
            bool add = false;
            uint32_t w = 0;
            if (t < b1) {
                uint32_t lo = 0, hi = 32;  // s_off[lo] <= t < s_off[hi]
                while (hi - lo > 1) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (s_off[mid] <= t) lo = mid;
                    else hi = mid;
                }
                if (!((s_bad >> lo) & 1u)) {
                    w = A.qnodes[t];
                    add = send(w, 1u << lo);
                }
            }
            queue(add, w);
        }
        __syncthreads();
        for (uint32_t head = 0;;) {
            const uint32_t tail = s_tail;
            __syncthreads();  // every thread has the same tail before any append
            if (head == tail) break;
            const uint32_t cnt = tail - head < (uint32_t)NT ? tail - head : (uint32_t)NT;
            if ((tid & ~63u) < cnt) {  // waves with an entry
                uint32_t m = 0, d = 0;
                uint64_t e0 = 0;
                if (tid < cnt) {
                    const Id *slot = R + (head + tid) % cap;
                    const uint32_t v = kLds ? (uint32_t)*slot : ld((const uint32_t *)slot);
                    e0 = ptr[v];
                    d = (uint32_t)(ptr[v + 1] - e0);
                    W::keep_bits(D + (v >> 5), ~(1u << (v & 31)));
                    sets_order();  // the dirty bit is off before the mask is read
                    m = W::get(M + v);
                }
                // the wave's out-edges laid end to end, 64 at a time
                uint32_t incl = d;
#pragma unroll
                for (uint32_t off = 1; off < 64; off <<= 1) {
                    const uint32_t y = __shfl_up(incl, off);
                    if (lane >= off) incl += y;
                }
                const uint32_t tot = (uint32_t)__shfl((int)incl, 63);
                for (uint32_t base = 0; base < tot; base += 64) {
                    const uint32_t j = base + lane;
                    uint32_t r = 0;
#pragma unroll
                    for (uint32_t step = 32; step > 0; step >>= 1) {
                        const uint32_t y = (uint32_t)__shfl((int)incl, (int)(r + step - 1));
                        if (y <= j) r += step;
                    }
                    r &= 63u;
                    const uint32_t first =
                        (uint32_t)__shfl((int)incl, (int)r) - (uint32_t)__shfl((int)d, (int)r);
                    const uint64_t re0 =
                        ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(e0 >> 32), (int)r) << 32) |
                        (uint32_t)__shfl((int)(uint32_t)e0, (int)r);
                    const uint32_t rm = (uint32_t)__shfl((int)m, (int)r);
                    bool add = false;
                    uint32_t w = 0;
                    if (j < tot) {
                        w = A.fadj[re0 + (j - first)];
                        add = send(w, rm);
                    }
                    queue(add, w);
                }
            }
            head += cnt;
            __syncthreads();  // this round's entries are in the ring and s_tail
        }
        // count the masks' bits and clear them: over the ring when it still
        // holds every entry (a repeated node counts once: its mask is taken),
        // else over all nodes
        {
            const uint32_t tail = s_tail;
            const bool sparse = tail <= cap && tail < n;
            const uint32_t items = sparse ? tail : n;
            uint32_t c[8] = {0, 0, 0, 0, 0, 0, 0, 0}, held = 0;
            for (uint32_t t0 = 0; t0 < items; t0 += NT) {  // uniform
                if (t0 + tid < items) {
                    uint32_t v = t0 + tid;
                    if (sparse) v = kLds ? (uint32_t)R[v] : ld((const uint32_t *)R + v);
                    const uint32_t m = W::take(M + v);
#pragma unroll
                    for (int j = 0; j < 8; ++j) c[j] += (m >> j) & 0x01010101u;
                }
                if (++held == 255) {
                    sets_flush(c, s_cnt);
                    held = 0;
                }
            }
            if (held) sets_flush(c, s_cnt);
        }
        __syncthreads();
        if (tid < nq && s_cnt[tid])
            atomicAdd((unsigned long long *)A.reach + j0 + tid, (unsigned long long)s_cnt[tid]);
    }
}

// The next exact-greedy seed: the largest gain among unselected nodes,
// smallest id on ties (one workgroup).
__global__ void __launch_bounds__(kEvalBlock) k_exact_pick(uint32_t n, const uint64_t *gain,
                                                           uint32_t *sel, uint32_t *x_out,
                                                           uint32_t *seed_out) {
    __shared__ unsigned long long best;
    if (threadIdx.x == 0) best = 0;
    __syncthreads();
    unsigned long long mine = 0;
    for (uint32_t v = threadIdx.x; v < n; v += kEvalBlock)
        if (!sel[v]) {
            // gains are at most 64 n < 2^32
            const unsigned long long key = (gain[v] << 32) | (0xFFFFFFFFu - v);
            mine = key > mine ? key : mine;
        }
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)mine, off);
        const uint32_t hi = __shfl_xor((uint32_t)(mine >> 32), off);
        const unsigned long long o = ((unsigned long long)hi << 32) | lo;
        mine = o > mine ? o : mine;
    }
    if ((threadIdx.x & 63) == 0) atomicMax(&best, mine);
    __syncthreads();
    if (threadIdx.x == 0) {
        // an unselected node always exists (the host checks s)
        const uint32_t v = 0xFFFFFFFFu - (uint32_t)best;
        const uint32_t x = (best != 0 && v < n) ? v : 0;
        sel[x] = 1;
        *x_out = x;
        *seed_out = x;
    }
}

// Adds the pairs of one finished search (its queue) to the covered bitmap.
__global__ void k_exact_cover(const uint32_t *Q, const uint64_t *count, uint32_t *covered) {
    const uint64_t c = *count;
    for (uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; t < c;
         t += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t p = Q[t];
        atomicOr(covered + (p >> 5), 1u << (p & 31));
    }
}

__global__ void k_iota(uint32_t n, uint64_t *off, uint32_t *nodes) {
    for (uint32_t v = blockIdx.x * blockDim.x + threadIdx.x; v <= n; v += gridDim.x * blockDim.x) {
        off[v] = v;
        if (v < n) nodes[v] = v;
    }
}

}  // namespace

}  // namespace skim

extern "C" skim_status skim_greedy_exact(const skim_graph *g, uint32_t ell, uint64_t seed,
                                         uint32_t s, uint32_t *seeds, uint64_t *gain_pairs,
                                         void *stream) {
    using namespace skim;
    clear_error();
    hipStream_t hs = (hipStream_t)stream;
    try {
        SKIM_REQUIRE(g != nullptr, "graph is NULL");
        SKIM_REQUIRE(ell >= 1 && ell <= 64, "l must be in [1, 64]");
        SKIM_REQUIRE(s <= g->n, "s exceeds n");
        SKIM_REQUIRE(s == 0 || (seeds && gain_pairs), "seeds/gain_pairs is NULL");
        Arena T(hs);
        uint32_t *esrc = T.alloc<uint32_t>(g->m ? g->m : 1);
        validate_graph(g, esrc, T);
        if (s == 0) return SKIM_OK;
        const uint32_t n = g->n;
        LiveLists fwd = build_live_lists(g, ell, seed, esrc, /*forward=*/true, T);
        const uint64_t qcap = (uint64_t)ell * n;
        const uint64_t per_slot = (2ull * n + qcap) * sizeof(uint32_t);
        uint64_t slots = std::max<uint64_t>(1, kEvalSlotBudget / per_slot);
        slots = std::min<uint64_t>(std::min<uint64_t>(slots, kEvalMaxSlots), n);
        EvalArgs A{};
        A.n = n;
        A.ell = ell;
        A.fptr = fwd.ptr;
        A.fadj = fwd.adj;
        A.bitmaps = T.alloc<uint32_t>(slots * 2 * n);
        A.queues = T.alloc<uint32_t>(slots * qcap);
        A.qcap = qcap;
        uint32_t *covered = T.alloc<uint32_t>(2ull * n);
        uint32_t *sel = T.alloc<uint32_t>(n);
        uint64_t *gain = T.alloc<uint64_t>(n);
        uint64_t *all_off = T.alloc<uint64_t>((uint64_t)n + 1);
        uint32_t *all_nodes = T.alloc<uint32_t>(n);
        uint64_t *one_off = T.alloc<uint64_t>(2);
        uint32_t *x = T.alloc<uint32_t>(1);
        fill_u32(A.bitmaps, 0, slots * 2 * n, hs);
        fill_u32(covered, 0, 2ull * n, hs);
        fill_u32(sel, 0, n, hs);
        k_iota<<<grid_for((uint64_t)n + 1, 256, 4096), 256, 0, hs>>>(n, all_off, all_nodes);
        SKIM_LAUNCH_CHECK();
        k_iota<<<1, 256, 0, hs>>>(1, one_off, x);  // one_off = {0, 1}
        SKIM_LAUNCH_CHECK();
        A.covered = covered;
        for (uint32_t step = 0; step < s; ++step) {
            // every node's marginal gain: a search that does not enter covered pairs
            A.q = n;
            A.qoff = all_off;
            A.qnodes = all_nodes;
            A.reach = gain;
            k_eval<<<(unsigned)slots, kEvalBlock, 0, hs>>>(A);
            SKIM_LAUNCH_CHECK();
            k_exact_pick<<<1, kEvalBlock, 0, hs>>>(n, gain, sel, x, seeds + step);
            SKIM_LAUNCH_CHECK();
            // the winner's search again, on slot 0, then cover what it reached
            A.q = 1;
            A.qoff = one_off;
            A.qnodes = x;
            A.reach = gain_pairs + step;
            k_eval<<<1, kEvalBlock, 0, hs>>>(A);
            SKIM_LAUNCH_CHECK();
            k_exact_cover<<<grid_for(qcap, 256, 4096), 256, 0, hs>>>(A.queues, gain_pairs + step,
                                                                    covered);
            SKIM_LAUNCH_CHECK();
        }
        SKIM_HIP(hipStreamSynchronize(hs));
        return SKIM_OK;
    } catch (const Fail &f) {
        return f.st;
    }
}

extern "C" skim_status skim_influence_batch(const skim_graph *g, uint32_t ell, uint64_t seed,
                                            uint64_t q, const uint64_t *qoff,
                                            const uint32_t *qnodes, uint64_t *reach_pairs,
                                            int32_t *qstatus, void *stream) {
    using namespace skim;
    clear_error();
    hipStream_t hs = (hipStream_t)stream;
    try {
        SKIM_REQUIRE(g != nullptr, "graph is NULL");
        SKIM_REQUIRE(ell >= 1 && ell <= 64, "l must be in [1, 64]");
        SKIM_REQUIRE(q == 0 || (qoff && reach_pairs), "qoff/reach_pairs is NULL");
        Arena T(hs);
        uint32_t *esrc = T.alloc<uint32_t>(g->m ? g->m : 1);
        validate_graph(g, esrc, T);
        if (q == 0) return SKIM_OK;
        uint32_t *err = T.alloc<uint32_t>(1);
        fill_u32(err, 0, 1, hs);
        k_eval_offsets<<<grid_for(q + 1, 256, 4096), 256, 0, hs>>>(qoff, q, err);
        SKIM_LAUNCH_CHECK();
        uint32_t herr = 0;
        read_back(&herr, err, sizeof herr, hs);
        SKIM_REQUIRE(herr == 0, "qoff must start at 0 and be non-decreasing");
        uint64_t total = 0;
        read_back(&total, qoff + q, sizeof total, hs);
        SKIM_REQUIRE(total == 0 || qnodes, "qnodes is NULL");
        const uint32_t n = g->n;
        const LiveLists fwd = build_live_lists(g, ell, seed, esrc, /*forward=*/true, T, nullptr,
                                               /*instance_major=*/true);
        SetsArgs A{};
        A.n = n;
        A.ell = ell;
        A.fptr = fwd.ptr;
        A.fadj = fwd.adj;
        A.q = q;
        A.width = sets_width(ell, q);
        A.words = (q + A.width - 1) / A.width;
        A.shift = ell >= 8 ? 3 : ell >= 4 ? 2 : ell >= 2 ? 1 : 0;
        A.qoff = qoff;
        A.qnodes = qnodes;  // never read when every set is empty
        A.reach = reach_pairs;
        uint8_t *bad = T.alloc<uint8_t>(q);
        A.bad = bad;
        k_sets_begin<<<grid_for(q, 4, 4096), 256, 0, hs>>>(n, q, qoff, qnodes, bad, reach_pairs,
                                                           qstatus);
        SKIM_LAUNCH_CHECK();
        const uint64_t units = sets_units(ell, A.shift, A.words);
        LaunchTimer t("k_eval_sets", hs);
        if (n <= kSetsLdsNodes) {
            const bool small = n <= kSetsSmallNodes;
            const uint64_t nt = small ? 256 : 1024;
            const size_t lds = sets_lds(n, nt);
            const void *f = small ? (const void *)k_eval_sets<true, 256>
                                  : (const void *)k_eval_sets<true, 1024>;
            // the limit belongs to the kernel, not to this call: always the
            // largest, which no thread with a smaller graph lowers for another
            static std::atomic<uint64_t> have[2];  // by device
            const uint64_t dev_bit = 1ull << T.device();
            if (!(have[small].load() & dev_bit)) {
                SKIM_HIP(hipFuncSetAttribute(
                    f, hipFuncAttributeMaxDynamicSharedMemorySize,
                    (int)sets_lds(small ? kSetsSmallNodes : kSetsLdsNodes, nt)));
                have[small] |= dev_bit;
            }
            const unsigned grid = (unsigned)std::min<uint64_t>(units, 4096);  // multiples of 8
            if (small) k_eval_sets<true, 256><<<grid, 256, lds, hs>>>(A);
            else k_eval_sets<true, 1024><<<grid, 1024, lds, hs>>>(A);
        } else {
            const uint64_t dwords = (n + 31) / 32, cap = (uint64_t)n + 1024;
            const uint64_t per_slot = (n + dwords + cap) * sizeof(uint32_t);
            uint64_t slots = std::max<uint64_t>(8, kEvalSlotBudget / per_slot / 8 * 8);
            slots = std::min<uint64_t>(std::min<uint64_t>(slots, kEvalMaxSlots), units);
            A.masks = T.alloc<uint32_t>(slots * n);
            A.dirty = T.alloc<uint32_t>(slots * dwords);
            A.ring = T.alloc<uint32_t>(slots * cap);
            fill_u32(A.masks, 0, slots * n, hs);
            fill_u32(A.dirty, 0, slots * dwords, hs);
            k_eval_sets<false, 1024><<<(unsigned)slots, 1024, 0, hs>>>(A);
        }
        SKIM_LAUNCH_CHECK();
        SKIM_HIP(hipStreamSynchronize(hs));
        return SKIM_OK;
    } catch (const Fail &f) {
        return f.st;
    }
}
