// skim_ic.hip -- sketches for the IC model itself (Section 3, "Sketches for
// an IC model"), with structured permutation ranks (Section 3, "Structured
// permutation ranks") in the limit of infinitely many instances.
//
// Positions t = 1 .. k n come in k chunks of n; each chunk holds every node
// once, in the order of a SplitMix64 hash (one rocPRIM radix sort of all
// chunks, the chunk leading the key).  Every position has an instance of its
// own, so the sketch of u is the k smallest positions t whose node v_t u reaches
// in instance t, and the influence estimate is n (k - 1) / (T - 1) with T the
// k-th smallest.  Nothing prunes a search here (an instance has one source),
// so:
//  * a wave runs the complete reverse searches of 12 positions together, over
//    the in-edges whose coin in the position's instance is live (coins on the
//    fly from a per-edge SplitMix64 stream), its queue and its visited set in
//    LDS (k_ic_wave); a wave whose searches outgrow them hands its positions on
//    to a wave each, and a search that outgrows that to a workgroup
//    (k_ic_heavy);
//  * a search's nodes are recorded (node, t), but a node that already
//    has k records from earlier chunks needs no more: the chunks go in phases
//    of fourfold length, and each node keeps the phase in which it had k;
//  * the records are radix-sorted; every node holds at least k of them (it
//    reaches itself in every chunk) and keeps its first k.
#include "skim_internal.h"
#include "skim_wave.h"

#include "skim_sort.h"

#include <algorithm>
#include <type_traits>

namespace skim {

namespace {

constexpr uint64_t kIcChunk = 1ull << 63;                  // counters of the chunk hashes
constexpr uint64_t kIcEdge = (1ull << 63) | (1ull << 62);  // counters of the per-edge streams
constexpr int kIcHeavyBlock = 1024;   // one workgroup per handed-over search
constexpr uint64_t kIcHeavyBudget = 2ull << 30;            // bytes of per-workgroup state
constexpr uint64_t kIcRecordCap = 1ull << 28;  // records of the single pass (2 GiB)
// A wave's searches: positions at a time, queue entries (all of them stay until
// the searches end) and visited-set slots.  Measured on the 20,000-node graph
// (k = 64), whole build: 12 positions 2.54 ms, 16 (512 entries) 2.79, 24 (768,
// 2048 slots) 3.14, 8 (320, 512) 2.76.
constexpr uint32_t kIcWave = 12, kIcQueue = 384, kIcSlots = 1024;
constexpr uint32_t kIcStage = 128;    // records staged per wave (256: fewer waves fit, 3.10 ms not 2.79)
constexpr uint32_t kIcAhead = 4;      // rounds of 64 in-edges loaded at once
constexpr uint32_t kIcOne = 1024;     // queue entries of a wave with one position
constexpr uint32_t kIcNodeBits = 26;  // node ids (64 n < 2^32)
constexpr uint32_t kIcOpen = 0xFFu;   // phase of a node with less than k records

// An in-edge (u -> w): its source, its threshold and the seed of its coin
// stream, SM(seed, kIcEdge + u n + w).
struct alignas(16) IcEdge {
    uint64_t stream;
    uint32_t src, thr;
};

// Its coin in the instance of position t (>= 1): the high (t - 1 even) or low
// (t - 1 odd) half of output floor((t - 1) / 2) of that stream.  `step` is
// ic_step(t), the stream position times the SplitMix64 increment.
__device__ __forceinline__ uint64_t ic_step(uint32_t t) {
    return ((uint64_t)((t - 1) / 2) + 1) * kGolden;
}
__device__ __forceinline__ bool ic_live(const IcEdge &e, uint64_t step, uint32_t t) {
    const uint64_t h = sm_mix(e.stream + step);
    return (((t - 1) & 1u) == 0 ? (uint32_t)(h >> 32) : (uint32_t)h) <= e.thr;
}

// In-edges grouped by head: the edges radix-sorted by head (key head << 32 |
// source, value the threshold), then their coin streams, and the heads' offsets
// from the places where the head changes.  (Counting and placing by an atomic
// per edge took 175 us on 320,000 edges, most of it queueing on the hubs.)
__global__ void k_ic_keys(const uint32_t *esrc, const uint32_t *col, uint64_t m, uint64_t *key) {
    for (uint64_t e = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; e < m;
         e += (uint64_t)gridDim.x * blockDim.x)
        key[e] = (uint64_t)col[e] << 32 | esrc[e];
}
__global__ void k_ic_rfill(const uint64_t *key, const uint32_t *thr, uint64_t m, uint32_t n,
                           uint64_t seed, uint64_t *rptr, IcEdge *redge) {
    for (uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; t < m;
         t += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t w = (uint32_t)(key[t] >> 32), u = (uint32_t)key[t];
        redge[t] = {sm_at(seed, kIcEdge + (uint64_t)u * n + w), u, thr[t]};
        // rptr of this head and of the heads without in-edges before it
        for (uint32_t x = t ? (uint32_t)(key[t - 1] >> 32) + 1 : 0; x <= w; ++x) rptr[x] = t;
        if (t + 1 == m)
            for (uint32_t x = w + 1; x <= n; ++x) rptr[x] = m;
    }
}

// Keys of the structured permutation: the chunk in the leading bits, then the
// leading bits of h_c(v); one sort orders every chunk.
__global__ void k_ic_hash(uint32_t n, uint32_t k, uint32_t chunk_bits, uint64_t seed,
                          uint64_t *keys, uint32_t *vals) {
    const uint64_t total = (uint64_t)n * k;
    for (uint64_t x = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; x < total;
         x += (uint64_t)gridDim.x * blockDim.x) {
        keys[x] = (x / n) << (64 - chunk_bits) | sm_at(seed, kIcChunk + x) >> chunk_bits;
        vals[x] = (uint32_t)(x % n);  // x = c n + v
    }
}

// The hash's last chunk_bits bits are not in the keys: runs of equal keys (about
// n^2 k / 2^(65 - chunk_bits) pairs) are put in order of the whole hash by the
// thread at their start.
__global__ void k_ic_ties(const uint64_t *keys, uint32_t *vals, uint32_t n, uint64_t total,
                          uint64_t seed) {
    for (uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; t + 1 < total;
         t += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t key = keys[t];
        if (keys[t + 1] != key || (t > 0 && keys[t - 1] == key)) continue;
        const uint64_t base = kIcChunk + t / n * n;  // the run lies within a chunk
        for (uint64_t i = t + 1; i < total && keys[i] == key; ++i) {
            const uint32_t v = vals[i];
            uint64_t j = i;
            for (; j > t && sm_at(seed, base + vals[j - 1]) > sm_at(seed, base + v); --j)
                vals[j] = vals[j - 1];
            vals[j] = v;
        }
    }
}

struct IcArgs {
    uint32_t n, k;
    const uint64_t *rptr;
    const IcEdge *redge;
    const uint32_t *node_at;  // [k n] node at position t = index + 1
    uint32_t *counts;         // [k n] pass 0 out
    const uint64_t *offsets;  // [k n + 1] pass 1 in
    uint64_t *records;        // pass 1 out (pass 2: appended, up to rcap)
    unsigned long long *rcount;  // pass 2: records appended
    uint64_t rcap;
    uint32_t tbits;           // a record is node << tbits | t
    uint32_t *ovf;            // pass 2: the records outgrew rcap
    uint32_t *had;            // [n] pass 2: records of a node, counted up to k
    uint8_t *full;            // [n] pass 2: phase in which it had k (kIcOpen: none yet)
    uint32_t *more;           // positions handed to a wave each
    unsigned long long *nmore;
    uint32_t *heavy;          // positions handed to the workgroup search
    unsigned long long *nheavy;
    uint32_t *hbitmaps;       // [workgroups][(n + 31) / 32]
    uint32_t *hqueues;        // [workgroups][n]
};

template <class T> __device__ __forceinline__ T ic_ld(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T> __device__ __forceinline__ void ic_st(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Phase of position index x: chunk 0 is phase 0, chunks 4^(p-1) .. 4^p - 1 are
// phase p (of twofold length the phases left the chip half empty at their ends
// more often than the fewer records paid for).
__device__ __forceinline__ uint32_t ic_phase(uint64_t x, uint32_t n) {
    const uint32_t c = (uint32_t)(x / n);
    return c ? (33u - (uint32_t)__clz((int)c)) / 2 : 0u;
}

// One wave, the searches of up to kB positions at once: positions x0 + first ..
// of an index range, or of a list.  All visited (search, node) entries stand in
// one queue in LDS, in the order found; a step takes the next 64 entries,
// whichever searches they belong to, lays their nodes' in-edges end to end and
// tests 64 at a time, so neither a search of a thousand nodes nor a hub's
// thousands of in-edges hold the other lanes.  An entry new to the wave's
// visited set (an LDS hash set of entries, at most half full) is appended.
//
// What bounds it: dependent LDS and L2 accesses per step, and the coins (213 M
// of them on the graph below).  With a thread per position, taking one node per
// step, and visited bitmaps in global memory, a wave took as many steps as its
// largest search had nodes and two device atomics per visited node: 3.3 ms on
// the 20,000-node weighted-cascade graph (k = 64, 1.28 M searches of 12 nodes on
// average, 200 at most); this 1.5 ms in
// all phases.
//
// kPass 0 counts each search's nodes, 1 writes its records at its offset, 2
// (the single pass, when the records fit a buffer sized up front) appends the
// records that can still matter.  A wave whose queue overflows hands its
// positions on: to `more` (a wave each), or with one position to `heavy`.
template <int kPass, uint32_t kB, uint32_t kCap, uint32_t kHash>
__global__ void __launch_bounds__(64) k_ic_wave(IcArgs A, uint64_t x0, uint64_t x1,
                                                const uint32_t *list) {
    __shared__ uint32_t F[kCap];   // search << kIcNodeBits | node
    __shared__ uint32_t H[kHash];  // entries, or all ones
    __shared__ uint64_t s_off[64], s_step[kB], s_stage[kPass == 2 ? kIcStage : 1];
    __shared__ uint32_t s_t[kB], s_cnt[kB];
    __shared__ uint8_t s_rank[64], s_mark[64 * kIcAhead];
    constexpr uint32_t kMask = (1u << kIcNodeBits) - 1;
    const uint32_t lane = threadIdx.x;
    const unsigned long long lower = (1ull << lane) - 1ull;
    uint32_t staged = 0;  // uniform
    auto flush = [&]() {
        wave_sync();
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(A.rcount, (unsigned long long)staged);
        base = ((unsigned long long)(uint32_t)__shfl((int)(uint32_t)(base >> 32), 0) << 32) |
               (uint32_t)__shfl((int)(uint32_t)base, 0);
        if (base + staged <= A.rcap) {
            for (uint32_t j = lane; j < staged; j += 64) A.records[base + j] = s_stage[j];
        } else if (lane == 0) {
            atomicOr(A.ovf, 1u);
        }
        staged = 0;
        wave_sync();
    };
    for (uint64_t b = x0 + (uint64_t)blockIdx.x * kB; b < x1; b += (uint64_t)gridDim.x * kB) {
        const uint32_t m = x1 - b < kB ? (uint32_t)(x1 - b) : kB;
        wave_sync();
        for (uint32_t j = lane; j < kHash; j += 64) H[j] = 0xFFFFFFFFu;
        if (lane < m) {
            const uint32_t x = list ? list[b + lane] : (uint32_t)(b + lane);
            s_t[lane] = x + 1;
            s_step[lane] = ic_step(x + 1);
            s_cnt[lane] = 0;
            F[lane] = lane << kIcNodeBits | A.node_at[x];
        }
        wave_sync();
        // true if `e` is new to the visited set
        auto insert = [&](uint32_t e) {
            uint32_t h = (e * 0x9E3779B1u) >> 16;
            for (;;) {
                h &= kHash - 1;
                const uint32_t old = atomicCAS(&H[h], 0xFFFFFFFFu, e);
                if (old == 0xFFFFFFFFu) return true;
                if (old == e) return false;
                ++h;
            }
        };
        if (lane < m) insert(F[lane]);
        uint32_t head = 0, tail = m;
        bool over = false;
        while (head < tail && !over) {  // uniform
            const uint32_t T = min(tail - head, 64u);
            uint32_t d = 0, r = 0;
            uint64_t e0 = 0;
            if (lane < T) {
                const uint32_t f = F[head + lane], y = f & kMask;
                r = f >> kIcNodeBits;
                e0 = A.rptr[y];
                d = (uint32_t)(A.rptr[y + 1] - e0);
            }
            head += T;
            const uint32_t incl = wave_scan_sum(d), first = incl - d;
            const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            s_off[lane] = e0 - first;  // in-edge of flat position j: s_off + j
            s_rank[lane] = (uint8_t)r;
            uint32_t carry = 0;  // owner (lane + 1) of the round's first positions
            for (uint32_t base = 0; base < tot && !over; base += 64 * kIcAhead) {
                // owners: lanes mark their first position, the last mark at or
                // before a position owns it
#pragma unroll
                for (uint32_t w = 0; w < kIcAhead; ++w) s_mark[64 * w + lane] = 0;
                wave_sync();
                if (d && first >= base && first - base < 64 * kIcAhead)
                    s_mark[first - base] = (uint8_t)(lane + 1);
                wave_sync();
                // the round's edges, all loads in flight before the first coin
                IcEdge e[kIcAhead];
                uint32_t rr[kIcAhead];
#pragma unroll
                for (uint32_t w = 0; w < kIcAhead; ++w) {
                    if (base + 64 * w >= tot) break;  // uniform
                    uint32_t o = wave_scan_max(s_mark[64 * w + lane]);
                    o = o ? o : carry;
                    carry = (uint32_t)__builtin_amdgcn_readlane((int)o, 63);
                    const uint32_t j = base + 64 * w + lane;
                    if (j < tot) {
                        rr[w] = s_rank[o - 1];
                        e[w] = A.redge[s_off[o - 1] + j];
                    }
                }
#pragma unroll
                for (uint32_t w = 0; w < kIcAhead; ++w) {
                    if (base + 64 * w >= tot || over) break;  // uniform
                    bool add = false;
                    uint32_t f = 0;
                    if (base + 64 * w + lane < tot && ic_live(e[w], s_step[rr[w]], s_t[rr[w]])) {
                        f = rr[w] << kIcNodeBits | e[w].src;
                        add = insert(f);
                    }
                    const unsigned long long am = __ballot(add);
                    const uint32_t c = (uint32_t)__popcll(am);
                    if (tail + c > kCap) {  // the set holds at most kCap + 64 entries
                        over = true;
                        break;
                    }
                    if (add) F[tail + (uint32_t)__popcll(am & lower)] = f;
                    tail += c;
                }
            }
            wave_sync();
        }
        if (over) {
            uint32_t *out = kB == 1 ? A.heavy : A.more;
            unsigned long long *cnt = kB == 1 ? A.nheavy : A.nmore;
            unsigned long long at = 0;
            if (lane == 0) at = atomicAdd(cnt, (unsigned long long)m);
            at = (uint32_t)__shfl((int)(uint32_t)at, 0);  // fewer than 2^32 positions
            if (lane < m) out[at + lane] = s_t[lane] - 1;
            continue;
        }
        for (uint32_t j0 = 0; j0 < tail; j0 += 64) {
            const uint32_t j = j0 + lane;
            const uint32_t f = j < tail ? F[j] : 0u, u = f & kMask, r = f >> kIcNodeBits;
            const uint32_t t = j < tail ? s_t[r] : 1u;
            if constexpr (kPass == 2) {
                bool rec = false;
                if (j < tail) {
                    const uint32_t ph = ic_phase(t - 1, A.n);
                    rec = ic_ld(A.full + u) >= ph;
                    // counted until it is known to have k: while the phases
                    // are run in order, those are of phases up to this one
                    // (positions handed on come after the last phase, and do
                    // not count)
                    if (rec && !list && ic_ld(A.had + u) < A.k && atomicAdd(A.had + u, 1u) + 1 == A.k)
                        ic_st(A.full + u, (uint8_t)ph);
                }
                const unsigned long long rm = __ballot(rec);
                if (staged + 64 > kIcStage) flush();
                if (rec)
                    s_stage[staged + (uint32_t)__popcll(rm & lower)] = ((uint64_t)u << A.tbits) | t;
                staged += (uint32_t)__popcll(rm);
            } else if (j < tail) {
                const uint32_t at = atomicAdd(&s_cnt[r], 1u);
                if (kPass == 1) A.records[A.offsets[t - 1] + at] = ((uint64_t)u << A.tbits) | t;
            }
        }
        if (kPass == 0) {
            wave_sync();
            if (lane < m) A.counts[s_t[lane] - 1] = s_cnt[lane];
        }
    }
    if (kPass == 2 && staged) flush();
}

// One workgroup per handed-over position: the breadth-first search takes up
// to kIcHeavyBlock queue entries per round, one per thread; new nodes are
// marked in the workgroup's bitmap with an atomic OR and appended with one
// LDS atomic per wave.
template <int kPass>
__global__ void __launch_bounds__(kIcHeavyBlock) k_ic_heavy(IcArgs A, uint64_t nheavy) {
    __shared__ unsigned long long s_tail;
    const uint32_t tid = threadIdx.x;
    const uint32_t words = (A.n + 31) / 32;
    uint32_t *bm = A.hbitmaps + (uint64_t)blockIdx.x * words;
    uint32_t *Q = A.hqueues + (uint64_t)blockIdx.x * A.n;
    for (uint64_t h = blockIdx.x; h < nheavy; h += gridDim.x) {
        const uint64_t x = A.heavy[h];
        const uint32_t t = (uint32_t)(x + 1);
        const uint64_t step = ic_step(t);
        if (tid == 0) {
            const uint32_t v = A.node_at[x];
            atomicOr(bm + (v >> 5), 1u << (v & 31));
            ic_st(Q, v);
            s_tail = 1;
        }
        __syncthreads();
        uint64_t head = 0;
        for (;;) {
            const uint64_t tail = s_tail;
            __syncthreads();  // every thread has the same tail before any append
            if (head >= tail) break;
            const uint64_t chunk = tail - head < (uint64_t)kIcHeavyBlock ? tail - head : kIcHeavyBlock;
            if (tid < chunk) {
                const uint32_t y = ic_ld(Q + head + tid);
                for (uint64_t e = A.rptr[y]; e < A.rptr[y + 1]; ++e) {
                    const IcEdge edge = A.redge[e];
                    const uint32_t u = edge.src, bit = 1u << (u & 31);
                    bool add = (ic_ld(bm + (u >> 5)) & bit) == 0 && ic_live(edge, step, t);
                    if (add) add = (atomicOr(bm + (u >> 5), bit) & bit) == 0;
                    const uint64_t slot = wave_reserve(&s_tail, add);
                    if (add) ic_st(Q + slot, u);
                }
            }
            head += chunk;
            __syncthreads();  // this round's appends are in the queue and s_tail
        }
        const uint64_t cnt = s_tail;
        if (kPass == 0) {
            if (tid == 0) A.counts[x] = (uint32_t)cnt;
        } else {
            uint64_t *out = A.records + A.offsets[x];
            for (uint64_t j = tid; j < cnt; j += kIcHeavyBlock)
                out[j] = ((uint64_t)ic_ld(Q + j) << A.tbits) | t;
        }
        for (uint64_t j = tid; j < cnt; j += kIcHeavyBlock) ic_st(bm + (ic_ld(Q + j) >> 5), 0u);
        __syncthreads();  // the bitmap is clean before the next position
    }
}

// start[u] = index of u's first record (every node has records).
__global__ void k_ic_starts(const uint64_t *rec, uint64_t R, uint32_t tbits, uint64_t *start) {
    for (uint64_t j = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; j < R;
         j += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t node = (uint32_t)(rec[j] >> tbits);
        if (j == 0 || (uint32_t)(rec[j - 1] >> tbits) != node) start[node] = j;
    }
}

// One wave per node.
__global__ void __launch_bounds__(256) k_ic_select(const uint64_t *rec, const uint64_t *start,
                                                   uint32_t n, uint32_t k, uint32_t tbits,
                                                   uint32_t *pos, double *est) {
    const uint64_t mask = (1ull << tbits) - 1;
    const uint64_t waves = (uint64_t)gridDim.x * 4;
    for (uint64_t u = blockIdx.x * 4ull + threadIdx.x / 64; u < n; u += waves) {
        const uint64_t s = start[u];
        for (uint32_t j = threadIdx.x & 63u; j < k; j += 64)
            pos[u * k + j] = (uint32_t)(rec[s + j] & mask);
        if (est && (threadIdx.x & 63u) == 0) {
            const uint32_t T = (uint32_t)(rec[s + k - 1] & mask);
            est[u] = ((double)n * (double)(k - 1)) / (double)(T - 1);
        }
    }
}

// ------------------------------------------------------------ union queries
// One wave per query; each lane keeps the current heads and thresholds of
// its members in registers, so a step of the k-way merge reads global memory
// only for the members holding the current minimum.
constexpr uint32_t kIcMaxMembers = 1024;
constexpr uint32_t kIcNoPos = 0xFFFFFFFFu;

__global__ void k_icq_offsets(const uint64_t *qoff, uint64_t q, uint32_t *err) {
    for (uint64_t j = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; j <= q;
         j += (uint64_t)gridDim.x * blockDim.x) {
        const bool bad = j == 0 ? qoff[0] != 0 : qoff[j - 1] > qoff[j];
        if (bad) atomicOr(err, 1u);
    }
}

__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t y = __shfl_xor(x, off);
        x = y < x ? y : x;
    }
    return x;
}

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t x) {
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t y = __shfl_xor(x, off);
        x = y > x ? y : x;
    }
    return x;
}

// The k-way merge over S members with R >= S / 64 register slots per lane:
// lane l keeps the current head and threshold of members l + 64 r.
template <int R>
__device__ __forceinline__ void ic_merge(const uint32_t *pos, uint32_t n, uint32_t k,
                                         uint32_t estimator, uint32_t S, const uint32_t *mnode,
                                         uint32_t &T, double &sum) {
    const uint32_t lane = threadIdx.x;
    const uint32_t lim = estimator == 1 ? k - 1 : k;  // CK leaves out each threshold
    uint32_t head[R], thr[R], at[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t t = lane + 64u * r;
        head[r] = kIcNoPos;
        thr[r] = 0;
        at[r] = 0;
        if (t < S) {
            const uint64_t row = (uint64_t)mnode[t] * k;
            head[r] = pos[row];
            thr[r] = pos[row + k - 1];
        }
    }
    uint32_t d = 0;
    for (;;) {
        uint32_t lmin = kIcNoPos;
#pragma unroll
        for (int r = 0; r < R; ++r) lmin = head[r] < lmin ? head[r] : lmin;
        const uint32_t g = wave_min_u32(lmin);
        if (g == kIcNoPos) break;
        uint32_t tmax = 0;
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (head[r] == g) {
                const uint32_t p = ++at[r];
                head[r] = p < lim ? pos[(uint64_t)mnode[lane + 64u * r] * k + p] : kIcNoPos;
                tmax = thr[r] > tmax ? thr[r] : tmax;
            }
        if (estimator == 1) {
            tmax = wave_max_u32(tmax);
            if (lane == 0) sum += (double)n / (double)(tmax - 1);
        } else if (++d == k) {
            T = g;
            break;
        }
    }
}

__global__ void __launch_bounds__(64) k_ic_query(const uint32_t *pos, uint32_t n, uint32_t k,
                                                 uint64_t q, const uint64_t *qoff,
                                                 const uint32_t *qnodes, uint32_t estimator,
                                                 double *est, int32_t *qstatus) {
    __shared__ uint32_t mnode[kIcMaxMembers];
    const uint32_t lane = threadIdx.x;
    for (uint64_t j = blockIdx.x; j < q; j += gridDim.x) {
        const uint64_t a = qoff[j], b = qoff[j + 1], S = b - a;
        bool bad = false;
        for (uint64_t t = a + lane; t < b; t += 64) bad |= qnodes[t] >= n;
        bad = __ballot(bad) != 0;
        if (bad || S == 0 || S > kIcMaxMembers) {
            if (lane == 0) {
                est[j] = 0.0;
                if (qstatus) qstatus[j] = bad ? -1 : (S == 0 ? 0 : -2);
            }
            continue;
        }
        for (uint32_t t = lane; t < S; t += 64) mnode[t] = qnodes[a + t];
        __syncthreads();
        uint32_t T = 0;
        double sum = 0.0;
        if (S <= 64)
            ic_merge<1>(pos, n, k, estimator, (uint32_t)S, mnode, T, sum);
        else if (S <= 256)
            ic_merge<4>(pos, n, k, estimator, (uint32_t)S, mnode, T, sum);
        else
            ic_merge<kIcMaxMembers / 64>(pos, n, k, estimator, (uint32_t)S, mnode, T, sum);
        if (lane == 0) {
            est[j] = estimator == 1 ? sum : ((double)n * (double)(k - 1)) / (double)(T - 1);
            if (qstatus) qstatus[j] = 0;
        }
        __syncthreads();  // LDS is reused by the next query of the stride
    }
}

}  // namespace

}  // namespace skim

extern "C" skim_status skim_ic_query_batch(const uint32_t *positions, uint32_t n, uint32_t k,
                                           uint64_t q, const uint64_t *qoff,
                                           const uint32_t *qnodes, uint32_t estimator,
                                           double *est, int32_t *qstatus, void *stream) {
    using namespace skim;
    clear_error();
    hipStream_t hs = (hipStream_t)stream;
    try {
        SKIM_REQUIRE(k >= 2 && k <= 256, "k must be in [2, 256]");
        SKIM_REQUIRE(n >= 1 && (uint64_t)n * k < (1ull << 32), "n must be >= 1 with k n < 2^32");
        SKIM_REQUIRE(estimator <= 1, "estimator must be 0 (bottom-k) or 1 (Cohen-Kaplan)");
        SKIM_REQUIRE(positions != nullptr, "positions is NULL");
        if (q == 0) return SKIM_OK;
        SKIM_REQUIRE(qoff && est, "qoff/est is NULL");
        Arena T(hs);
        uint32_t *err = T.alloc<uint32_t>(1);
        fill_u32(err, 0, 1, hs);
        k_icq_offsets<<<grid_for(q + 1, 256, 4096), 256, 0, hs>>>(qoff, q, err);
        SKIM_LAUNCH_CHECK();
        uint32_t herr = 0;
        read_back(&herr, err, sizeof herr, hs);
        SKIM_REQUIRE(herr == 0, "qoff must start at 0 and be non-decreasing");
        uint64_t total = 0;
        read_back(&total, qoff + q, sizeof total, hs);
        SKIM_REQUIRE(total == 0 || qnodes, "qnodes is NULL");
        {
            LaunchTimer t("k_ic_query", hs);
            k_ic_query<<<(unsigned)std::min<uint64_t>(q, 16384), 64, 0, hs>>>(
                positions, n, k, q, qoff, qnodes, estimator, est, qstatus);
            SKIM_LAUNCH_CHECK();
        }
        SKIM_HIP(hipStreamSynchronize(hs));
        return SKIM_OK;
    } catch (const Fail &f) {
        return f.st;
    }
}

extern "C" skim_status skim_build_ic_sketches(const skim_graph *g, uint32_t k, uint64_t seed,
                                              uint32_t *positions, double *est, void *stream) {
    using namespace skim;
    clear_error();
    hipStream_t hs = (hipStream_t)stream;
    try {
        SKIM_REQUIRE(g != nullptr, "graph is NULL");
        SKIM_REQUIRE(k >= 2 && k <= 256, "k must be in [2, 256]");
        SKIM_REQUIRE(positions != nullptr, "positions is NULL");
        SKIM_REQUIRE((uint64_t)g->n * k < (1ull << 32), "k n must be below 2^32");
        Arena T(hs);
        const uint32_t n = g->n;
        const uint64_t m = g->m;
        uint32_t *esrc = T.alloc<uint32_t>(m ? m : 1);
        validate_graph(g, esrc, T);
        // reverse graph with thresholds
        int node_bits = 1;
        while (node_bits < 32 && (1ull << node_bits) < n) ++node_bits;
        uint64_t *rptr = T.alloc<uint64_t>((uint64_t)n + 1);
        IcEdge *redge = T.alloc<IcEdge>(m ? m : 1);
        if (m) {
            uint64_t *key = T.alloc<uint64_t>(m), *skey = T.alloc<uint64_t>(m);
            uint32_t *sthr = T.alloc<uint32_t>(m);
            k_ic_keys<<<grid_for(m, 256, 16384), 256, 0, hs>>>(esrc, g->col, m, key);
            SKIM_LAUNCH_CHECK();
            size_t tb = 0;
            SKIM_HIP(rocprim::radix_sort_pairs<FewBits>(nullptr, tb, key, skey,
                                                        (const uint32_t *)g->thr, sthr, (size_t)m,
                                                        32, 32 + node_bits, hs));
            void *tmp = T.get(tb ? tb : 1);
            SKIM_HIP(rocprim::radix_sort_pairs<FewBits>(tmp, tb, key, skey,
                                                        (const uint32_t *)g->thr, sthr, (size_t)m,
                                                        32, 32 + node_bits, hs));
            k_ic_rfill<<<grid_for(m, 256, 16384), 256, 0, hs>>>(skey, sthr, m, n, seed, rptr,
                                                               redge);
            SKIM_LAUNCH_CHECK();
            for (void *p : {(void *)key, (void *)skey, (void *)sthr, tmp}) T.release(p);
        } else {
            fill_u64(rptr, 0, (uint64_t)n + 1, hs);
        }
        // the structured permutation: chunk c orders the nodes by their hash
        const uint64_t total = (uint64_t)n * k;
        uint64_t *hkeys = T.alloc<uint64_t>(total);
        uint64_t *hkeys2 = T.alloc<uint64_t>(total);
        uint32_t *hvals = T.alloc<uint32_t>(total);
        uint32_t *node_at = T.alloc<uint32_t>(total);
        uint32_t chunk_bits = 1;
        while ((1u << chunk_bits) < k) ++chunk_bits;
        k_ic_hash<<<grid_for(total, 256, 16384), 256, 0, hs>>>(n, k, chunk_bits, seed, hkeys,
                                                              hvals);
        SKIM_LAUNCH_CHECK();
        size_t tmp_bytes = 0;
        SKIM_HIP(rocprim::radix_sort_pairs(nullptr, tmp_bytes, hkeys, hkeys2, hvals, node_at,
                                           (size_t)total, 0u, 64u, hs));
        void *tmp = T.get(tmp_bytes);
        SKIM_HIP(rocprim::radix_sort_pairs(tmp, tmp_bytes, hkeys, hkeys2, hvals, node_at,
                                           (size_t)total, 0u, 64u, hs));
        k_ic_ties<<<grid_for(total, 256, 16384), 256, 0, hs>>>(hkeys2, node_at, n, total, seed);
        SKIM_LAUNCH_CHECK();
        T.release(tmp);
        T.release(hkeys);
        T.release(hkeys2);
        T.release(hvals);
        const uint32_t words = (n + 31) / 32;
        IcArgs A{};
        A.n = n;
        A.k = k;
        A.rptr = rptr;
        A.redge = redge;
        A.node_at = node_at;
        A.tbits = 1;
        while ((total >> A.tbits) != 0) ++A.tbits;  // t <= k n < 2^32
        A.counts = T.alloc<uint32_t>(total);
        A.had = T.alloc<uint32_t>(n);
        A.full = T.alloc<uint8_t>((uint64_t)n + 4);
        A.more = T.alloc<uint32_t>(total);
        A.heavy = T.alloc<uint32_t>(total);
        A.nmore = T.alloc<unsigned long long>(1);
        A.nheavy = T.alloc<unsigned long long>(1);
        // One pass when the records fit a buffer sized up front (32 per
        // position, at most kIcRecordCap): they are appended as the searches
        // end.  Otherwise, or for the workgroup searches, a counting pass, a
        // scan and a writing pass.
        uint64_t rcap = std::min<uint64_t>(std::max<uint64_t>(total * 32, 1u << 20), kIcRecordCap);
        if (take_fault(kFaultIcRecords)) rcap = 1;  // tests of the counting path
        uint64_t *recbuf = T.alloc<uint64_t>(rcap);
        A.records = recbuf;
        A.rcap = rcap;
        A.rcount = T.alloc<unsigned long long>(1);
        A.ovf = T.alloc<uint32_t>(1);
        fill_u64((uint64_t *)A.rcount, 0, 1, hs);
        fill_u32(A.ovf, 0, 1, hs);
        fill_u32(A.counts, 0, total, hs);  // a workgroup search's count comes from its own pass
        fill_u32(A.had, 0, n, hs);
        fill_u32((uint32_t *)A.full, kIcOpen * 0x01010101u, (n + 3) / 4, hs);
        // two batches of positions per wave, one where that leaves waves idle
        // (equal shares of all of them: waves idle at the ends of the phases;
        // four 2.76 ms, eight 3.35 ms)
        constexpr unsigned kGrid = 1u << 20;
        auto grid_of = [&](uint64_t batches) {
            return grid_for(batches, batches > 8192 ? 2 : 1, kGrid);
        };
        // every position, then the ones a wave handed on; leaves nheavy
        uint64_t nheavy = 0;
        auto searches = [&](auto pass) {
            constexpr int kPass = decltype(pass)::value;
            fill_u64((uint64_t *)A.nmore, 0, 1, hs);
            fill_u64((uint64_t *)A.nheavy, 0, 1, hs);
            LaunchTimer t("k_ic_search", hs);
            for (uint64_t c0 = 0, c1 = 1; c0 < k; c0 = c1, c1 = 4 * c1) {
                if (kPass != 2) c1 = k;  // phases only matter to the appending pass
                const uint64_t x0 = c0 * n, x1 = std::min<uint64_t>(c1, k) * n;
                k_ic_wave<kPass, kIcWave, kIcQueue, kIcSlots>
                    <<<grid_of((x1 - x0 + kIcWave - 1) / kIcWave), 64, 0, hs>>>(A, x0, x1, nullptr);
                SKIM_LAUNCH_CHECK();
            }
            uint64_t nmore = 0;
            read_back(&nmore, A.nmore, sizeof nmore, hs);
            if (nmore) {
                k_ic_wave<kPass, 1, kIcOne, 2 * kIcOne>
                    <<<grid_of(nmore), 64, 0, hs>>>(A, 0, nmore, A.more);
                SKIM_LAUNCH_CHECK();
                read_back(&nheavy, A.nheavy, sizeof nheavy, hs);
            }
        };
        searches(std::integral_constant<int, 2>{});
        uint32_t ovf = 0;
        uint64_t rlight = 0;
        read_back(&ovf, A.ovf, sizeof ovf, hs);
        read_back(&rlight, A.rcount, sizeof rlight, hs);
        if (ovf) {  // back to counting first
            rlight = 0;
            searches(std::integral_constant<int, 0>{});
        }
        unsigned hgrid = 1;
        if (nheavy) {
            const uint64_t per_block = ((uint64_t)words + n) * sizeof(uint32_t);
            uint64_t blocks = std::max<uint64_t>(1, kIcHeavyBudget / per_block);
            blocks = std::min<uint64_t>(std::min<uint64_t>(blocks, 1024), nheavy);
            hgrid = (unsigned)blocks;
            A.hbitmaps = T.alloc<uint32_t>(blocks * words);
            A.hqueues = T.alloc<uint32_t>(blocks * n);
            fill_u32(A.hbitmaps, 0, blocks * words, hs);
            LaunchTimer t("k_ic_heavy", hs);
            k_ic_heavy<0><<<hgrid, kIcHeavyBlock, 0, hs>>>(A, nheavy);
            SKIM_LAUNCH_CHECK();
        }
        // offsets of what is still to be written: every search after a
        // counting pass, the workgroup searches after the single pass
        uint64_t rrest = 0;
        if (ovf || nheavy) {
            uint64_t *offsets = T.alloc<uint64_t>(total + 1);
            exclusive_scan_u32(A.counts, offsets, total, T);
            read_back(&rrest, offsets + total, sizeof rrest, hs);
            A.offsets = offsets;
        }
        const uint64_t R = rlight + rrest;
        uint64_t *records = recbuf;
        if (R > rcap) {  // room for the rest after the appended records
            records = T.alloc<uint64_t>(R);
            if (rlight)
                SKIM_HIP(hipMemcpyAsync(records, recbuf, rlight * sizeof(uint64_t),
                                        hipMemcpyDeviceToDevice, hs));
            T.release(recbuf);
        }
        A.records = records + rlight;
        if (ovf) searches(std::integral_constant<int, 1>{});
        if (nheavy) {
            LaunchTimer t("k_ic_heavy", hs);
            k_ic_heavy<1><<<hgrid, kIcHeavyBlock, 0, hs>>>(A, nheavy);
            SKIM_LAUNCH_CHECK();
        }
        A.records = records;
        if (nheavy) {
            T.release(A.hbitmaps);
            T.release(A.hqueues);
        }
        // records by (node, position); every node keeps its first k
        uint64_t *sorted = T.alloc<uint64_t>(R);
        // the keys' bits above the node id are zero: large sorts skip them
        // (small ones take the whole key)
        const unsigned end_bit = R > (1ull << 20) ? A.tbits + (unsigned)node_bits : 64u;
        tmp_bytes = 0;
        SKIM_HIP(rocprim::radix_sort_keys(nullptr, tmp_bytes, A.records, sorted, (size_t)R, 0u,
                                          end_bit, hs));
        tmp = T.get(tmp_bytes);
        SKIM_HIP(rocprim::radix_sort_keys(tmp, tmp_bytes, A.records, sorted, (size_t)R, 0u, end_bit,
                                          hs));
        uint64_t *start = T.alloc<uint64_t>(n);
        k_ic_starts<<<grid_for(R, 256, 16384), 256, 0, hs>>>(sorted, R, A.tbits, start);
        SKIM_LAUNCH_CHECK();
        k_ic_select<<<grid_for(n, 4, 16384), 256, 0, hs>>>(sorted, start, n, k, A.tbits, positions,
                                                           est);
        SKIM_LAUNCH_CHECK();
        SKIM_HIP(hipStreamSynchronize(hs));
        return SKIM_OK;
    } catch (const Fail &f) {
        return f.st;
    }
}
