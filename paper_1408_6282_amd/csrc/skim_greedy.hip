// skim_greedy.hip -- SKIM greedy seed selection (Section 4, Algorithm 1).
//
// State on the device: live reverse and forward lists of every pair, the
// pairs sorted by rank, covered[pair], size[node], and the inverted index
// (for every processed pair, the nodes its reverse search reached).
//
// One persistent workgroup runs the selection loop (the loop is sequential
// per seed); residual searches that grow large continue on the whole grid:
//  * scan: the next B pairs in rank order each run their complete reverse
//    search in parallel (one thread per pair; an uncovered pair never reaches
//    a covered one, so the searches are independent of each other's
//    increments).  If some node's size reaches k with all B pairs, the first
//    prefix length T at which one does is the smallest position at which a
//    filling node receives its (k - size)-th entry, found from the entries
//    of the filling nodes alone (binary search over prefixes when there are
//    too many); pairs [0, T) are committed (size increments, index entries),
//    the rest are re-scanned later.  The nodes that reached k all sit in
//    pair T-1's search; the smallest id among them is the seed.  Batches
//    with a long search spread the per-entry work over the block by flat
//    position instead of per thread.
//  * exhaustion: with every rank processed, the unselected node with the
//    largest size (smallest id on ties) is the seed.
//  * records: before the residual update, the rank tau of the pair that filled
//    the seed's sketch and the second largest sketch k' (largest size among
//    the other unselected nodes, one less for nodes in that pair's search)
//    are stored per seed for the adaptive error estimate (Section 4).
//  * residual: a level-synchronous forward search from the seed over all
//    instances at once (each level's frontier of pairs shared by the block)
//    over live out-edges, not entering covered pairs; every newly covered
//    pair counts towards the seed's gain and decrements the size of every
//    node in its index entry, which is then erased.  A level of more than
//    kSkimHandoff pairs, or a seed with more than kSkimHandoffEdges live
//    out-edges, ends the workgroup's launch; the host runs the rest of that
//    search level by level on the whole grid (k_resid_level; pairs of long
//    out-lists are expanded edge-balanced by the next level's launch) and then
//    relaunches the loop; a search whose next level there is small again is
//    handed back, and the relaunched loop resumes it at that level.
//
// The adaptive error estimate itself (skim_discrepancy_tail) bounds each
// seed's discrepancy with eq. (chernoff) on a grid of discrepancy values and
// convolves the per-seed distributions pairwise in a tree of launches.
#include "skim_internal.h"
#include "skim_wave.h"

#include <mutex>

#include <rocprim/device/device_radix_sort.hpp>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <utility>

namespace skim {

namespace {

constexpr int kSkimBlock = 1024;
constexpr uint32_t kSkimLdsNodes = 20480;  // graphs up to this size keep size[] in LDS
constexpr uint32_t kSkimPairListNodes = 1u << 17;  // from this size, in-lists as pair words
constexpr uint32_t kSkimLdsWords = kSkimLdsNodes / 2;
constexpr uint32_t kFlagPool = 1u, kFlagAhead = 2u;
// Items whose search, index entry or out-list is at most this long are
// walked by their own thread; a batch or level with a longer one spreads
// its work over the block by flat position.
constexpr uint32_t kSkimSerial = 32;
// ... and a wave whose items all have at most this many walks them lane by
// lane; with a longer one the wave lays them end to end.
constexpr uint32_t kSkimFlat = 4;
// A residual level with more pairs than this continues on the whole grid.
constexpr uint64_t kSkimHandoff = 4096;
// ... and so does a seed whose own live out-edges are more than this.
constexpr uint64_t kSkimHandoffEdges = 65536;
// A search on the grid whose next level has at most this many pairs goes
// back to the workgroup (a level there costs less than two launches).
constexpr uint64_t kSkimHandBack = 2048;
// On the grid, pairs with more live out-edges than this are deferred to the
// next level's launch, which spreads their edges over every workgroup before
// it takes its own frontier (their heads join the level after it: the
// covered set does not depend on the order of the expansions).  At most
// kHeavyItems per level; more are expanded where they are.
constexpr uint64_t kSplitEdges = 1024;
constexpr uint32_t kHeavyItems = 1u << 16;
// Entries of the nodes that fill within a batch, kept to find the filling
// prefix directly (more: binary search over prefixes).
constexpr uint32_t kSkimCand = 1024;
// Entries of a batch that fit in LDS.
constexpr uint32_t kSkimStage = 8192;
// The first kSkimLdsFront entries of a residual level in the workgroup live
// in LDS (the rest in the queue area): small levels never go through global
// memory between one level and the next.
constexpr uint32_t kSkimLdsFront = 2048;
constexpr int kResidBlock = 256;
constexpr uint32_t kResidGrid = 512;

struct SkCtl {
    unsigned long long cursor;     // next position in the rank order
    unsigned long long pool_used;  // index entries in use
    unsigned long long need;       // pool entries a failed batch needed
    uint32_t done;                 // seeds completed by the last launch
    uint32_t flags;
    // A residual search handed to the whole grid (its frontier outgrew the
    // workgroup): the seed, the frontier buffer of its current level, the
    // pairs covered so far, and the level sizes (each counter on a line of
    // its own; level L reads rsize[L % 3], appends to rsize[(L + 1) % 3]).
    uint32_t pend, px, rcur, pad;
    unsigned long long rgain;
    // The window of searches ahead: positions [a_lo, a_lo + min(a_w, a_fail)),
    // pool entries taken, searches left to the wave and workgroup kernels.
    unsigned long long a_lo, a_w, a_fail, a_used, nlong, ngiant;
    unsigned long long pad2[4];
    unsigned long long rsize[3 * 16];
    unsigned long long hsize[3 * 16];  // pairs level L deferred: hsize[16 (L % 3)]
};

struct SkArgs {
    uint32_t n, ell, k;
    uint64_t nsrc;
    // live in-lists: on large graphs the words of the sketch build ([64 n],
    // rlive, with rsrc), else a CSR over pairs (rptr [64 n + 1], radj)
    const uint64_t *rlive;
    const uint32_t *rsrc;
    const uint64_t *rptr;
    const uint32_t *radj;
    const uint64_t *fptr;
    const uint32_t *fadj;
    const uint32_t *order;  // pair ids by increasing rank
    uint64_t ordered;       // of them, in place so far
    uint32_t *covered;      // [64 n] 0/1
    uint32_t *size;         // [size_words(n)] packed 16-bit counters
    uint32_t *sel;          // [n] 0/1
    uint64_t *idx;          // [64 n] first pool entry << 32 | entries, 0 = no entry
    uint32_t *pool;
    uint64_t pool_cap;
    uint32_t *front;        // [2 * 64 n] residual levels
    uint64_t *ahead;        // [kAheadMax] searches of the window
    uint32_t *apool;        // [apool_cap] their nodes
    uint64_t apool_cap;
    uint32_t *along;        // [2 kAheadMax] searches left to the wave kernel, to the workgroup kernel
    uint32_t *gqueue;       // [kAheadGiants * n]
    uint64_t *heavy;        // [3][2 kHeavyItems] grid residual, deferred (pair, count), first out-edge
    uint32_t *vis;          // [kAheadGiants * vis_words] visited bitmaps, kept zero
    uint32_t vis_words;     // ceil(n / 32)
    SkCtl *ctl;
    uint64_t seed;
    uint64_t *rec_tau;      // [n] per selected seed: rank that filled its sketch
    uint32_t *rec_second;   // [n] per selected seed: second largest sketch
};

// size[] is 16-bit halves of 32-bit words (sizes stay at most 65535, see the
// scan), so twice as many nodes fit in LDS.  Adds and subtracts never carry
// across halves.  Whole 16-byte groups, zero beyond n.
__host__ __device__ inline uint32_t size_words(uint32_t n) { return (n + 7) / 8 * 4; }
__device__ __forceinline__ uint32_t half_shift(uint32_t v) { return (v & 1u) << 4; }

// State shared between the block's threads goes through agent-scope atomic
// loads and stores, so no thread reads a stale cached copy of it.
template <class T> __device__ __forceinline__ T ld(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T> __device__ __forceinline__ void st(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t cget(const uint32_t *c, uint32_t v) {
    return (ld(c + (v >> 1)) >> half_shift(v)) & 0xFFFFu;
}
__device__ __forceinline__ void cadd(uint32_t *c, uint32_t v, uint32_t d) {
    atomicAdd(c + (v >> 1), d << half_shift(v));
}
__device__ __forceinline__ void csub(uint32_t *c, uint32_t v, uint32_t d) {
    atomicSub(c + (v >> 1), d << half_shift(v));
}
__device__ __forceinline__ uint32_t cadd_old(uint32_t *c, uint32_t v, uint32_t d) {
    return (atomicAdd(c + (v >> 1), d << half_shift(v)) >> half_shift(v)) & 0xFFFFu;
}

// Exclusive prefix sum of v over the block (NT threads, called by all of
// them) and the block total; wsum holds one word per wave.
template <uint32_t NT>
__device__ __forceinline__ uint64_t block_excl_scan(uint64_t v, uint64_t *wsum, uint64_t &total) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint64_t x = v;
#pragma unroll
    for (uint32_t off = 1; off < 64; off <<= 1) {
        const uint32_t lo = __shfl_up((uint32_t)x, off), hi = __shfl_up((uint32_t)(x >> 32), off);
        if (lane >= off) x += ((uint64_t)hi << 32) | lo;
    }
    __syncthreads();  // earlier readers of wsum are done
    if (lane == 63u) wsum[wave] = x;
    __syncthreads();
    uint64_t before = 0, tot = 0;
    for (uint32_t w = 0; w < NT / 64; ++w) {
        const uint64_t s = wsum[w];
        before += w < wave ? s : 0;
        tot += s;
    }
    total = tot;
    return before + x - v;
}

// The run that holds flat position t: the largest r with ex[r] <= t, for
// exclusive prefix sums ex[0..NT] (runs of length zero are never returned
// for t below the total).
template <uint32_t NT>
__device__ __forceinline__ uint32_t run_of(const uint64_t *ex, uint64_t t) {
    uint32_t lo = 0, hi = NT;  // ex[lo] <= t < ex[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (ex[mid] <= t) lo = mid;
        else hi = mid;
    }
    return lo;
}

// Inclusive prefix sum over the wave's 64 lanes, and the lane whose range
// holds flat position j of the wave's items laid end to end (binary lifting
// over the prefix sums; j below the wave's total).
__device__ __forceinline__ uint32_t wave_incl(uint32_t v) {
    const uint32_t lane = threadIdx.x & 63u;
#pragma unroll
    for (uint32_t off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(v, off);
        if (lane >= off) v += y;
    }
    return v;
}
__device__ __forceinline__ uint32_t wave_owner(uint32_t incl, uint32_t j) {
    uint32_t r = 0;
#pragma unroll
    for (uint32_t step = 32; step > 0; step >>= 1) {
        const uint32_t v = (uint32_t)__shfl((int)incl, (int)(r + step - 1));
        if (v <= j) r += step;
    }
    return r & 63u;
}

// Work that depends on the length of a search or of an adjacency list is
// spread over the whole block by flat position (prefix sums over the
// block's items, then a binary search per position), so one long item
// does not hold up a level.
template <uint32_t NT> struct FlatShared {
    uint64_t ex[NT + 1];   // scan: queue lengths; residual: out-edges
    uint64_t ex2[NT + 1];  // residual: index entries
    uint64_t f0[NT];       // residual: first out-edge
    uint32_t q[NT];        // residual: the pair
    uint32_t o[NT];        // residual: first index entry
    uint64_t wsum[NT / 64];
};

// Appends of a grid-wide residual level, staged in LDS and reserved in
// global memory once per chunk (one counter serves the whole grid).
struct ResidStage {
    uint32_t buf[8 * kResidBlock];
    uint32_t n;
    unsigned long long base;
};

struct ScanShared {
    uint64_t cand[kSkimCand];    // (pair position << 32) | node, nodes that fill
    uint32_t seen[kSkimCand];
    uint32_t entry[kSkimStage];  // the batch's searches, laid end to end
    uint32_t ncand;
};

// One chunk of a residual level: frontier entries [base, base + NT) of
// Fin (fc entries).  Each newly covered pair's index entry is erased (its
// nodes lose one from their sizes), and its live out-edges cover the pairs
// they reach in the same instance, appended to Fout (counted in *next).
// Called by all NT threads of the block.
// Precheck: read a pair's covered flag before the CAS (fewer atomics when
// many targets are covered already; one more step of latency).
template <uint32_t NT, bool Precheck>
__device__ __forceinline__ void resid_chunk(const SkArgs &A, uint32_t *SZ, const uint32_t *Fin,
                                            uint32_t *Fout, uint64_t fc, uint64_t base,
                                            FlatShared<NT> &X, unsigned long long *next,
                                            ResidStage *stage, unsigned long long *hcount,
                                            uint64_t *hbuf, const uint32_t *lfin = nullptr,
                                            uint32_t *lfout = nullptr) {
    const uint32_t tid = threadIdx.x;
    // one wave's newly covered pairs: to the stage (when there is one) or
    // straight to Fout
    auto push = [&](bool add, uint32_t qw) {
        if (!stage) {
            const uint64_t slot = wave_reserve(next, add);
            if (add) {
                if (lfout && slot < kSkimLdsFront) lfout[slot] = qw;
                else st(Fout + slot, qw);
            }
            return;
        }
        const unsigned long long m = __ballot(add);
        if (!m) return;
        const int leader = __ffsll((long long)m) - 1;
        const uint32_t lane = lane_id();
        uint32_t pos0 = 0;
        if ((int)lane == leader) pos0 = atomicAdd(&stage->n, (uint32_t)__popcll(m));
        const uint32_t pos = (uint32_t)__shfl((int)pos0, leader) +
                             (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        if (!add) return;
        if (pos < 8 * kResidBlock) stage->buf[pos] = qw;
        else Fout[atomicAdd(next, 1ull)] = qw;  // stage full
    };
    auto flush = [&]() {
        if (!stage) return;
        __syncthreads();
        const uint32_t ns = stage->n < 8 * kResidBlock ? stage->n : 8 * kResidBlock;
        if (tid == 0 && ns) stage->base = atomicAdd(next, (unsigned long long)ns);
        __syncthreads();
        const unsigned long long b = stage->base;
        for (uint32_t j = tid; j < ns; j += NT) Fout[b + j] = stage->buf[j];
        __syncthreads();
        if (tid == 0) stage->n = 0;  // before the next chunk's first barrier
    };
    const uint64_t e = base + tid;
    uint32_t q = 0, o = 0, c = 0;
    uint64_t f0 = 0, deg = 0;
    if (e < fc) {
        q = lfin && e < kSkimLdsFront ? lfin[e] : Fin[e];
        const uint64_t ix = ld(A.idx + q);
        c = (uint32_t)ix;
        if (c) {
            o = (uint32_t)(ix >> 32);
            st(A.idx + q, (uint64_t)0);
        }
        f0 = A.fptr[q];
        deg = A.fptr[q + 1] - f0;
        if (hcount && deg > kSplitEdges) {  // deferred to the next level's launch
            const unsigned long long slot = atomicAdd(hcount, 1ull);
            if (slot < kHeavyItems) {
                hbuf[2 * slot] = ((uint64_t)q << 32) | (uint32_t)deg;
                hbuf[2 * slot + 1] = f0;
                deg = 0;
            }
        }
    }
    const bool light = __syncthreads_or(c > kSkimSerial || deg > kSkimSerial) == 0;
    if (light) {
        // each wave lays its 64 items' index entries, then their out-edges,
        // end to end and takes them 64 at a time
        const uint32_t lane = tid & 63u;
        if (!__any(c > kSkimFlat)) {  // short everywhere: each lane its own
            for (uint32_t j = 0; j < c; ++j) csub(SZ, ld(A.pool + o + j), 1u);
        } else {
            const uint32_t incl = wave_incl(c), total = (uint32_t)__shfl((int)incl, 63);
            for (uint32_t base = 0; base < total; base += 64) {
                const uint32_t j = base + lane, r = wave_owner(incl, j);
                const uint32_t first = (uint32_t)__shfl((int)incl, (int)r) -
                                       (uint32_t)__shfl((int)c, (int)r);
                const uint32_t ro = (uint32_t)__shfl((int)o, (int)r);
                if (j < total) csub(SZ, ld(A.pool + ro + (j - first)), 1u);
            }
        }
        const uint32_t d = (uint32_t)deg;  // <= kSkimSerial here
        if (!__any(d > kSkimFlat)) {  // short everywhere: each lane its own
            for (uint64_t x2 = f0; x2 < f0 + d; ++x2) {
                const uint32_t qw = A.fadj[x2] * kPairStride + q % kPairStride;
                const bool add = (!Precheck || !ld(A.covered + qw)) &&
                                 atomicCAS(A.covered + qw, 0u, 1u) == 0u;
                push(add, qw);
            }
            flush();
            return;
        }
        const uint32_t incl = wave_incl(d), total = (uint32_t)__shfl((int)incl, 63);
        for (uint32_t base = 0; base < total; base += 64) {
            const uint32_t j = base + lane, r = wave_owner(incl, j);
            const uint32_t first = (uint32_t)__shfl((int)incl, (int)r) -
                                   (uint32_t)__shfl((int)d, (int)r);
            const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)f0, (int)r);
            const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(f0 >> 32), (int)r);
            const uint32_t rq = (uint32_t)__shfl((int)q, (int)r);
            bool add = false;
            uint32_t qw = 0;
            if (j < total) {
                qw = A.fadj[(((uint64_t)hi << 32) | lo) + (j - first)] * kPairStride +
                     rq % kPairStride;
                add = (!Precheck || !ld(A.covered + qw)) &&
                      atomicCAS(A.covered + qw, 0u, 1u) == 0u;
            }
            push(add, qw);
        }
        flush();
        return;
    }
    uint64_t ctot, dtot;
    const uint64_t cex = block_excl_scan<NT>(c, X.wsum, ctot);
    const uint64_t dex = block_excl_scan<NT>(deg, X.wsum, dtot);
    X.ex2[tid] = cex;
    X.ex[tid] = dex;
    X.q[tid] = q;
    X.o[tid] = o;
    X.f0[tid] = f0;
    if (tid == 0) {
        X.ex2[NT] = ctot;
        X.ex[NT] = dtot;
    }
    __syncthreads();
    for (uint64_t t = tid; t < ctot; t += NT) {
        const uint32_t r = run_of<NT>(X.ex2, t);
        csub(SZ, ld(A.pool + X.o[r] + (t - X.ex2[r])), 1u);
    }
    for (uint64_t t = tid; t < dtot; t += NT) {
        const uint32_t r = run_of<NT>(X.ex, t);
        const uint32_t qw = A.fadj[X.f0[r] + (t - X.ex[r])] * kPairStride + X.q[r] % kPairStride;
        const bool add =
            (!Precheck || !ld(A.covered + qw)) && atomicCAS(A.covered + qw, 0u, 1u) == 0u;
        push(add, qw);
    }
    flush();
    __syncthreads();  // the chunk's LDS arrays are reused
}

// ------------------------------------------------------- searches ahead
// The reverse searches of the next pairs in rank order (the window: positions
// [a_lo, a_lo + a_w)), on the whole grid, before k_skim scans them.  A search
// does not depend on the seeds chosen meanwhile: an uncovered pair reaches no
// covered one, so it stays as it is until its pair is covered, and k_skim
// passes over covered pairs.  (Searched by k_skim's own threads as they were
// scanned, the 100 batches of 50 seeds on 10^6 nodes took 8 ms of one
// workgroup's time, a long chain of dependent loads in one lane each, and a
// seed that committed 75 pairs searched 1024.)
//
// Search r of the window is ahead[r] = first entry in apool << 32 | entries
// (0 entries: covered).  Three kernels: a lane per search up to kAheadShort
// nodes, then a wave per search up to kAheadWave nodes (queue and visited set
// in LDS), then a workgroup per search.  A search that no longer fits in the
// pool ends the window before its position.
constexpr uint32_t kAheadShort = 16;
constexpr uint32_t kAheadWave = 1024, kAheadHash = 4096;
constexpr uint32_t kAheadFirst = 1024, kAheadMax = 1u << 16;  // positions of a window
constexpr uint64_t kAheadEntries = 1ull << 20;  // entries a window is sized for
constexpr uint32_t kAheadPoolNodes = 512;       // the pool holds this many searches of n nodes
constexpr int kAheadBlock = 256, kAheadGiantBlock = 1024;
constexpr uint32_t kAheadGiants = 128;  // workgroups with a queue and a bitmap of their own

// The live in-list of pair q: node `one` (count 1, not stored), or a range.
struct InList {
    uint64_t begin;
    uint32_t count, one;
    bool stored;
};
__device__ __forceinline__ InList in_list(const SkArgs &A, uint32_t q) {
    if (!A.rlive) {
        const uint64_t e0 = A.rptr[q];
        return {e0, (uint32_t)(A.rptr[q + 1] - e0), 0u, true};
    }
    const uint64_t lw = A.rlive[q];
    if (lw & kLiveOne) return {0, 1u, (uint32_t)lw, false};
    return {lw >> kLiveCountBits, (uint32_t)(lw & ((1u << kLiveCountBits) - 1)), 0u, true};
}
__device__ __forceinline__ uint32_t in_node(const SkArgs &A, const InList &L, uint32_t j) {
    if (!L.stored) return L.one;
    return A.rlive ? A.rsrc[L.begin + j] : A.radj[L.begin + j];
}
__device__ __forceinline__ void ahead_fail(const SkArgs &A, uint32_t r) {
    A.ahead[r] = 0;
    atomicMin(&A.ctl->a_fail, (unsigned long long)r);
}

__global__ void __launch_bounds__(kAheadBlock) k_ahead_short(SkArgs A) {
    __shared__ uint32_t s_q[kAheadShort][kAheadBlock];
    const uint32_t tid = threadIdx.x;
    const uint64_t lo = A.ctl->a_lo;
    const uint32_t w = (uint32_t)min(A.ctl->a_w, (unsigned long long)(A.ordered - lo));
    for (uint32_t r0 = blockIdx.x * kAheadBlock; r0 < w; r0 += gridDim.x * kAheadBlock) {
        const uint32_t r = r0 + tid;
        uint32_t cnt = 0;
        bool more = false;
        if (r < w) {
            const uint32_t p = A.order[lo + r];
            if (!A.covered[p]) {
                const uint32_t i = p % kPairStride;
                s_q[0][tid] = p / kPairStride;
                cnt = 1;
                for (uint32_t head = 0; head < cnt && !more; ++head) {
                    const InList L = in_list(A, s_q[head][tid] * kPairStride + i);
                    for (uint32_t j = 0; j < L.count && !more; ++j) {
                        const uint32_t v = in_node(A, L, j);
                        bool seen = false;
                        for (uint32_t c = 0; c < cnt; ++c) seen |= s_q[c][tid] == v;
                        if (seen) continue;
                        if (cnt == kAheadShort) more = true;
                        else s_q[cnt++][tid] = v;
                    }
                }
            }
        }
        // a pair alone needs no pool entries
        const uint32_t take = more || cnt < 2 ? 0u : cnt;
        const uint32_t incl = wave_scan_sum(take);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        unsigned long long base = 0;
        if (total && (tid & 63u) == 0) base = atomicAdd(&A.ctl->a_used, (unsigned long long)total);
        base = ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(base >> 32)) << 32) |
               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base);
        base += incl - take;
        if (r < w && !more) {
            if (base + take > A.apool_cap) {
                if (take) ahead_fail(A, r);
                else A.ahead[r] = cnt;
            } else {
                A.ahead[r] = (base << 32) | cnt;
                for (uint32_t j = 0; j < take; ++j) A.apool[base + j] = s_q[j][tid];
            }
        }
        const uint64_t slot = wave_reserve(&A.ctl->nlong, more);
        if (more) A.along[slot] = r;
    }
}

constexpr uint32_t kAheadWaves = 4, kAheadWaveGrid = 1024;
__global__ void __launch_bounds__(64 * kAheadWaves) k_ahead_wave(SkArgs A) {
    __shared__ uint32_t s_hash[kAheadWaves][kAheadHash / 2], s_q[kAheadWaves][kAheadWave];
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    uint32_t *H = s_hash[wave], *Q = s_q[wave];
    constexpr uint32_t kSlots = kAheadHash / 2;
    const uint32_t nlong = (uint32_t)A.ctl->nlong;
    const uint64_t lo = A.ctl->a_lo;
    for (uint32_t x = blockIdx.x * kAheadWaves + wave; x < nlong; x += gridDim.x * kAheadWaves) {
        const uint32_t r = A.along[x], p = A.order[lo + r], i = p % kPairStride;
        for (uint32_t s = lane; s < kSlots; s += 64) H[s] = 0xFFFFFFFFu;
        __builtin_amdgcn_wave_barrier();
        // true when v was not in the set yet (at most kAheadWave + 64 nodes in
        // kSlots places)
        auto insert = [&](uint32_t v) {
            for (uint32_t s = (v * 0x9E3779B1u) >> 21;; s = (s + 1) & (kSlots - 1)) {
                const uint32_t was = atomicCAS(&H[s], 0xFFFFFFFFu, v);
                if (was == v) return false;
                if (was == 0xFFFFFFFFu) return true;
            }
        };
        static_assert(kSlots == 2048, "the hash takes 11 bits");
        if (lane == 0) {
            Q[0] = p / kPairStride;
            insert(Q[0]);
        }
        __builtin_amdgcn_wave_barrier();
        uint32_t cnt = 1;
        bool more = false;
        for (uint32_t head = 0; head < cnt && !more;) {
            const uint32_t take = min(64u, cnt - head);
            InList L = {0, 0, 0, true};
            if (lane < take) L = in_list(A, Q[head + lane] * kPairStride + i);
            head += take;
            // the lists end to end, 64 entries at a time
            const uint64_t big = __ballot(L.count >= (1u << 24));
            const uint32_t incl = wave_scan_sum(L.count);
            const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
            if (big) {  // (a prefix sum of longer lists could wrap)
                more = true;
                break;
            }
            for (uint32_t b = 0; b < total; b += 64) {
                const uint32_t j = b + lane, o = wave_owner(incl, j);
                InList M;
                M.count = 0;
                M.begin = ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(L.begin >> 32), (int)o) << 32) |
                          (uint32_t)__shfl((int)(uint32_t)L.begin, (int)o);
                M.one = (uint32_t)__shfl((int)L.one, (int)o);
                M.stored = __shfl((int)L.stored, (int)o) != 0;
                const uint32_t first = (uint32_t)__shfl((int)(incl - L.count), (int)o);
                bool add = false;
                uint32_t v = 0;
                if (j < total) {
                    v = in_node(A, M, j - first);
                    add = insert(v);
                }
                const uint64_t m = __ballot(add);
                const uint32_t pos = cnt + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                if (add && pos < kAheadWave) Q[pos] = v;
                cnt += (uint32_t)__popcll(m);
                if (cnt > kAheadWave) {
                    more = true;
                    break;
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
        if (more) {
            if (lane == 0) A.along[kAheadMax + atomicAdd(&A.ctl->ngiant, 1ull)] = r;
            continue;
        }
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd(&A.ctl->a_used, (unsigned long long)cnt);
        base = ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(base >> 32)) << 32) |
               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base);
        if (base + cnt > A.apool_cap) {
            if (lane == 0) ahead_fail(A, r);
            continue;
        }
        for (uint32_t j = lane; j < cnt; j += 64) A.apool[base + j] = Q[j];
        if (lane == 0) A.ahead[r] = (base << 32) | cnt;
    }
}

// Each workgroup searches in a queue and a visited bitmap of its own (kept
// zero), kAheadGiantBlock queue entries at a time, every wave over its 64
// entries' lists laid end to end.
__global__ void __launch_bounds__(kAheadGiantBlock) k_ahead_giant(SkArgs A) {
    __shared__ uint32_t s_tail;
    __shared__ unsigned long long s_base;
    const uint32_t tid = threadIdx.x, lane = tid & 63u;
    const uint32_t ngiant = (uint32_t)A.ctl->ngiant;
    const uint64_t lo = A.ctl->a_lo;
    uint32_t *Q = A.gqueue + (uint64_t)blockIdx.x * A.n;
    uint32_t *V = A.vis + (uint64_t)blockIdx.x * A.vis_words;
    for (uint32_t x = blockIdx.x; x < ngiant; x += gridDim.x) {
        const uint32_t r = A.along[kAheadMax + x], p = A.order[lo + r], i = p % kPairStride;
        if (tid == 0) {
            const uint32_t v = p / kPairStride;
            st(Q, v);
            atomicOr(V + (v >> 5), 1u << (v & 31u));
            s_tail = 1;
        }
        __syncthreads();
        for (uint32_t head = 0;;) {
            const uint32_t tail = s_tail;
            __syncthreads();
            if (head >= tail) break;  // uniform
            const uint32_t take = min((uint32_t)kAheadGiantBlock, tail - head);
            InList L = {0, 0, 0, true};
            if (tid < take) L = in_list(A, ld(Q + head + tid) * kPairStride + i);
            head += take;
            uint32_t at = 0;  // entries of this lane's list laid out so far
            while (__any(at < L.count)) {
                // at most 2^16 of each list at a time: their sum does not wrap
                const uint32_t part = min(L.count - at, 1u << 16);
                const uint32_t incl = wave_scan_sum(part);
                const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                for (uint32_t b = 0; b < total; b += 64) {
                    const uint32_t j = b + lane, o = wave_owner(incl, j);
                    InList M;
                    M.count = 0;
                    const uint64_t from = L.begin + at;
                    M.begin = ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(from >> 32), (int)o) << 32) |
                              (uint32_t)__shfl((int)(uint32_t)from, (int)o);
                    M.one = (uint32_t)__shfl((int)L.one, (int)o);
                    M.stored = __shfl((int)L.stored, (int)o) != 0;
                    const uint32_t first = (uint32_t)__shfl((int)(incl - part), (int)o);
                    bool add = false;
                    uint32_t v = 0;
                    if (j < total) {
                        v = in_node(A, M, j - first);
                        const uint32_t bit = 1u << (v & 31u);
                        add = !(ld(V + (v >> 5)) & bit) && !(atomicOr(V + (v >> 5), bit) & bit);
                    }
                    const uint64_t m = __ballot(add);
                    if (m) {
                        uint32_t pos = 0;
                        if (lane == (uint32_t)__ffsll((long long)m) - 1u)
                            pos = atomicAdd(&s_tail, (uint32_t)__popcll(m));
                        pos = (uint32_t)__shfl((int)pos, __ffsll((long long)m) - 1) +
                              (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                        if (add) st(Q + pos, v);  // each node once: at most n
                    }
                }
                at += part;
            }
            __syncthreads();
        }
        const uint32_t cnt = s_tail;
        if (tid == 0) s_base = atomicAdd(&A.ctl->a_used, (unsigned long long)cnt);
        __syncthreads();
        const unsigned long long base = s_base;
        const bool fits = base + cnt <= A.apool_cap;
        for (uint32_t j = tid; j < cnt; j += kAheadGiantBlock) {
            const uint32_t v = ld(Q + j);
            st(V + (v >> 5), 0u);
            if (fits) A.apool[base + j] = v;
        }
        if (tid == 0) {
            if (fits) A.ahead[r] = (base << 32) | cnt;
            else ahead_fail(A, r);
        }
        __syncthreads();  // the queue, the bitmap and s_tail are reused
    }
}

// The selection loop.  kLds: size[] is in LDS (graphs of at most
// kSkimLdsNodes nodes: every search adds to it, and device atomics from
// different waves on one cache line are serialised).
template <bool kLds>
__global__ void __launch_bounds__(kSkimBlock) k_skim(SkArgs A, uint32_t goal, uint64_t handoff,
                                                     uint32_t *seeds, uint64_t *gains,
                                                     double *gain_d, uint64_t *rec_tau,
                                                     uint32_t *rec_second) {
    __shared__ unsigned long long s_cursor, s_pool, s_gain, s_best, s_tau, s_fcnt[2];
    __shared__ int s_x;
    __shared__ uint32_t s_stop, s_second, s_xmin, s_resume, s_rcur;
    __shared__ unsigned long long s_fill0, s_fill1;
    __shared__ __align__(16) uint32_t s_size[kLds ? kSkimLdsWords : 4];
    __shared__ FlatShared<kSkimBlock> X;
    __shared__ ScanShared C;
    __shared__ uint32_t s_front[2][kSkimLdsFront];
    const uint32_t tid = threadIdx.x;
    const uint32_t n = A.n, k = A.k;
    uint32_t *SZ = kLds ? s_size : A.size;
    const uint32_t swords = size_words(n);
    if constexpr (kLds)
        for (uint32_t w = tid; w < swords; w += kSkimBlock) s_size[w] = ld(A.size + w);
    const uint64_t a_lo = A.ctl->a_lo;
    const uint64_t a_hi = min((unsigned long long)A.ordered,
                              a_lo + min(A.ctl->a_w, A.ctl->a_fail));
    if (tid == 0) {
        s_cursor = A.ctl->cursor;
        s_pool = A.ctl->pool_used;
        s_stop = 0;
        C.ncand = 0;
        // a residual search the grid handed back (its frontier got small):
        // the launch starts by finishing that seed
        s_resume = A.ctl->pend == 2;
        if (s_resume) {
            A.ctl->pend = 0;
            s_x = (int)A.ctl->px;
            s_rcur = A.ctl->rcur;
            s_gain = A.ctl->rgain;
            s_fcnt[s_rcur] = A.ctl->rsize[0];
        }
    }
    __syncthreads();
    // Entry t of the batch's searches, laid end to end in thread order:
    // staged in LDS when there is room for all of them.
    bool staged = true;
    auto far_entry = [&](uint64_t t) {
        const uint32_t r = run_of<kSkimBlock>(X.ex, t);
        const uint32_t j = (uint32_t)(t - X.ex[r]);
        return j ? A.apool[(uint64_t)X.o[r] + j] : X.q[r];
    };
    auto entry = [&](uint64_t t) { return staged ? C.entry[t] : far_entry(t); };
    uint32_t done = 0;
    for (uint32_t it = 0; it < goal; ++it) {
        const bool resumed = it == 0 && s_resume;  // uniform
        if (!resumed) {
        if (tid == 0) {
            s_x = -1;
            s_fill0 = s_fill1 = 0;
        }
        __syncthreads();
        // ------------------------------------------------ scan pairs by rank
        while (s_x < 0 && s_cursor < A.nsrc) {
            const uint64_t cursor = s_cursor;
            if (cursor >= a_hi) {  // the window is used up: the host has the next one searched
                if (tid == 0) {
                    s_stop = 1;
                    const uint64_t w = A.ctl->a_w, used = A.ctl->a_used;
                    // four times as long, if that is about kAheadEntries
                    // entries; a window that outgrew the pool, a quarter
                    uint64_t next = min(4 * w, w * kAheadEntries / (used ? used : 1));
                    next = min(max(next, (uint64_t)kAheadFirst), (uint64_t)kAheadMax);
                    if (A.ctl->a_fail < w) next = (w + 3) / 4;
                    A.ctl->a_lo = cursor;
                    A.ctl->a_w = next;
                    A.ctl->a_fail = ~0ull;
                    A.ctl->a_used = A.ctl->nlong = A.ctl->ngiant = 0;
                    A.ctl->flags |= kFlagAhead;
                }
                __syncthreads();
                break;
            }
            // sizes are below k here and grow by at most one per pair: they
            // stay in 16 bits with all of a batch added
            const uint32_t B = (uint32_t)min(a_hi - cursor,
                                             (uint64_t)min((uint32_t)kSkimBlock, 65536u - k));
            uint32_t cnt = 0, p = 0, first = 0;
            if (tid < B) {
                p = A.order[cursor + tid];
                const uint64_t a = A.ahead[cursor - a_lo + tid];
                if (!ld(A.covered + p)) {
                    cnt = (uint32_t)a;
                    first = (uint32_t)(a >> 32);
                }
            }
            uint64_t tot;
            const uint64_t ex = block_excl_scan<kSkimBlock>(cnt, X.wsum, tot);
            X.ex[tid] = ex;
            X.q[tid] = p / kPairStride;
            X.o[tid] = first;
            if (tid == 0) {
                X.ex[kSkimBlock] = tot;
                s_xmin = 0xFFFFFFFFu;
            }
            staged = tot <= kSkimStage;
            if (staged) {
                if (__syncthreads_or(cnt > kSkimSerial)) {
                    for (uint64_t t = tid; t < tot; t += kSkimBlock) C.entry[t] = far_entry(t);
                } else if (cnt) {
                    C.entry[ex] = p / kPairStride;
                    for (uint32_t j = 1; j < cnt; ++j)
                        C.entry[ex + j] = A.apool[(uint64_t)first + j];
                }
            }
            __syncthreads();
            // All of the batch is added to the sizes.  If some node reaches k
            // the entries of all that did are kept, and the first filling
            // prefix is the smallest position at which one of them receives
            // its k-th (a search holds a node at most once); with too many
            // such entries it is found by binary search over prefixes.  The
            // pairs after that prefix are then taken back.
            bool f = false;
            for (uint64_t t = tid; t < tot; t += kSkimBlock)
                f |= cadd_old(SZ, entry(t), 1u) + 1 >= k;
            const bool filled = __syncthreads_or(f) != 0;
            uint32_t T = B;
            if (filled) {
                for (uint64_t t = tid; t < tot; t += kSkimBlock) {
                    const uint32_t v = entry(t);
                    if (cget(SZ, v) < k) continue;
                    const uint32_t slot = atomicAdd(&C.ncand, 1u);
                    if (slot < kSkimCand) {
                        C.cand[slot] = ((uint64_t)run_of<kSkimBlock>(X.ex, t) << 32) | v;
                        C.seen[slot] = 0;
                    }
                }
                __syncthreads();
                // moves the sizes from prefix `from` of the batch to prefix `to`
                auto move = [&](uint32_t from, uint32_t to) {
                    for (uint64_t t = X.ex[min(from, to)] + tid; t < X.ex[max(from, to)];
                         t += kSkimBlock) {
                        if (from < to) cadd(SZ, entry(t), 1u);
                        else csub(SZ, entry(t), 1u);
                    }
                    __syncthreads();
                };
                const uint32_t nc = C.ncand;
                uint32_t at = B;
                if (nc <= kSkimCand) {
                    // per candidate: entries of its node in the batch (high
                    // half) and those at earlier positions, the other
                    // candidates dealt over the block's threads
                    const uint32_t parts = kSkimBlock / nc, c = tid % nc, part = tid / nc;
                    if (part < parts) {
                        const uint64_t e = C.cand[c];
                        uint32_t seen = 0;
                        for (uint32_t c2 = part; c2 < nc; c2 += parts) {
                            const uint64_t e2 = C.cand[c2];
                            if ((uint32_t)e2 == (uint32_t)e) seen += e2 < e ? 0x10001u : 0x10000u;
                        }
                        if (seen) atomicAdd(&C.seen[c], seen);
                    }
                    __syncthreads();
                    for (uint32_t c = tid; c < nc; c += kSkimBlock) {
                        const uint64_t e = C.cand[c];
                        const uint32_t seen = C.seen[c];
                        if (cget(SZ, (uint32_t)e) - (seen >> 16) + (seen & 0xFFFFu) + 1 == k)
                            atomicMin(&s_xmin, (uint32_t)(e >> 32));
                    }
                    __syncthreads();
                    T = s_xmin + 1;
                } else {
                    uint32_t none = 0;  // prefixes none and T: nothing fills, something does
                    while (T - none > 1) {
                        const uint32_t mid = none + (T - none) / 2;
                        move(at, mid);
                        at = mid;
                        bool g = false;
                        for (uint64_t t = tid; t < X.ex[mid]; t += kSkimBlock)
                            g |= cget(SZ, entry(t)) >= k;
                        if (__syncthreads_or(g)) T = mid;
                        else none = mid;
                    }
                }
                move(at, T);
                if (tid == 0) s_xmin = 0xFFFFFFFFu;
            }
            // does the committed prefix fit in the index pool?
            const uint64_t need = X.ex[T], pbase = s_pool;
            if (pbase + need > A.pool_cap) {
                for (uint64_t t = tid; t < need; t += kSkimBlock) csub(SZ, entry(t), 1u);
                if (tid == 0) {
                    A.ctl->flags |= kFlagPool;
                    A.ctl->need = pbase + need;
                    s_stop = 1;
                    C.ncand = 0;
                }
                __syncthreads();
                break;
            }
            // commit pairs [0, T): index entries in pair order
            for (uint64_t t = tid; t < need; t += kSkimBlock) st(A.pool + pbase + t, entry(t));
            if (tid < T && cnt) st(A.idx + p, ((pbase + ex) << 32) | cnt);
            if (filled) {
                // the nodes that just reached k are in pair T - 1's search;
                // the seed is the smallest of them
                __syncthreads();
                for (uint64_t t = X.ex[T - 1] + tid; t < need; t += kSkimBlock) {
                    const uint32_t v = entry(t);
                    if (cget(SZ, v) >= k) atomicMin(&s_xmin, v);
                }
                if (tid == T - 1) s_tau = pair_rank(A.seed, p);
                __syncthreads();
            }
            if (tid == 0) {
                if (filled) {
                    s_x = s_xmin == 0xFFFFFFFFu ? -1 : (int)s_xmin;
                    s_fill0 = X.ex[T - 1];
                    s_fill1 = need;
                }
                s_cursor = cursor + T;
                s_pool = pbase + need;
                C.ncand = 0;
            }
            __syncthreads();
        }
        if (s_stop) break;
        // --------------------------------------------------- exhaustion rule
        if (s_x < 0) {
            if (tid == 0) s_best = 0;
            __syncthreads();
            unsigned long long best = 0;
            for (uint32_t v = tid; v < n; v += kSkimBlock)
                if (!ld(A.sel + v)) {
                    const unsigned long long key =
                        ((unsigned long long)cget(SZ, v) << 32) | (0xFFFFFFFFu - v);
                    best = key > best ? key : best;
                }
            atomicMax(&s_best, best);
            __syncthreads();
            // an unselected node always exists (the host checks s); keep the
            // index in range regardless
            if (tid == 0) {
                const uint32_t v = 0xFFFFFFFFu - (uint32_t)s_best;
                s_x = (s_best && v < n) ? (int)v : 0;
            }
            __syncthreads();
        }
        const uint32_t xs = (uint32_t)s_x;  // the seed
        // ------------------------------------ records for the error estimate
        // The filling pair's search is still the batch's; its nodes' sizes
        // are one less, and the seed's is 0, while the sizes are scanned.
        // Selected nodes need no test: every pair a seed reaches is covered,
        // so its size is 0 from then on and no later search reaches it.
        const uint64_t fill0 = s_fill0, fill1 = s_fill1;
        for (uint64_t t = fill0 + tid; t < fill1; t += kSkimBlock) {
            const uint32_t v = entry(t);
            if (v != xs) csub(SZ, v, 1u);
        }
        uint32_t xsize = 0;
        if (tid == 0) {
            s_second = 0;
            xsize = cget(SZ, xs);
            csub(SZ, xs, xsize);
        }
        // (the atomics above have reached the L2 before the barrier; the
        // fence after it drops this CU's cached copies of the sizes)
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if constexpr (!kLds) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        {
            // eight sizes per load, eight loads in flight: one workgroup reads
            // the 2 MB of 10^6 nodes
            typedef unsigned short us2 __attribute__((ext_vector_type(2)));
            us2 best2 = {0, 0};
            auto upto = [&](uint32_t w) {
                best2 = __builtin_elementwise_max(best2, __builtin_bit_cast(us2, w));
            };
            const uint4 *SZ4 = reinterpret_cast<const uint4 *>(SZ);
            const uint32_t nw = swords / 4;
            for (uint32_t w0 = tid; w0 < nw; w0 += 8 * kSkimBlock) {
                uint4 a[8];
#pragma unroll
                for (uint32_t u = 0; u < 8; ++u) {
                    const uint32_t w = w0 + u * kSkimBlock;
                    a[u] = w < nw ? SZ4[w] : uint4{0, 0, 0, 0};
                }
#pragma unroll
                for (uint32_t u = 0; u < 8; ++u) upto(a[u].x), upto(a[u].y), upto(a[u].z), upto(a[u].w);
            }
            // one LDS atomic per wave: lanes on one address are serialised
            uint32_t b = max((uint32_t)best2.x, (uint32_t)best2.y);
            b = 0xFFFFFFFFu - group_min_u32<64>(0xFFFFFFFFu - b);
            if ((tid & 63) == 0 && b) atomicMax(&s_second, b);
        }
        __syncthreads();
        for (uint64_t t = fill0 + tid; t < fill1; t += kSkimBlock) {
            const uint32_t v = entry(t);
            if (v != xs) cadd(SZ, v, 1u);
        }
        if (tid == 0) {
            cadd(SZ, xs, xsize);
            rec_tau[it] = fill1 ? (uint64_t)s_tau : ~0ull;
            rec_second[it] = s_second;
        }
        }  // !resumed
        const uint32_t x = (uint32_t)s_x;
        // ------------------------------------------------- residual problem
        // Level-synchronous over all instances at once: a frontier of pairs
        // (64 v + i) in two halves of the queue area.  A pair is
        // claimed by the CAS that covers it; its index entry is erased then.
        // A level with more than `handoff` pairs (0: none) and the rest of
        // the search go to the whole grid (k_resid_level); the host then
        // completes the seed.
        uint32_t *F[2] = {A.front, A.front + (uint64_t)A.n * kPairStride};
        if (!resumed) {
        if (tid == 0) {
            s_gain = 0;
            s_fcnt[0] = 0;
        }
        __syncthreads();
        {
            bool add = false;
            uint32_t px = 0;
            if (tid < A.ell) {
                px = x * kPairStride + tid;
                add = atomicCAS(A.covered + px, 0u, 1u) == 0u;
            }
            if (tid < 64) {  // the first wave holds every instance (l <= 64)
                const uint64_t slot = wave_reserve(&s_fcnt[0], add);
                if (add) s_front[0][slot] = px;
            }
        }
        } else {
            // the grid left the pending level in the queue area
            const uint64_t fc = s_fcnt[s_rcur];
            for (uint32_t e = tid; e < fc && e < kSkimLdsFront; e += kSkimBlock)
                s_front[s_rcur][e] = F[s_rcur][e];
        }
        bool handed = false;
        const uint64_t seed_edges = A.fptr[(uint64_t)x * kPairStride + kPairStride] -
                                    A.fptr[(uint64_t)x * kPairStride];
        // a resumed search continues at its pending level (not level 0)
        for (uint32_t cur = resumed ? s_rcur : 0u, level = resumed ? 1u : 0u;;
             cur ^= 1u, ++level) {
            __syncthreads();
            // (the counter reset below is of the next level's counter, read
            // by nobody in this level)
            const uint64_t fc = s_fcnt[cur];
            if (fc == 0) break;
            if (handoff && (fc > handoff || (level == 0 && seed_edges > kSkimHandoffEdges))) {
                // the grid reads the level from the queue area
                for (uint32_t e = tid; e < fc && e < kSkimLdsFront; e += kSkimBlock)
                    st(F[cur] + e, s_front[cur][e]);
                if (tid == 0) {
                    A.ctl->pend = 1;
                    A.ctl->px = x;
                    A.ctl->rcur = cur;
                    A.ctl->rsize[0] = fc;
                    A.ctl->rsize[16] = 0;
                    A.ctl->rsize[32] = 0;
                    A.ctl->hsize[0] = A.ctl->hsize[16] = A.ctl->hsize[32] = 0;
                    A.ctl->rgain = s_gain;
                }
                handed = true;
                break;
            }
            if (tid == 0) {
                s_fcnt[cur ^ 1u] = 0;
                s_gain += fc;
            }
            for (uint64_t base = 0; base < fc; base += kSkimBlock)
                resid_chunk<kSkimBlock, false>(A, SZ, F[cur], F[cur ^ 1u], fc, base, X,
                                               &s_fcnt[cur ^ 1u], nullptr, nullptr, nullptr,
                                               s_front[cur], s_front[cur ^ 1u]);
        }
        if (handed) break;  // uniform
        __syncthreads();
        if (tid == 0) {
            st(A.sel + x, 1u);
            seeds[it] = x;
            gains[it] = s_gain;
            if (gain_d) gain_d[it] = (double)s_gain / (double)A.ell;
        }
        ++done;
        __syncthreads();
    }
    if constexpr (kLds) {
        __syncthreads();
        for (uint32_t w = tid; w < swords; w += kSkimBlock) st(A.size + w, s_size[w]);
    }
    if (tid == 0) {
        A.ctl->cursor = s_cursor;
        A.ctl->pool_used = s_pool;
        A.ctl->done = done;
    }
}

// Level L of a residual search handed over by k_skim, on the whole grid:
// frontier buffer (r0 + L) & 1 of the queue area, sizes in global memory.
// First the pairs level L - 1 deferred (long out-lists), their edges laid end
// to end and split evenly over every workgroup, kResidBlock pairs at a time;
// then the level's own frontier.  Both append to level L + 1.  A launch with
// nothing to do returns at once, so the host launches levels in batches and
// reads the sizes back after each batch.
__global__ void __launch_bounds__(kResidBlock) k_resid_level(SkArgs A, uint32_t L, uint32_t r0) {
    __shared__ FlatShared<kResidBlock> X;
    __shared__ ResidStage S;
    __shared__ unsigned long long s_fc, s_nh;
    const uint32_t tid = threadIdx.x;
    if (tid == 0) {
        S.n = 0;
        s_fc = ld(&A.ctl->rsize[16 * (L % 3)]);
        s_nh = ld(&A.ctl->hsize[16 * ((L + 2) % 3)]);  // deferred by level L - 1
        if (blockIdx.x == 0) {
            A.ctl->rsize[16 * ((L + 2) % 3)] = 0;  // level L + 1 appends there
            A.ctl->hsize[16 * ((L + 1) % 3)] = 0;  // and defers there
            A.ctl->rgain += s_fc;
        }
    }
    __syncthreads();
    const uint64_t fc = s_fc;
    const uint32_t nh = s_nh < kHeavyItems ? (uint32_t)s_nh : kHeavyItems;
    if (fc == 0 && nh == 0) return;  // uniform
    const uint32_t cur = (r0 + L) & 1u;
    const uint64_t half = (uint64_t)A.n * kPairStride;
    const uint32_t *Fin = A.front + cur * half;
    uint32_t *Fout = A.front + (cur ^ 1u) * half;
    unsigned long long *next = &A.ctl->rsize[16 * ((L + 1) % 3)];
    const uint64_t *hin = A.heavy + 2 * (uint64_t)kHeavyItems * ((L + 2) % 3);
    for (uint32_t h0 = 0; h0 < nh; h0 += kResidBlock) {
        uint64_t deg = 0, f0 = 0;
        uint32_t q = 0;
        if (h0 + tid < nh) {
            const uint64_t w = hin[2 * (h0 + tid)];
            q = (uint32_t)(w >> 32);
            deg = (uint32_t)w;
            f0 = hin[2 * (h0 + tid) + 1];
        }
        uint64_t tot;
        const uint64_t e = block_excl_scan<kResidBlock>(deg, X.wsum, tot);
        X.ex[tid] = e;
        X.q[tid] = q;
        X.f0[tid] = f0;
        if (tid == 0) X.ex[kResidBlock] = tot;
        __syncthreads();
        const uint64_t a = tot * blockIdx.x / gridDim.x, b = tot * (blockIdx.x + 1) / gridDim.x;
        for (uint64_t base = a; base < b; base += kResidBlock) {
            const uint64_t t = base + tid;
            bool add = false;
            uint32_t qw = 0;
            if (t < b) {
                const uint32_t r = run_of<kResidBlock>(X.ex, t);
                qw = A.fadj[X.f0[r] + (t - X.ex[r])] * kPairStride + X.q[r] % kPairStride;
                add = !ld(A.covered + qw) && atomicCAS(A.covered + qw, 0u, 1u) == 0u;
            }
            const unsigned long long m = __ballot(add);
            if (m) {
                const int leader = __ffsll((long long)m) - 1;
                const uint32_t lane = lane_id();
                uint32_t pos0 = 0;
                if ((int)lane == leader) pos0 = atomicAdd(&S.n, (uint32_t)__popcll(m));
                const uint32_t pos = (uint32_t)__shfl((int)pos0, leader) +
                                     (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                if (add) {
                    if (pos < 8 * kResidBlock) S.buf[pos] = qw;
                    else Fout[atomicAdd(next, 1ull)] = qw;
                }
            }
            __syncthreads();
            const uint32_t ns = S.n < 8 * kResidBlock ? S.n : 8 * kResidBlock;
            __syncthreads();  // every thread has read S.n: the test below is uniform
            if (ns > 7 * kResidBlock || base + kResidBlock >= b) {
                if (tid == 0 && ns) S.base = atomicAdd(next, (unsigned long long)ns);
                __syncthreads();
                for (uint32_t j = tid; j < ns; j += kResidBlock) Fout[S.base + j] = S.buf[j];
                __syncthreads();
                if (tid == 0) S.n = 0;
                __syncthreads();
            }
        }
        __syncthreads();  // X is reused
    }
    uint64_t *hout = A.heavy + 2 * (uint64_t)kHeavyItems * (L % 3);
    for (uint64_t base = (uint64_t)blockIdx.x * kResidBlock; base < fc;
         base += (uint64_t)gridDim.x * kResidBlock)
        resid_chunk<kResidBlock, true>(A, A.size, Fin, Fout, fc, base, X, next, &S,
                                       &A.ctl->hsize[16 * (L % 3)], hout);
}

// The handed-over search's next level (L) is small: k_skim finishes it.
__global__ void k_resid_handback(SkArgs A, uint32_t L, uint32_t r0) {
    A.ctl->rsize[0] = A.ctl->rsize[16 * (L % 3)];
    A.ctl->rcur = (r0 + L) & 1u;
    A.ctl->pend = 2;
}

// The handed-over seed is complete: outputs, and the node leaves the
// candidates.
__global__ void k_resid_finish(SkArgs A, uint32_t *seeds, uint64_t *gains, double *gain_d) {
    const uint32_t x = A.ctl->px;
    const unsigned long long g = A.ctl->rgain;
    A.sel[x] = 1u;
    seeds[0] = x;
    gains[0] = g;
    if (gain_d) gain_d[0] = (double)g / (double)A.ell;
    A.ctl->pend = 0;
}

__global__ void k_pair_keys(uint32_t n, uint32_t ell, uint64_t seed, uint64_t *keys,
                            uint32_t *vals) {
    const uint64_t total = (uint64_t)n * ell;
    for (uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; t < total;
         t += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t p = (uint32_t)(t / ell) * kPairStride + (uint32_t)(t % ell);
        keys[t] = pair_rank(seed, p);
        vals[t] = p;
    }
}

// A run uses the lowest ranks only (50 seeds on 10^6 nodes: 74 thousand of 64
// million), so past kOrderWhole pairs the order is made in steps, kOrderFirst
// pairs first and four times as many in each later step: the pairs with ranks
// in [r0, r1] are counted, collected in any order and sorted, which continues
// the order exactly (ranks are distinct: they are one SplitMix64 sequence).
// Ranks are uniform, so a step is about as long as aimed at.  10^6 nodes,
// l = 64: all ranks 2.8 ms, the first step 0.3 ms.
constexpr uint64_t kOrderFirst = 1ull << 18, kOrderWhole = 1ull << 20;
constexpr int kOrderBlock = 256;
constexpr uint32_t kOrderGrid = 2048;
__global__ void __launch_bounds__(kOrderBlock) k_rank_count(uint32_t n, uint32_t ell, uint64_t seed,
                                                            uint64_t r0, uint64_t r1,
                                                            uint32_t *counts,
                                                            unsigned long long *total) {
    __shared__ uint32_t s_count;
    if (threadIdx.x == 0) s_count = 0;
    __syncthreads();
    uint32_t c = 0;
    for (uint64_t p = blockIdx.x * (uint64_t)kOrderBlock + threadIdx.x; p < (uint64_t)n * kPairStride;
         p += (uint64_t)gridDim.x * kOrderBlock) {
        const uint64_t r = pair_rank(seed, (uint32_t)p);
        c += p % kPairStride < ell && r >= r0 && r <= r1;
    }
    atomicAdd(&s_count, c);
    __syncthreads();
    if (threadIdx.x == 0) {
        counts[blockIdx.x] = s_count;
        atomicAdd(total, (unsigned long long)s_count);
    }
}
__global__ void __launch_bounds__(kOrderBlock) k_rank_take(uint32_t n, uint32_t ell, uint64_t seed,
                                                           uint64_t r0, uint64_t r1,
                                                           const uint32_t *counts,
                                                           unsigned long long *taken,
                                                           uint64_t *keys, uint32_t *vals) {
    __shared__ unsigned long long s_base;
    __shared__ uint32_t s_at;
    if (threadIdx.x == 0) {
        s_base = atomicAdd(taken, (unsigned long long)counts[blockIdx.x]);
        s_at = 0;
    }
    __syncthreads();
    for (uint64_t p = blockIdx.x * (uint64_t)kOrderBlock + threadIdx.x; p < (uint64_t)n * kPairStride;
         p += (uint64_t)gridDim.x * kOrderBlock) {
        const uint64_t r = pair_rank(seed, (uint32_t)p);
        if (p % kPairStride < ell && r >= r0 && r <= r1) {
            const uint64_t slot = s_base + atomicAdd(&s_at, 1u);
            keys[slot] = r;
            vals[slot] = (uint32_t)p;
        }
    }
}

// The pairs are radix-sorted on the high halves of their ranks only (four
// passes instead of eight).  Equal high halves are rare (about (n l)^2 / 2^33
// pairs of pairs for uniform ranks); the thread at the start of each such run
// puts it in full-rank order by a stable insertion sort, which gives exactly
// the order of a full sort (by rank, then by pair as listed).  Within a run
// the high halves are all equal, so the other threads' run tests read the
// same values whatever the owners are moving.
constexpr uint64_t kHalfSortPairs = 1ull << 21;
__global__ void k_rank_ties(uint64_t *keys, uint32_t *vals, uint64_t count) {
    for (uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; t + 1 < count;
         t += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t hi = (uint32_t)(keys[t] >> 32);
        if ((uint32_t)(keys[t + 1] >> 32) != hi) continue;   // no tie follows
        if (t > 0 && (uint32_t)(keys[t - 1] >> 32) == hi) continue;  // not the run's start
        uint64_t e = t + 2;
        while (e < count && (uint32_t)(keys[e] >> 32) == hi) ++e;
        for (uint64_t i = t + 1; i < e; ++i) {
            const uint64_t key = keys[i];
            const uint32_t val = vals[i];
            uint64_t j = i;
            for (; j > t && keys[j - 1] > key; --j) {
                keys[j] = keys[j - 1];
                vals[j] = vals[j - 1];
            }
            keys[j] = key;
            vals[j] = val;
        }
    }
}

// ------------------------------------------------ adaptive error estimate
// Section 4 (adaptive error estimation), eq. (chernoff).  Discrepancies are
// counted on a grid of step h = max_rel_error * I / bins pairs, I the sum of
// the gains; every distribution is held as its survival function
// S[j] = P[D >= j h], j = 0..bins, with everything at or beyond bins * h kept
// in the last cell.

constexpr uint32_t kTailMaxBins = 1u << 16;
constexpr uint64_t kTailMaxCells = 1ull << 30;  // seeds * (bins + 1)
constexpr int kTailBlock = 256;

constexpr uint32_t kTailCounters = 1024;  // arrival counters, cleared at the start of a tail
__global__ void __launch_bounds__(kTailBlock) k_tail_total(uint32_t s, const uint64_t *gain,
                                                           uint64_t *total, uint32_t *arrived) {
    __shared__ unsigned long long acc;
    if (threadIdx.x == 0) acc = 0;
    for (uint32_t c = threadIdx.x; c < kTailCounters; c += kTailBlock) arrived[c] = 0;
    __syncthreads();
    unsigned long long t = 0;
    for (uint32_t r = threadIdx.x; r < s; r += kTailBlock) t += gain[r];
    atomicAdd(&acc, t);
    __syncthreads();
    if (threadIdx.x == 0) *total = acc;
}

// eq. (chernoff) with Z = z and nu = 1 - z / mu, in logarithms:
// (e^-nu / (1 - nu)^(1 - nu))^mu = exp(z - mu + z ln(mu / z)); 1 when z >= mu.
__device__ __forceinline__ double chernoff_bound(double mu, double z) {
    if (z >= mu) return 1.0;
    if (z == 0.0) return exp(-mu);
    return exp(z - mu + z * log(mu / z));
}

// S_r[j] >= P[D_r > (j-1) h] for record r: a seed whose sketch filled at rank
// tau with second largest sketch k' and gain Delta has
// P[D > eps Delta] <= bound(mu = rho(tau) Delta (1 + eps), k').  An exhaustion
// seed (tau = all ones) is exact (D = 0); a filled record with no gain gives
// no bound (S = 1).
__global__ void __launch_bounds__(kTailBlock) k_tail_survival(
    uint32_t s, const uint64_t *tau, const uint32_t *second, const uint64_t *gain,
    const uint64_t *total, uint32_t bins, double max_rel, double *S) {
    const uint64_t W = (uint64_t)bins + 1, work = (uint64_t)s * W;
    const uint64_t I = *total;
    const double h = max_rel * (double)I / (double)bins;
    for (uint64_t t = blockIdx.x * (uint64_t)kTailBlock + threadIdx.x; t < work;
         t += (uint64_t)gridDim.x * kTailBlock) {
        const uint64_t r = t / W;
        const uint32_t j = (uint32_t)(t - r * W);
        double v;
        if (j == 0) {
            v = 1.0;
        } else if (I == 0 || tau[r] == ~0ull) {
            v = 0.0;
        } else if (gain[r] == 0) {
            v = 1.0;
        } else {
            const double d = (double)gain[r];
            const double rho = (double)((tau[r] >> 11) + 1) * 0x1p-53;
            const double eps = (double)(j - 1) * h / d;
            const double mu = rho * d * (1.0 + eps);
            v = fmin(1.0, chernoff_bound(mu, (double)second[r]));
        }
        S[t] = v;
    }
}

// One level of the pairwise tree: out[p] = the capped sum of rows 2p and
// 2p+1 of in (an odd last row is copied).  With a[i] = Sa[i] - Sa[i+1],
//   Sc[j] = P[A + B >= j] = Sa[j+1] + sum_{i <= j} a[i] Sb[j-i],  Sa[bins+1] = 0.
// The convolution on the fp64 matrix cores: with j = 16 c + r and
// i = 16 b + t it is a sum over D = c - b of 16 x 16 x 16 products,
//   out[r][c] = sum_D sum_t T_D[r][t] a[16 (c - D) + t],
//   T_D[r][t] = Sb[16 D + r - t]  (zero outside 0 .. bins),
// so a tile of 16 columns (256 outputs) takes four 16x16x4 products per D
// = 0 .. its last column, all of them needed but for the triangles at both
// ends.  A workgroup's four waves split the D range 8 steps at a time and
// share the staged values; their sums are added in a fixed order.
//
// The last levels have few tiles and long D ranges (one pair: 17 tiles of up
// to 272 steps at 4097 cells), a serial chain on a few CUs.  There a tile's D
// range is cut into parts of `part` steps, one workgroup each; the parts' sums
// go to scratch and the workgroup that finishes last adds them in order.  The
// result does not depend on which one that is.
//
// 200 seeds, 4096 bins (3.34 GFLOP, 55 us at the 61 TFLOP/s that a large fp64
// matrix product reaches here): vector units, 8 waves per 256 outputs, 0.58 ms;
// this 0.18 ms (the first level 53 us, the last three 8 us each).
constexpr int kTailTile = 256, kTailChunk = 32, kTailWaves = 4;
constexpr int kTailPairBlock = 64 * kTailWaves;
constexpr int kTailBlocks = kTailChunk + 15;       // 16-cell blocks of a that a chunk meets
constexpr int kTailPad = 18;
constexpr uint64_t kTailSplit = kTailCounters;     // fewer tiles than this: split their D ranges
constexpr uint64_t kTailPartials = 2 * kTailSplit;  // at most, kTailTile values each
typedef double v4d __attribute__((ext_vector_type(4)));

// Tiles of a row and, with `part` D steps per workgroup, the workgroups of a
// pair (tile t takes 16 t + 16 steps).
__host__ __device__ inline uint32_t tail_tiles(uint64_t W) {
    return (uint32_t)((W + kTailTile - 1) / kTailTile);
}
__host__ __device__ inline uint32_t tail_parts(uint32_t tile, uint32_t part) {
    return (16 * tile + 16 + part - 1) / part;
}

__global__ void __launch_bounds__(kTailPairBlock) k_tail_pair(const double *in, double *out,
                                                              uint32_t rows, uint32_t bins,
                                                              uint32_t part, uint64_t per_pair,
                                                              double *partial, uint32_t *arrived) {
    __shared__ double s_a[kTailBlocks * kTailPad];  // blocks of 16, padded: no bank conflicts
    __shared__ double s_b[16 * kTailChunk + 16];
    __shared__ double s_red[kTailWaves][kTailTile];
    __shared__ uint32_t s_last;
    const int64_t W = (int64_t)bins + 1;
    const uint32_t T = tail_tiles((uint64_t)W);
    const uint64_t pairs = rows / 2, items = pairs * per_pair + (rows % 2 ? T : 0);
    const int tid = (int)threadIdx.x, wave = tid / 64, lane = tid % 64;
    const int li = lane % 16, lk = lane / 16;
    for (uint64_t item = blockIdx.x; item < items; item += gridDim.x) {
        const uint64_t p = item / per_pair;
        if (p >= pairs) {  // the odd last row
            const int64_t j = (int64_t)(item - pairs * per_pair) * kTailTile + tid;
            if (j < W) out[pairs * W + j] = in[2 * pairs * W + j];
            continue;
        }
        uint64_t rest = item - p * per_pair;
        uint32_t tile = T - 1;  // the longest first
        int more = -1;          // a second tile for this workgroup
        if (part >= 16 * T) {   // whole tiles, a long one with a short one
            more = (int)rest < (int)tile - (int)rest ? (int)rest : -1;
            tile -= (uint32_t)rest;
            rest = 0;
        } else {
            while (rest >= tail_parts(tile, part)) rest -= tail_parts(tile--, part);
        }
        const uint32_t nparts = tail_parts(tile, part);
        for (;; tile = (uint32_t)more, more = -1) {
        const int64_t c0 = 16 * (int64_t)tile;
        const int64_t d0 = (int64_t)rest * part;
        const int64_t d1 = d0 + part < c0 + 16 ? d0 + part : c0 + 16;
        const double *a = in + 2 * p * W, *b = a + W;
        v4d acc0 = {0, 0, 0, 0}, acc1 = {0, 0, 0, 0};
        // the next chunk's values are on their way while this one is multiplied
        constexpr int kA = (16 * kTailBlocks + kTailPairBlock - 1) / kTailPairBlock;
        constexpr int kB = (16 * kTailChunk + 15 + kTailPairBlock - 1) / kTailPairBlock;
        double va[kA], vn[kA], vb[kB];
        auto fetch = [&](int64_t D0) {
            // block x of s_a is block c0 - D0 - 31 + x of a
            const int64_t ia = 16 * (c0 - D0 - (kTailChunk - 1)), ib = 16 * D0 - 15;
#pragma unroll
            for (int q = 0; q < kA; ++q) {
                const int64_t i = ia + tid + q * kTailPairBlock;
                va[q] = i >= 0 && i < W ? a[i] : 0.0;
                vn[q] = i >= 0 && i + 1 < W ? a[i + 1] : 0.0;
            }
#pragma unroll
            for (int q = 0; q < kB; ++q) {
                const int64_t i = ib + tid + q * kTailPairBlock;
                vb[q] = i >= 0 && i < W ? b[i] : 0.0;
            }
        };
        fetch(d0);
        for (int64_t D0 = d0; D0 < d1; D0 += kTailChunk) {
            __syncthreads();  // the previous chunk is consumed
#pragma unroll
            for (int q = 0; q < kA; ++q) {
                const int x = tid + q * kTailPairBlock;
                if (x < 16 * kTailBlocks) s_a[(x / 16) * kTailPad + x % 16] = va[q] - vn[q];
            }
#pragma unroll
            for (int q = 0; q < kB; ++q) {
                const int x = tid + q * kTailPairBlock;
                if (x < 16 * kTailChunk + 15) s_b[x] = vb[q];
            }
            __syncthreads();
            if (D0 + kTailChunk < d1) fetch(D0 + kTailChunk);
            const int steps = d1 - D0 < kTailChunk ? (int)(d1 - D0) : kTailChunk;
#pragma unroll 2
            for (int e = wave; e < steps; e += kTailWaves) {  // uniform over the wave
                const double *sa = s_a + (li - e + kTailChunk - 1) * kTailPad + lk;
                const double *sb = s_b + 16 * e + li - lk + 15;
                acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(sb[0], sa[0], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(sb[-4], sa[4], acc1, 0, 0, 0);
                acc0 = __builtin_amdgcn_mfma_f64_16x16x4f64(sb[-8], sa[8], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f64_16x16x4f64(sb[-12], sa[12], acc1, 0, 0, 0);
            }
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q)  // row 4 q + lk, column li
            s_red[wave][16 * li + 4 * q + lk] = acc0[q] + acc1[q];
        __syncthreads();
        double v = 0.0;
        for (int w = 0; w < kTailWaves; ++w) v += s_red[w][tid];
        const int64_t j = 16 * c0 + tid;
        if (nparts > 1) {
            // item numbers of a tile's parts are consecutive
            // (agent-scope stores and loads reach the memory all XCDs see, so
            // no fence has to write back or invalidate a whole cache; the
            // stores have arrived before the counter is touched)
            st(partial + item * kTailTile + tid, v);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (tid == 0) {
                uint32_t *cnt = arrived + p * T + tile;
                const uint32_t before = atomicAdd(cnt, 1u);
                s_last = before + 1 == nparts;
                if (s_last) atomicExch(cnt, 0u);  // ready for the next level
            }
            __syncthreads();
            if (!s_last) break;  // uniform
            const double *first = partial + (item - rest) * kTailTile;
            v = 0.0;
            for (uint32_t q = 0; q < nparts; ++q)
                v += ld(first + (uint64_t)q * kTailTile + tid);
        }
        if (j < W) out[p * W + j] = v + (j + 1 < W ? a[j + 1] : 0.0);
        if (more < 0) break;
        }
    }
}

// Scratch of a tail: the gain total and the tiles' arrival counters (cleared
// by k_tail_total), the parts' sums, and two buffers of survival functions.
struct TailScratch {
    uint64_t *total;
    uint32_t *arrived;  // [kTailSplit]
    double *partial;    // [kTailPartials * kTailTile]
    double *bufA, *bufB;  // s W and ceil(s / 2) W values
};

// Survival functions of the s >= 1 records, then the tree; enqueued only.
void tail_enqueue(uint32_t s, const uint64_t *tau, const uint32_t *second, const uint64_t *gain,
                  uint32_t bins, double max_rel, const TailScratch &T, double *tail,
                  hipStream_t hs) {
    const uint64_t W = (uint64_t)bins + 1;
    k_tail_total<<<1, kTailBlock, 0, hs>>>(s, gain, T.total, T.arrived);
    SKIM_LAUNCH_CHECK();
    double *in = s == 1 ? tail : T.bufA, *out = T.bufB;
    k_tail_survival<<<grid_for((uint64_t)s * W, kTailBlock), kTailBlock, 0, hs>>>(
        s, tau, second, gain, T.total, bins, max_rel, in);
    SKIM_LAUNCH_CHECK();
    const uint32_t tiles = tail_tiles(W);
    for (uint32_t rows = s; rows > 1; rows = (rows + 1) / 2) {
        const uint64_t pairs = rows / 2;
        uint32_t part = 16 * tiles;
        uint64_t per_pair = (tiles + 1) / 2;
        if (pairs * tiles < kTailSplit) {
            // about kTailSplit parts in all, none below one chunk of steps: a
            // tile adds at most one more than its share, so there are at most
            // kTailPartials of them
            const uint64_t steps = pairs * 8 * tiles * (tiles + 1);
            part = (uint32_t)std::max<uint64_t>(kTailChunk, (steps + kTailSplit - 1) / kTailSplit);
            per_pair = 0;
            for (uint32_t t = 0; t < tiles; ++t) per_pair += tail_parts(t, part);
        }
        const uint64_t items = pairs * per_pair + (rows % 2 ? tiles : 0);
        if (rows == 2) out = tail;
        k_tail_pair<<<(unsigned)std::min<uint64_t>(items, 1u << 20), kTailPairBlock, 0, hs>>>(
            in, out, rows, bins, part, per_pair, T.partial, T.arrived);
        SKIM_LAUNCH_CHECK();
        std::swap(in, out);
    }
}

}  // namespace

}  // namespace skim

struct skim_greedy_state {
    int device = 0;
    std::unique_ptr<skim::Arena> mem;
    uint32_t n = 0, ell = 0, k = 0;
    uint64_t seed = 0, m = 0;
    const uint64_t *row_ptr = nullptr;
    const uint32_t *col = nullptr;
    const uint32_t *thr = nullptr;
    uint32_t selected = 0;
    uint64_t rank_next = 0;   // the order holds every pair of a rank below this one
    uint32_t *order = nullptr;
    uint64_t order_step = 0;  // pairs the next step aims at
    bool ahead_due = true;    // the window has not been searched yet
    uint64_t cursor = 0;      // pairs used, as the last launch left it
    skim::SkArgs args{};
};

namespace skim {

// The control block of a run that has used `cursor` pairs; the next window
// has not been searched.
void greedy_set_ctl(skim_greedy_state *st, uint64_t cursor, uint64_t pool_used, hipStream_t s) {
    SkCtl c{};
    c.cursor = c.a_lo = cursor;
    c.pool_used = pool_used;
    c.a_w = kAheadFirst;
    c.a_fail = ~0ull;
    st->ahead_due = true;
    st->cursor = cursor;
    SKIM_HIP(hipMemcpyAsync(st->args.ctl, &c, sizeof c, hipMemcpyHostToDevice, s));
    SKIM_HIP(hipStreamSynchronize(s));
}

// The next step of the pairs' order by rank.
void greedy_extend_order(skim_greedy_state *st, hipStream_t s) {
    SkArgs &A = st->args;
    const uint64_t left = A.nsrc - A.ordered;
    const bool whole = A.nsrc <= kOrderWhole;
    Arena T(s);
    uint64_t count = A.nsrc;
    uint64_t *keys;
    uint32_t *vals;
    if (whole) {
        keys = T.alloc<uint64_t>(count);
        vals = T.alloc<uint32_t>(count);
        k_pair_keys<<<grid_for(count, 256, 8192), 256, 0, s>>>(A.n, A.ell, A.seed, keys, vals);
        SKIM_LAUNCH_CHECK();
    } else {
        // the last step (the one that would leave less than it takes) ends
        // at the highest rank
        const double width = std::ldexp((double)st->order_step / (double)A.nsrc, 64);
        const bool last = left <= 2 * st->order_step ||
                          (double)st->rank_next + width >= std::ldexp(1.0, 64) * (1 - 1e-9);
        const uint64_t r0 = st->rank_next, r1 = last ? ~0ull : r0 + (uint64_t)width;
        uint32_t *counts = T.alloc<uint32_t>(kOrderGrid);
        unsigned long long *totals = T.alloc<unsigned long long>(2);
        fill_u64((uint64_t *)totals, 0, 2, s);
        k_rank_count<<<kOrderGrid, kOrderBlock, 0, s>>>(A.n, A.ell, A.seed, r0, r1, counts, totals);
        SKIM_LAUNCH_CHECK();
        read_back(&count, totals, sizeof count, s);
        keys = T.alloc<uint64_t>(count ? count : 1);
        vals = T.alloc<uint32_t>(count ? count : 1);
        k_rank_take<<<kOrderGrid, kOrderBlock, 0, s>>>(A.n, A.ell, A.seed, r0, r1, counts,
                                                       totals + 1, keys, vals);
        SKIM_LAUNCH_CHECK();
        st->rank_next = r1 + 1;
        st->order_step *= 4;
    }
    if (count) {
        uint64_t *keys2 = T.alloc<uint64_t>(count);
        uint32_t *out = st->order + A.ordered;
        size_t tmp_bytes = 0;
        // large sorts on the high halves (then k_rank_ties); small ones go to
        // another rocPRIM algorithm, which on the high halves alone did not
        // order the pairs of a 1000-node graph, and are cheap: the whole rank
        const unsigned begin_bit = count > kHalfSortPairs ? 32u : 0u;
        SKIM_HIP(rocprim::radix_sort_pairs(nullptr, tmp_bytes, keys, keys2, vals, out, (size_t)count,
                                           begin_bit, 64u, s));
        void *tmp = T.get(tmp_bytes);
        SKIM_HIP(rocprim::radix_sort_pairs(tmp, tmp_bytes, keys, keys2, vals, out, (size_t)count,
                                           begin_bit, 64u, s));
        if (begin_bit) {
            k_rank_ties<<<grid_for(count, 256, 8192), 256, 0, s>>>(keys2, out, count);
            SKIM_LAUNCH_CHECK();
        }
    }
    SKIM_HIP(hipStreamSynchronize(s));
    A.ordered += count;
}

skim_greedy_state *greedy_create(const skim_graph *g, uint32_t ell, uint32_t k, uint64_t seed,
                                        hipStream_t s) {
    SKIM_REQUIRE(ell >= 1 && ell <= 64, "l must be in [1, 64]");
    // sizes and batch counters are 16-bit halves of words
    SKIM_REQUIRE(k >= 2 && k <= 65535, "k must be in [2, 65535]");
    SKIM_REQUIRE(g != nullptr, "graph is NULL");
    if ((uint64_t)g->n > (1ull << 22)) {
        set_error("skim_greedy supports n <= 4194304 (per-thread search queues of n entries)");
        throw Fail{SKIM_EUNSUPPORTED};
    }
    auto st = std::make_unique<skim_greedy_state>();
    SKIM_HIP(hipGetDevice(&st->device));
    st->mem = std::make_unique<Arena>(s, /*persistent=*/true);
    Arena &M = *st->mem;
    const uint32_t n = g->n;
    {
        Arena T(s);
        uint32_t *esrc = T.alloc<uint32_t>(g->m ? g->m : 1);
        validate_graph(g, esrc, T);
        // on large graphs the in-lists as the sketch build makes them and the
        // out-lists by the same chunked passes (no atomic per entry, scratch
        // in T); on small ones both from one coin pass (fewer launches)
        LiveLists fwd;
        if (n >= kSkimPairListNodes) {
            const PairLists rev = build_pair_lists(g, ell, seed, esrc, T, &M);
            fwd = build_out_lists(g, ell, seed, esrc, T, &M);
            st->args.rlive = rev.live;
            st->args.rsrc = rev.adj;
        } else {
            const LiveLists rev = build_live_lists(g, ell, seed, esrc, /*forward=*/false, M, &fwd);
            st->args.rptr = rev.ptr;
            st->args.radj = rev.adj;
        }
        st->args.fptr = fwd.ptr;
        st->args.fadj = fwd.adj;
        SKIM_HIP(hipStreamSynchronize(s));
    }
    const uint64_t nsrc = (uint64_t)n * ell;
    st->order = M.alloc<uint32_t>(nsrc);
    st->order_step = kOrderFirst;
    st->args.order = st->order;
    st->args.nsrc = nsrc;
    const uint64_t npairs = (uint64_t)n * kPairStride;
    SkArgs &A = st->args;
    A.n = n;
    A.ell = ell;
    A.k = k;
    A.covered = M.alloc<uint32_t>(npairs);
    const uint64_t cwords = size_words(n);
    A.size = M.alloc<uint32_t>(cwords);
    A.sel = M.alloc<uint32_t>(n);
    A.idx = M.alloc<uint64_t>(npairs);
    A.heavy = M.alloc<uint64_t>(3 * 2 * (uint64_t)kHeavyItems);
    A.front = M.alloc<uint32_t>(2 * npairs);
    A.ahead = M.alloc<uint64_t>(kAheadMax);
    A.apool_cap = std::max<uint64_t>(1ull << 16, (uint64_t)kAheadPoolNodes * n);
    A.apool = M.alloc<uint32_t>(A.apool_cap);
    A.along = M.alloc<uint32_t>(2 * kAheadMax);
    A.gqueue = M.alloc<uint32_t>((uint64_t)kAheadGiants * n);
    A.vis_words = (n + 31) / 32;
    A.vis = M.alloc<uint32_t>((uint64_t)kAheadGiants * A.vis_words);
    fill_u32(A.vis, 0, (uint64_t)kAheadGiants * A.vis_words, s);
    A.pool_cap = std::max<uint64_t>(1ull << 16, 2 * A.nsrc);
    A.pool = M.alloc<uint32_t>(A.pool_cap);
    A.ctl = M.alloc<SkCtl>(1);
    A.seed = seed;
    A.rec_tau = M.alloc<uint64_t>(n);
    A.rec_second = M.alloc<uint32_t>(n);
    fill_u32(A.covered, 0, npairs, s);
    fill_u32(A.size, 0, cwords, s);
    fill_u32(A.sel, 0, n, s);
    fill_u64(A.idx, 0, npairs, s);
    greedy_set_ctl(st.get(), 0, 0, s);
    st->n = n;
    st->ell = ell;
    st->k = k;
    st->seed = seed;
    st->m = g->m;
    st->row_ptr = g->row_ptr;
    st->col = g->col;
    st->thr = g->thr;
    SKIM_HIP(hipStreamSynchronize(s));
    return st.release();
}

void greedy_run(skim_greedy_state *st, uint32_t s_goal, uint32_t *seeds, uint64_t *gains,
                       double *gain_d, hipStream_t s) {
    SkArgs &A = st->args;
    uint32_t done = 0;
    int growths = 0;
    while (done < s_goal) {
        if (st->ahead_due) {
            while (A.ordered < A.nsrc && A.ordered <= st->cursor) greedy_extend_order(st, s);
            k_ahead_short<<<kAheadMax / kAheadBlock, kAheadBlock, 0, s>>>(A);
            SKIM_LAUNCH_CHECK();
            k_ahead_wave<<<kAheadWaveGrid, 64 * kAheadWaves, 0, s>>>(A);
            SKIM_LAUNCH_CHECK();
            k_ahead_giant<<<kAheadGiants, kAheadGiantBlock, 0, s>>>(A);
            SKIM_LAUNCH_CHECK();
            st->ahead_due = false;
        }
        auto skim = A.n <= kSkimLdsNodes ? k_skim<true> : k_skim<false>;
        skim<<<1, kSkimBlock, 0, s>>>(A, s_goal - done, kSkimHandoff, seeds + done, gains + done,
                                      gain_d ? gain_d + done : nullptr, A.rec_tau + st->selected,
                                      A.rec_second + st->selected);
        SKIM_LAUNCH_CHECK();
        SkCtl c;
        read_back(&c, A.ctl, sizeof c, s);
        st->cursor = c.cursor;
        done += c.done;
        st->selected += c.done;
        if (c.flags & kFlagPool) {
            SKIM_REQUIRE(++growths < 40, "SKIM index pool did not converge");
            // grow the inverted-index pool, keep its contents, continue
            const uint64_t cap = std::max<uint64_t>(2 * A.pool_cap, c.need + c.need / 2);
            uint32_t *np = st->mem->alloc<uint32_t>(cap);
            SKIM_HIP(hipMemcpyAsync(np, A.pool, c.pool_used * sizeof(uint32_t),
                                    hipMemcpyDeviceToDevice, s));
            st->mem->release(A.pool);
            A.pool = np;
            A.pool_cap = cap;
            fill_u32(&A.ctl->flags, 0, 1, s);
        } else if (c.flags & kFlagAhead) {
            st->ahead_due = true;
            fill_u32(&A.ctl->flags, 0, 1, s);
        } else if (c.pend) {
            // the seed's residual search continues on the whole grid, levels
            // in batches (an empty level's launch does nothing); every level
            // covers at least one new pair
            const uint64_t max_levels = (uint64_t)A.n * kPairStride + 1;
            const uint32_t r0 = c.rcur;
            uint32_t L = 0;
            bool back = false;
            for (;;) {
                for (int j = 0; j < 8; ++j, ++L) {
                    k_resid_level<<<kResidGrid, kResidBlock, 0, s>>>(A, L, r0);
                    SKIM_LAUNCH_CHECK();
                }
                read_back(&c, A.ctl, sizeof c, s);
                // level L's frontier, and the pairs level L - 1 deferred
                const uint64_t f = c.rsize[16 * (L % 3)], h = c.hsize[16 * ((L + 2) % 3)];
                if (f == 0 && h == 0) break;
                if (h == 0 && f <= kSkimHandBack) {  // k_skim resumes the search at level L
                    k_resid_handback<<<1, 1, 0, s>>>(A, L, r0);
                    SKIM_LAUNCH_CHECK();
                    back = true;
                    break;
                }
                SKIM_REQUIRE(L < max_levels, "SKIM residual search did not end");
            }
            if (back) continue;
            k_resid_finish<<<1, 1, 0, s>>>(A, seeds + done, gains + done,
                                           gain_d ? gain_d + done : nullptr);
            SKIM_LAUNCH_CHECK();
            ++done;
            ++st->selected;
        } else if (done < s_goal) {
            set_error("SKIM stopped early");
            throw Fail{SKIM_EDEVICE};
        }
    }
}

}  // namespace skim

extern "C" skim_status skim_greedy(const skim_graph *g, uint32_t ell, uint32_t k, uint64_t seed,
                                   uint32_t s, uint32_t *seeds, uint64_t *gain_pairs, double *gain,
                                   skim_greedy_state **state, void *stream) {
    skim::clear_error();
    hipStream_t hs = (hipStream_t)stream;
    skim_greedy_state *own = nullptr;
    try {
        SKIM_REQUIRE(s == 0 || (seeds && gain_pairs), "seeds/gain_pairs is NULL");
        skim_greedy_state *st = state ? *state : nullptr;
        if (st) {
            SKIM_REQUIRE(g && g->n == st->n && g->m == st->m && g->row_ptr == st->row_ptr &&
                             g->col == st->col && g->thr == st->thr && ell == st->ell &&
                             k == st->k && seed == st->seed,
                         "resumed state belongs to a different graph or parameters");
        } else {
            st = skim::greedy_create(g, ell, k, seed, hs);
            own = st;
        }
        SKIM_REQUIRE(s <= st->n - st->selected, "s exceeds the number of unselected nodes");
        if (s) skim::greedy_run(st, s, seeds, gain_pairs, gain, hs);
        SKIM_HIP(hipStreamSynchronize(hs));
        if (state) *state = st;
        else delete st;
        return SKIM_OK;
    } catch (const skim::Fail &f) {
        if (own && !(state && *state == own)) delete own;
        return f.st;
    }
}

extern "C" void skim_greedy_state_free(skim_greedy_state *state) { delete state; }

extern "C" uint32_t skim_greedy_state_selected(const skim_greedy_state *state) {
    return state ? state->selected : 0;
}

// ------------------------------------------------- suspend / resume a run
// A saved state: a header, then the run's progress arrays, each at an
// offset rounded up to 8 bytes.
namespace skim {
namespace {

constexpr char kImageMagic[8] = {'S', 'K', 'I', 'M', 'G', 'R', 'D', '1'};

struct ImageHeader {
    char magic[8];
    uint32_t n, ell, k, pad;
    uint64_t m, seed, selected, cursor, pool_used;
};

struct ImageLayout {
    uint64_t covered, size, sel, idx, pool, tau, second, total;
};

uint64_t round8(uint64_t x) { return (x + 7) & ~7ull; }

ImageLayout image_layout(uint32_t n, uint64_t selected, uint64_t pool_used) {
    const uint64_t npairs = (uint64_t)n * kPairStride, cwords = 2 * (((uint64_t)n + 3) / 4);
    ImageLayout L;
    L.covered = round8(sizeof(ImageHeader));
    L.size = round8(L.covered + npairs * 4);
    L.sel = round8(L.size + cwords * 4);
    L.idx = round8(L.sel + (uint64_t)n * 4);
    L.pool = round8(L.idx + npairs * 8);
    L.tau = round8(L.pool + pool_used * 4);
    L.second = round8(L.tau + selected * 8);
    L.total = round8(L.second + selected * 4);
    return L;
}

}  // namespace
}  // namespace skim

extern "C" skim_status skim_greedy_state_save(const skim_greedy_state *state, void *buf,
                                              uint64_t *bytes, void *stream) {
    skim::clear_error();
    hipStream_t hs = (hipStream_t)stream;
    try {
        SKIM_REQUIRE(state != nullptr && bytes != nullptr, "state or bytes is NULL");
        const skim::SkArgs &A = state->args;
        skim::SkCtl c;
        skim::read_back(&c, A.ctl, sizeof c, hs);
        const skim::ImageLayout L = skim::image_layout(state->n, state->selected, c.pool_used);
        if (!buf) {
            *bytes = L.total;
            return SKIM_OK;
        }
        SKIM_REQUIRE(*bytes >= L.total, "buffer of %llu bytes; the state needs %llu",
                     (unsigned long long)*bytes, (unsigned long long)L.total);
        uint8_t *b = (uint8_t *)buf;
        skim::ImageHeader h{};
        std::memcpy(h.magic, skim::kImageMagic, sizeof h.magic);
        h.n = state->n;
        h.ell = state->ell;
        h.k = state->k;
        h.m = state->m;
        h.seed = state->seed;
        h.selected = state->selected;
        h.cursor = c.cursor;
        h.pool_used = c.pool_used;
        std::memcpy(b, &h, sizeof h);
        const uint64_t npairs = (uint64_t)state->n * skim::kPairStride;
        const uint64_t cwords = 2 * (((uint64_t)state->n + 3) / 4);
        const struct {
            uint64_t off;
            const void *src;
            uint64_t len;
        } parts[] = {{L.covered, A.covered, npairs * 4},
                     {L.size, A.size, cwords * 4},
                     {L.sel, A.sel, (uint64_t)state->n * 4},
                     {L.idx, A.idx, npairs * 8},
                     {L.pool, A.pool, c.pool_used * 4},
                     {L.tau, A.rec_tau, (uint64_t)state->selected * 8},
                     {L.second, A.rec_second, (uint64_t)state->selected * 4}};
        for (const auto &pt : parts)
            if (pt.len)
                SKIM_HIP(hipMemcpyAsync(b + pt.off, pt.src, pt.len, hipMemcpyDeviceToHost, hs));
        SKIM_HIP(hipStreamSynchronize(hs));
        *bytes = L.total;
        return SKIM_OK;
    } catch (const skim::Fail &f) {
        return f.st;
    }
}

extern "C" skim_status skim_greedy_state_load(const skim_graph *g, uint32_t ell, uint32_t k,
                                              uint64_t seed, const void *buf, uint64_t bytes,
                                              skim_greedy_state **state, void *stream) {
    skim::clear_error();
    hipStream_t hs = (hipStream_t)stream;
    skim_greedy_state *st = nullptr;
    try {
        SKIM_REQUIRE(g != nullptr && buf != nullptr && state != nullptr,
                     "graph, buffer or state is NULL");
        SKIM_REQUIRE(bytes >= sizeof(skim::ImageHeader), "buffer too small for a saved state");
        skim::ImageHeader h;
        std::memcpy(&h, buf, sizeof h);
        SKIM_REQUIRE(std::memcmp(h.magic, skim::kImageMagic, sizeof h.magic) == 0,
                     "not a saved SKIM state");
        SKIM_REQUIRE(h.n == g->n && h.m == g->m && h.ell == ell && h.k == k && h.seed == seed,
                     "the saved state belongs to another graph or parameters");
        SKIM_REQUIRE(h.selected <= h.n && h.cursor <= (uint64_t)h.n * ell,
                     "saved state is inconsistent");
        const skim::ImageLayout L = skim::image_layout(h.n, h.selected, h.pool_used);
        SKIM_REQUIRE(bytes >= L.total, "saved state truncated (%llu of %llu bytes)",
                     (unsigned long long)bytes, (unsigned long long)L.total);
        st = skim::greedy_create(g, ell, k, seed, hs);
        skim::SkArgs &A = st->args;
        if (h.pool_used > A.pool_cap) {
            const uint64_t cap = h.pool_used + h.pool_used / 2;
            uint32_t *np = st->mem->alloc<uint32_t>(cap);
            st->mem->release(A.pool);
            A.pool = np;
            A.pool_cap = cap;
        }
        const uint8_t *b = (const uint8_t *)buf;
        const uint64_t npairs = (uint64_t)h.n * skim::kPairStride;
        const uint64_t cwords = 2 * (((uint64_t)h.n + 3) / 4);
        const struct {
            void *dst;
            uint64_t off, len;
        } parts[] = {{A.covered, L.covered, npairs * 4},
                     {A.size, L.size, cwords * 4},
                     {A.sel, L.sel, (uint64_t)h.n * 4},
                     {A.idx, L.idx, npairs * 8},
                     {A.pool, L.pool, h.pool_used * 4},
                     {A.rec_tau, L.tau, h.selected * 8},
                     {A.rec_second, L.second, h.selected * 4}};
        for (const auto &pt : parts)
            if (pt.len)
                SKIM_HIP(hipMemcpyAsync(pt.dst, b + pt.off, pt.len, hipMemcpyHostToDevice, hs));
        skim::greedy_set_ctl(st, h.cursor, h.pool_used, hs);
        st->selected = (uint32_t)h.selected;
        *state = st;
        return SKIM_OK;
    } catch (const skim::Fail &f) {
        delete st;
        return f.st;
    }
}

extern "C" skim_status skim_greedy_records(const skim_greedy_state *state, uint32_t first,
                                           uint32_t count, uint64_t *tau, uint32_t *second,
                                           void *stream) {
    skim::clear_error();
    hipStream_t hs = (hipStream_t)stream;
    try {
        SKIM_REQUIRE(state != nullptr, "state is NULL");
        SKIM_REQUIRE(first <= state->selected && count <= state->selected - first,
                     "records [%u, %u) outside the %u selected seeds", first, first + count,
                     state->selected);
        SKIM_REQUIRE(count == 0 || tau || second, "tau and second are both NULL");
        if (count && tau)
            SKIM_HIP(hipMemcpyAsync(tau, state->args.rec_tau + first, count * sizeof(uint64_t),
                                    hipMemcpyDeviceToDevice, hs));
        if (count && second)
            SKIM_HIP(hipMemcpyAsync(second, state->args.rec_second + first,
                                    count * sizeof(uint32_t), hipMemcpyDeviceToDevice, hs));
        SKIM_HIP(hipStreamSynchronize(hs));
        return SKIM_OK;
    } catch (const skim::Fail &f) {
        return f.st;
    }
}

// ------------------------------------------- the tail without allocation
// skim_discrepancy_tail_noalloc: the same kernels, with their scratch (the
// gain total, the per-seed survival functions and one level of the pairwise
// convolution tree) in a file-scope device array instead of memory the call
// allocates.  Each GPU holds its own copy of `scratch` at its own address,
// looked up once per device with hipGetSymbolAddress; host code only ever
// uses that address.
namespace skim {
namespace {

// seeds * (bins + 1) at most; the words hold the gain total (one 256-byte
// slot), the tiles' arrival counters, the parts' sums, s (bins + 1) survival
// values and ceil(s / 2) (bins + 1) values of a tree level (at most half the
// cells plus half a row): about 16.3 MiB.
constexpr uint64_t kNoAllocCells = 1ull << 20;
constexpr uint64_t kNoAllocHead = 32 + kTailSplit / 2 + kTailPartials * kTailTile;
constexpr uint64_t kNoAllocWords = kNoAllocHead + kNoAllocCells + kNoAllocCells / 2 + 32800;

}  // namespace
}  // namespace skim

static __device__ __align__(256) double scratch[skim::kNoAllocWords];

namespace skim {
namespace {

std::mutex g_scratch_mu;
double *g_scratch_ptr[64] = {};

double *scratch_on_device(int dev) {
    SKIM_REQUIRE(dev >= 0 && dev < 64, "device index %d out of range", dev);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        SKIM_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        g_scratch_ptr[dev] = (double *)ptr;
    }
    return g_scratch_ptr[dev];
}

}  // namespace
}  // namespace skim

extern "C" skim_status skim_discrepancy_tail_noalloc(uint32_t s, const uint64_t *tau,
                                                     const uint32_t *second,
                                                     const uint64_t *gain_pairs, uint32_t bins,
                                                     double max_rel_error, double *tail,
                                                     void *stream) {
    using namespace skim;
    clear_error();
    hipStream_t hs = (hipStream_t)stream;
    try {
        SKIM_REQUIRE(bins >= 1 && bins <= kTailMaxBins, "bins must be in [1, %u]", kTailMaxBins);
        SKIM_REQUIRE(max_rel_error > 0.0 && max_rel_error <= 1e300,
                     "max_rel_error must be positive and finite");
        SKIM_REQUIRE(tail != nullptr, "tail is NULL");
        SKIM_REQUIRE(s == 0 || (tau && second && gain_pairs), "tau/second/gain_pairs is NULL");
        const uint64_t W = (uint64_t)bins + 1;
        if ((uint64_t)s * W > kNoAllocCells) {
            set_error("seeds * (bins + 1) = %llu exceeds the %llu cells of the no-allocation "
                      "scratch", (unsigned long long)((uint64_t)s * W),
                      (unsigned long long)kNoAllocCells);
            throw Fail{SKIM_EUNSUPPORTED};
        }
        if (s == 0) {  // the empty sum is 0 with certainty
            fill_u64((uint64_t *)tail, 0, W, hs);
            fill_u64((uint64_t *)tail, 0x3FF0000000000000ull, 1, hs);  // 1.0
            return SKIM_OK;
        }
        int dev = 0;
        SKIM_HIP(hipGetDevice(&dev));
        double *base = scratch_on_device(dev);
        TailScratch S;
        S.total = (uint64_t *)base;
        S.arrived = (uint32_t *)(base + 32);
        S.partial = base + 32 + kTailSplit / 2;
        S.bufA = base + kNoAllocHead;
        S.bufB = S.bufA + (uint64_t)s * W;
        tail_enqueue(s, tau, second, gain_pairs, bins, max_rel_error, S, tail, hs);
        return SKIM_OK;
    } catch (const Fail &f) {
        return f.st;
    }
}

extern "C" skim_status skim_discrepancy_tail(uint32_t s, const uint64_t *tau,
                                             const uint32_t *second, const uint64_t *gain_pairs,
                                             uint32_t bins, double max_rel_error, double *tail,
                                             void *stream) {
    using namespace skim;
    clear_error();
    hipStream_t hs = (hipStream_t)stream;
    try {
        SKIM_REQUIRE(bins >= 1 && bins <= kTailMaxBins, "bins must be in [1, %u]", kTailMaxBins);
        SKIM_REQUIRE(max_rel_error > 0.0 && max_rel_error <= 1e300,
                     "max_rel_error must be positive and finite");
        SKIM_REQUIRE(tail != nullptr, "tail is NULL");
        SKIM_REQUIRE(s == 0 || (tau && second && gain_pairs), "tau/second/gain_pairs is NULL");
        const uint64_t W = (uint64_t)bins + 1;
        if ((uint64_t)s * W > kTailMaxCells) {
            set_error("seeds * (bins + 1) exceeds %llu", (unsigned long long)kTailMaxCells);
            throw Fail{SKIM_EUNSUPPORTED};
        }
        if (s == 0) {  // the empty sum is 0 with certainty
            fill_u64((uint64_t *)tail, 0, W, hs);
            fill_u64((uint64_t *)tail, 0x3FF0000000000000ull, 1, hs);  // 1.0
            SKIM_HIP(hipStreamSynchronize(hs));
            return SKIM_OK;
        }
        Arena T(hs);
        TailScratch S;
        S.total = T.alloc<uint64_t>(1);
        S.arrived = T.alloc<uint32_t>(kTailSplit);
        S.partial = T.alloc<double>(kTailPartials * kTailTile);
        S.bufA = T.alloc<double>((uint64_t)s * W);
        S.bufB = T.alloc<double>(((uint64_t)s + 1) / 2 * W);
        tail_enqueue(s, tau, second, gain_pairs, bins, max_rel_error, S, tail, hs);
        SKIM_HIP(hipStreamSynchronize(hs));
        return SKIM_OK;
    } catch (const Fail &f) {
        return f.st;
    }
}
