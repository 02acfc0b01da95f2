// skim_greedy.hip -- SKIM greedy seed selection (Section 4, Algorithm 1).
//
// State on the device: live reverse and forward lists of every pair, the
// pairs sorted by rank, a few bits per pair, size[node], and the inverted index
// (for every processed pair, the nodes its reverse search reached).
//
// One persistent workgroup runs the selection loop (the loop is sequential
// per seed); the searches it scans are made ahead on the whole grid, and
// residual searches that grow large continue there:
//  * rank order: made in steps as the loop gets there, the lowest ranks first.
//  * scan: the reverse searches of the next pairs in rank order (an uncovered
//    pair never reaches a covered one, so a search is independent of the
//    others and of the seeds chosen since it was made) are added to the sizes
//    a batch at a time.  If some node's size reaches k, the first prefix at
//    which one does is the smallest position at which a filling node receives
//    its k-th entry, found from the entries of the filling nodes alone (binary
//    search over prefixes when there are too many); the pairs after it are
//    taken back and scanned again later, the others are committed (index
//    entries).  The nodes that reached k all sit in the last committed pair's
//    search; the smallest id among them is the seed.
//  * exhaustion: with every rank processed, the unselected node with the
//    largest size (smallest id on ties) is the seed.
//  * records: before the residual update, the rank tau of the pair that filled
//    the seed's sketch and the second largest sketch k' (largest size among
//    the other unselected nodes, one less for nodes in that pair's search)
//    are stored per seed for the adaptive error estimate (Section 4).
//  * residual: a level-synchronous forward search from the seed over all
//    instances at once over live out-edges, not entering covered pairs; every
//    newly covered pair counts towards the seed's gain and decrements the size
//    of every node in its index entry, which is then erased.  A level of more
//    than kSkimHandoff pairs, or a seed with more than kSkimHandoffEdges live
//    out-edges, ends the workgroup's launch; the rest of that search runs level
//    by level on the whole grid (k_resid_level); a search whose next level
//    there is small again is handed back, and the relaunched loop resumes it.
//
// The adaptive error estimate itself (skim_discrepancy_tail) bounds each
// seed's discrepancy with eq. (chernoff) on a grid of discrepancy values and
// convolves the per-seed distributions pairwise in a tree of launches.
#include "skim_internal.h"
#include "skim_tail.h"
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
// ... and up to this size, in the same LDS words, the bits of their pairs (34
// bytes per node in all).
constexpr uint32_t kSkimStateNodes = 1200;
static_assert(kSkimStateNodes % 8 == 0 && kSkimStateNodes / 2 + 8 * kSkimStateNodes <= kSkimLdsWords, "");
constexpr uint32_t kFlagPool = 1u, kFlagAhead = 2u;
// Searches of at most this many nodes are staged by their own thread; a batch
// with a longer one is staged by flat position.
constexpr uint32_t kSkimSerial = 32;
// A pair with more live out-edges than this is expanded apart from the other
// pairs of its level, its edges spread over the whole block or grid: a wave
// with a few such pairs is the last of a level (10^6 nodes, 50 seeds, with
// lists above 32, 64, 128 and 256: 20.0, 20.0, 20.6 and 21.4 ms).
constexpr uint64_t kLongEdges = 64;
// A residual level with more pairs than this continues on the whole grid.
constexpr uint64_t kSkimHandoff = 4096;
// ... and so does a seed whose own live out-edges are more than this.
constexpr uint64_t kSkimHandoffEdges = 65536;
// A search on the grid whose next level has at most this many pairs goes
// back to the workgroup (a level there costs less than two launches).
constexpr uint64_t kSkimHandBack = 2048;
// Long pairs of a level: in the workgroup at most kBlockItems, on the grid at
// most kHeavyItems; more are expanded with the others.
constexpr uint32_t kBlockItems = 64, kHeavyItems = 1u << 16;
// Levels of a round on the grid: after one, a search that has ended or become
// small goes back to k_skim.  A multiple of 6: the level counters (three) and
// the frontier buffers (two) are again where they were.
constexpr int kRoundLevels = 6;
// Rounds enqueued before the host reads the control block.
constexpr int kRounds = 8;
// Entries of the nodes that fill within a batch, kept to find the filling
// prefix directly (more: binary search over prefixes).
constexpr uint32_t kSkimCand = 1024;
// Entries of a batch that fit in LDS.
constexpr uint32_t kSkimStage = 8192;
// Positions of the window whose pairs and searches are in LDS.
constexpr uint32_t kSkimAt = 2 * kSkimBlock;

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
    uint32_t done;                 // seeds completed in this call (cleared with flags)
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
    unsigned long long rsize[3 * 16];  // pairs of the level (low half); newly covered (high half)
    unsigned long long hsize[3 * 16];  // long pairs of the level
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
    uint64_t *state;        // [4 n] bits of 16 pairs, see kCovered
    uint32_t *size;         // [size_words(n)] packed 16-bit counters
    uint32_t *sel;          // [n] 0/1
    uint64_t *idx;          // [64 n] first pool entry << 32 | entries, of committed pairs
    uint32_t *pool;
    uint64_t pool_cap;
    uint32_t *front;        // [2 * 64 n] residual levels
    uint64_t *ahead;        // [kAheadMax] searches of the window
    uint32_t *apool;        // [apool_cap] their nodes
    uint64_t apool_cap;
    uint32_t *along;        // [2 kAheadMax] searches left to the wave kernel, to the workgroup kernel
    uint32_t *gqueue;       // [kAheadGiants * n]
    uint32_t *heavy;        // [2][kHeavyItems] long pairs of a grid level
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

// Relaxed atomic accesses at scope kScope: kGroup where one workgroup alone
// reads and writes the data of a launch (k_skim: they are served by the CU's
// cache and its XCD's L2), kAgent where workgroups on several XCDs share it
// (atomics then go to the memory side, several times as long).
constexpr int kGroup = __HIP_MEMORY_SCOPE_WORKGROUP, kAgent = __HIP_MEMORY_SCOPE_AGENT;
template <int kScope, class T> __device__ __forceinline__ T ld(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, kScope);
}
template <int kScope, class T> __device__ __forceinline__ void st(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, kScope);
}
template <int kScope> __device__ __forceinline__ uint32_t or_old(uint32_t *p, uint32_t v) {
    return __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, kScope);
}

// The bits of 16 pairs in a word: covered (a seed reached it), committed (it
// has an index entry), and of its live out-list, whether it is not empty and
// whether it is long (more than kLongEdges).  The atomic that covers a pair
// returns all four: a pair with neither out-edges nor an entry goes no
// further, a long list goes to the level's own list of them at once.  (A word
// per pair and an index word read for each covered pair were 768 MB of random
// lines on 10^6 nodes; these words are 32 MB.)
constexpr uint64_t kCovered = 1, kCommitted = 1ull << 16, kHasEdges = 1ull << 32, kLong = 1ull << 48;
constexpr uint64_t kPairBits = kCovered | kCommitted | kHasEdges | kLong;
template <int kScope>
__device__ __forceinline__ bool is_covered(const uint64_t *state, uint32_t p) {
    return (ld<kScope>(reinterpret_cast<const uint32_t *>(state + (p >> 4))) >> (p & 15u)) & 1u;
}
// Sets the covered bit and gives the bits as they were.
template <int kScope> __device__ __forceinline__ uint64_t cover(uint64_t *state, uint32_t p) {
    return (__hip_atomic_fetch_or(state + (p >> 4), kCovered << (p & 15u), __ATOMIC_RELAXED, kScope) >>
            (p & 15u)) & kPairBits;
}
template <int kScope> __device__ __forceinline__ void commit(uint64_t *state, uint32_t p) {
    __hip_atomic_fetch_or(state + (p >> 4), kCommitted << (p & 15u), __ATOMIC_RELAXED, kScope);
}
// Frontier entries are a pair and whether it has an index entry.
constexpr uint32_t kHasEntry = 1u << 31;

template <int kScope> __device__ __forceinline__ uint32_t cget(const uint32_t *c, uint32_t v) {
    return (ld<kScope>(c + (v >> 1)) >> half_shift(v)) & 0xFFFFu;
}
template <int kScope>
__device__ __forceinline__ uint32_t cadd(uint32_t *c, uint32_t v, uint32_t d) {  // the count as it was
    return (__hip_atomic_fetch_add(c + (v >> 1), d << half_shift(v), __ATOMIC_RELAXED, kScope) >>
            half_shift(v)) & 0xFFFFu;
}
template <int kScope> __device__ __forceinline__ void csub(uint32_t *c, uint32_t v, uint32_t d) {
    __hip_atomic_fetch_sub(c + (v >> 1), d << half_shift(v), __ATOMIC_RELAXED, kScope);
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

// The same for 32-bit values (wave totals below 2^31); `any` is whether flag is
// set in some thread.
template <uint32_t NT>
__device__ __forceinline__ uint64_t block_excl_scan32(uint32_t v, bool flag, uint32_t *wsum,
                                                      uint64_t &total, bool &any) {
    const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
    const uint32_t x = wave_scan_sum(v);
    const bool mine = __any(flag);
    if (lane == 63u) wsum[wave] = x | (mine ? 1u << 31 : 0u);
    __syncthreads();
    uint64_t before = 0, tot = 0;
    uint32_t flags = 0;
#pragma unroll
    for (uint32_t w = 0; w < NT / 64; ++w) {
        const uint32_t word = wsum[w], s = word & ~(1u << 31);
        flags |= word;
        before += w < wave ? s : 0;
        tot += s;
    }
    total = tot;
    any = flags >> 31;
    return before + x - v;
}

// The run that holds flat position t: the largest r with ex[r] <= t, for
// exclusive prefix sums ex[0..NT] (runs of length zero are never returned
// for t below the total).
template <uint32_t NT, class T>
__device__ __forceinline__ uint32_t run_of(const T *ex, T t) {
    uint32_t lo = 0, hi = NT;  // ex[lo] <= t < ex[hi]
    while (hi - lo > 1) {
        const uint32_t mid = (lo + hi) >> 1;
        if (ex[mid] <= t) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The lane whose range holds flat position j of the wave's items laid end to end
// (binary lifting over the lanes' inclusive prefix sums; j below the wave's total).
__device__ __forceinline__ uint32_t wave_owner(uint32_t incl, uint32_t j) {
    uint32_t r = 0;
#pragma unroll
    for (uint32_t step = 32; step > 0; step >>= 1) {
        const uint32_t v = (uint32_t)__shfl((int)incl, (int)(r + step - 1));
        if (v <= j) r += step;
    }
    return r & 63u;
}

// Long pairs of a grid level, their out-edges laid end to end.
struct FlatShared {
    uint64_t ex[kResidBlock + 1], f0[kResidBlock];
    uint32_t q[kResidBlock];
    uint64_t wsum[kResidBlock / 64];
};

// Appends of a grid-wide residual level, staged in LDS and reserved in
// global memory once per chunk (one counter serves the whole grid).
struct ResidStage {
    uint32_t buf[8 * kResidBlock];
    uint32_t n, gain;
    unsigned long long base;
};

struct ScanShared {
    uint64_t ex[kSkimBlock + 1];  // the batch's searches, laid end to end
    uint32_t entry[kSkimStage];
    uint32_t q[kSkimBlock], o[kSkimBlock];  // root and first pool entry of a search
    uint64_t cand[kSkimCand];     // (flat position << 32) | node, nodes that fill
    uint32_t seen[kSkimCand];
};

// Erases the index entries (words ix) of a wave's covered pairs q that have
// one: their nodes lose one from their sizes.  Called by all lanes.
template <int kScope>
__device__ __forceinline__ void erase_entry(const SkArgs &A, uint32_t *SZ, uint32_t q, uint64_t ix) {
    const uint32_t lane = lane_id();
    const bool has = q & kHasEntry;
    if (!__any(has)) return;
    // the search's first node is the pair's own
    if (has) csub<kScope>(SZ, (q & ~kHasEntry) / kPairStride, 1u);
    const uint32_t c = has ? (uint32_t)ix - 1u : 0u, o = (uint32_t)(ix >> 32) + 1u;
    if (__any(c >= (1u << 24))) {  // (a prefix sum of longer entries could wrap)
        for (uint32_t j = 0; j < c; ++j) csub<kScope>(SZ, ld<kScope>(A.pool + o + j), 1u);
        return;
    }
    const uint32_t incl = wave_scan_sum(c);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    for (uint32_t b = 0; b < total; b += 64) {
        const uint32_t j = b + lane, w = wave_owner(incl, j);
        const uint32_t first = (uint32_t)__shfl((int)(incl - c), (int)w);
        const uint32_t wo = (uint32_t)__shfl((int)o, (int)w);
        if (j < total) csub<kScope>(SZ, ld<kScope>(A.pool + wo + (j - first)), 1u);
    }
}

// One wave's share of a residual level: frontier entries base + 0 .. 64 R - 1
// of fc, R per lane so that R accesses per lane are in flight at each step of
// the chain (out-list, out-edge, cover).  The out-edges are laid end to end,
// kResidEdges per lane at a time, and the bits of the pairs they reach, as
// they were, go to `push`.  Index entries of
// the frontier's pairs are erased.
constexpr int kResidEdges = 4;
template <int R> struct ResidWave {
    uint64_t f0[64 * R];
    uint32_t ex[64 * R + 1], q[64 * R];
};
template <int kScope, int R, class Fin, class Push>
__device__ __forceinline__ void resid_wave(const SkArgs &A, uint32_t *SZ, uint64_t *ST, uint64_t base,
                                           uint64_t fc, ResidWave<R> &W, Fin fin,
                                           Push push) {
    const uint32_t lane = lane_id();
    uint32_t q[R];
    uint64_t f0[R], deg[R], ix[R];
#pragma unroll
    for (int r = 0; r < R; ++r) q[r] = base + 64 * r + lane < fc ? fin(base + 64 * r + lane) : 0u;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        f0[r] = deg[r] = 0;
        if (base + 64 * r + lane < fc) {
            const uint32_t p = q[r] & ~kHasEntry;
            f0[r] = A.fptr[p];
            deg[r] = A.fptr[p + 1] - f0[r];
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) ix[r] = q[r] & kHasEntry ? A.idx[q[r] & ~kHasEntry] : 0ull;
    for (;;) {
        // at most 2^22 edges of a pair at a time: their sum does not wrap
        uint32_t total = 0, part[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            part[r] = (uint32_t)min(deg[r], (uint64_t)(1u << 22));
            const uint32_t incl = wave_scan_sum(part[r]);
            W.ex[64 * r + lane] = total + incl - part[r];
            W.f0[64 * r + lane] = f0[r];
            W.q[64 * r + lane] = q[r] % kPairStride;
            total += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        }
        if (total == 0) break;
        if (lane == 0) W.ex[64 * R] = total;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (uint32_t b = 0; b < total; b += 64 * kResidEdges) {
            uint32_t qw[kResidEdges];
            bool add[kResidEdges];
#pragma unroll
            for (int u = 0; u < kResidEdges; ++u) {
                const uint32_t t = b + 64 * u + lane;
                add[u] = t < total;
                qw[u] = 0;
                if (add[u]) {
                    const uint32_t r = run_of<64 * R>(W.ex, t);
                    qw[u] = A.fadj[W.f0[r] + (t - W.ex[r])] * kPairStride + W.q[r];
                }
            }
            uint64_t was[kResidEdges];
#pragma unroll
            for (int u = 0; u < kResidEdges; ++u) was[u] = add[u] ? cover<kScope>(ST, qw[u]) : kCovered;
            push(was, qw);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            f0[r] += part[r];
            deg[r] -= part[r];
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) erase_entry<kScope>(A, SZ, q[r], ix[r]);
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
            if (!is_covered<kAgent>(A.state, p)) {
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
            st<kGroup>(Q, v);
            or_old<kGroup>(V + (v >> 5), 1u << (v & 31u));
            s_tail = 1;
        }
        __syncthreads();
        for (uint32_t head = 0;;) {
            const uint32_t tail = s_tail;
            __syncthreads();
            if (head >= tail) break;  // uniform
            const uint32_t take = min((uint32_t)kAheadGiantBlock, tail - head);
            InList L = {0, 0, 0, true};
            if (tid < take) L = in_list(A, ld<kGroup>(Q + head + tid) * kPairStride + i);
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
                        add = !(ld<kGroup>(V + (v >> 5)) & bit) && !(or_old<kGroup>(V + (v >> 5), bit) & bit);
                    }
                    const uint64_t m = __ballot(add);
                    if (m) {
                        uint32_t pos = 0;
                        if (lane == (uint32_t)__ffsll((long long)m) - 1u)
                            pos = atomicAdd(&s_tail, (uint32_t)__popcll(m));
                        pos = (uint32_t)__shfl((int)pos, __ffsll((long long)m) - 1) +
                              (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
                        if (add) st<kGroup>(Q + pos, v);  // each node once: at most n
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
            const uint32_t v = ld<kGroup>(Q + j);
            st<kGroup>(V + (v >> 5), 0u);
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
// different waves on one cache line are serialised).  kLdsState: so are the
// pairs' bits (at most kSkimStateNodes nodes), one access to the L2 less, of
// 0.5 us, per batch and per residual level (1000 nodes, 200 seeds: 3.5 to 3.1 ms).
//
// What bounds it: the chain of accesses and barriers, about 3 us per batch,
// 3 us per seed's first filling prefix and 2 us per residual level.  1000
// nodes, l = k = 64, 200 seeds: 6.0 ms with a search per thread in each batch
// and six barriers per level, 2.7 ms now (a call 3.0); 10^6 nodes, 50 seeds: 20 and 5 ms.
template <bool kLds, bool kLdsState>
__global__ void __launch_bounds__(kSkimBlock) k_skim(SkArgs A, uint32_t goal, bool begin, uint64_t handoff,
                                                     uint32_t *seeds, uint64_t *gains,
                                                     double *gain_d, uint64_t *rec_tau,
                                                     uint32_t *rec_second) {
    __shared__ unsigned long long s_cursor, s_pool, s_gain, s_best, s_tau;
    __shared__ int s_x;
    __shared__ uint32_t s_stop, s_second, s_xmin, s_ncand, s_resume, s_rcur, s_T, s_found;
    __shared__ unsigned long long s_fill0, s_fill1;
    __shared__ uint32_t s_fcnt[3], s_hcnt[3], s_wsum[kSkimBlock / 64];
    __shared__ __align__(16) uint32_t s_size[kLds ? kSkimLdsWords : 4];
    __shared__ union {
        ScanShared scan;                     // while pairs are scanned
        ResidWave<4> wave[kSkimBlock / 64];  // in the residual search
    } s_u;
    ScanShared &C = s_u.scan;
    __shared__ uint64_t s_ahead[kSkimAt];
    __shared__ uint32_t s_pair[kSkimAt];
    __shared__ uint32_t s_front[2][kSkimLdsFront];
    __shared__ uint32_t s_long[2][kBlockItems];
    const uint32_t tid = threadIdx.x;
    const uint32_t n = A.n, k = A.k;
    // launches are enqueued ahead: nothing to do while a search is on the
    // grid, a request waits for the host or the call's seeds are complete
    const uint32_t it0 = begin ? 0u : A.ctl->done;
    if (A.ctl->pend == 1 || A.ctl->flags || it0 >= goal) return;
    uint32_t *SZ = kLds ? s_size : A.size;
    const uint32_t swords = size_words(n);
    uint64_t *ST = kLdsState ? reinterpret_cast<uint64_t *>(s_size + size_words(kSkimStateNodes))
                             : A.state;
    if constexpr (kLdsState)
        for (uint32_t w = tid; w < 4 * n; w += kSkimBlock) ST[w] = ld<kGroup>(A.state + w);
    if constexpr (kLds)
        for (uint32_t w = tid; w < swords; w += kSkimBlock) s_size[w] = ld<kGroup>(A.size + w);
    const uint64_t a_lo = A.ctl->a_lo;
    const uint64_t a_hi = min((unsigned long long)A.ordered,
                              a_lo + min(A.ctl->a_w, A.ctl->a_fail));
    if (tid == 0) {
        s_cursor = A.ctl->cursor;
        s_pool = A.ctl->pool_used;
        s_stop = 0;
        s_ncand = s_found = 0;
        // a residual search the grid handed back (its frontier got small):
        // the launch starts by finishing that seed
        s_resume = A.ctl->pend == 2;
        if (s_resume) {
            A.ctl->pend = 0;
            s_x = (int)A.ctl->px;
            s_rcur = A.ctl->rcur;
            s_gain = A.ctl->rgain + (A.ctl->rsize[0] >> 32);
            s_fcnt[0] = (uint32_t)A.ctl->rsize[0];
        }
    }
    __syncthreads();
    // Entry t of the batch's searches, laid end to end in thread order:
    // staged in LDS when there is room for all of them.
    bool staged = true;
    auto far_entry = [&](uint64_t t) {
        const uint32_t r = run_of<kSkimBlock>(C.ex, t);
        const uint32_t j = (uint32_t)(t - C.ex[r]);
        return j ? A.apool[(uint64_t)C.o[r] + j] : C.q[r];
    };
    auto entry = [&](uint64_t t) { return staged ? C.entry[t] : far_entry(t); };
    uint64_t at0 = 0, at1 = 0;  // positions in s_pair and s_ahead
    uint32_t tag = 0;            // of the batch, in s_found if some node reaches k
    uint32_t batch = kSkimBlock, taken = 0;  // pairs of a batch; taken since the last seed
    uint32_t it = it0;
    for (; it < goal; ++it) {
        const bool resumed = it == it0 && s_resume;  // uniform
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
            // The batch: what a seed took before, four times, so that most
            // batches of a run of filling ones fill and few pairs are added
            // in vain.
            // Sizes are below k here and grow by at most one per pair: they
            // stay in 16 bits with all of a batch added
            const uint32_t B = (uint32_t)min(a_hi - cursor, (uint64_t)min(batch, 65536u - k));
            if (cursor < at0 || cursor + B > at1) {  // uniform
                at0 = cursor;
                at1 = min(a_hi, cursor + kSkimAt);
                for (uint32_t j = tid; j < at1 - at0; j += kSkimBlock) {
                    s_pair[j] = A.order[cursor + j];
                    s_ahead[j] = A.ahead[cursor - a_lo + j];
                }
                __syncthreads();
            }
            uint32_t cnt = 0, p = 0, first = 0, next = 0;
            if (tid < B) {
                p = s_pair[cursor - at0 + tid];
                const uint64_t a = s_ahead[cursor - at0 + tid];
                first = (uint32_t)(a >> 32);
                // (the second node is on its way with the pair's bits)
                if ((uint32_t)a > 1) next = A.apool[(uint64_t)first + 1];
                if (!is_covered<kGroup>(ST, p)) cnt = (uint32_t)a;
            }
            uint64_t tot;
            bool longer;
            const uint64_t ex =
                block_excl_scan32<kSkimBlock>(cnt, cnt > kSkimSerial, s_wsum, tot, longer);
            C.ex[tid] = ex;
            C.q[tid] = p / kPairStride;
            C.o[tid] = first;
            if (tid == 0) {
                C.ex[kSkimBlock] = tot;
                s_xmin = 0xFFFFFFFFu;
            }
            staged = tot <= kSkimStage;
            if (staged) {
                if (longer) {
                    __syncthreads();  // C.ex and the roots are in place
                    for (uint64_t t = tid; t < tot; t += kSkimBlock) C.entry[t] = far_entry(t);
                } else if (cnt) {
                    C.entry[ex] = p / kPairStride;
                    if (cnt > 1) C.entry[ex + 1] = next;
                    for (uint32_t j = 2; j < cnt; ++j)
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
                f |= cadd<kGroup>(SZ, entry(t), 1u) + 1 >= k;
            ++tag;
            if (__any(f) && (tid & 63u) == 0) s_found = tag;
            __syncthreads();
            const bool filled = s_found == tag;
            uint32_t T = B;
            if (filled) {
                for (uint64_t t0 = 0; t0 < tot; t0 += kSkimBlock) {
                    const uint64_t t = t0 + tid;
                    const uint32_t v = t < tot ? entry(t) : 0u;
                    const bool fills = t < tot && cget<kGroup>(SZ, v) >= k;
                    const uint64_t m = __ballot(fills);
                    if (!m) continue;
                    uint32_t slot = 0;
                    if ((tid & 63u) == 0) slot = atomicAdd(&s_ncand, (uint32_t)__popcll(m));
                    slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)slot) +
                           (uint32_t)__popcll(m & ((1ull << (tid & 63u)) - 1ull));
                    if (fills && slot < kSkimCand) {
                        C.cand[slot] = (t << 32) | v;  // (t below 1024 n <= 2^32)
                        C.seen[slot] = 0;
                    }
                }
                __syncthreads();
                // moves the sizes from prefix `from` of the batch to prefix `to`
                auto move = [&](uint32_t from, uint32_t to) {
                    for (uint64_t t = C.ex[min(from, to)] + tid; t < C.ex[max(from, to)];
                         t += kSkimBlock) {
                        if (from < to) cadd<kGroup>(SZ, entry(t), 1u);
                        else csub<kGroup>(SZ, entry(t), 1u);
                    }
                    __syncthreads();
                };
                const uint32_t nc = s_ncand;
                uint32_t at = B;
                if (nc <= 64) {
                    // every wave by itself, a candidate per lane: entries of
                    // its node in the batch and those at earlier positions
                    const uint32_t lane = tid & 63u;
                    const uint64_t e = lane < nc ? C.cand[lane] : ~0ull;
                    const uint32_t v = (uint32_t)e, pos = (uint32_t)(e >> 32);
                    uint32_t same = 0, before = 0;
                    for (uint32_t c2 = 0; c2 < nc; ++c2) {
                        const uint32_t v2 = (uint32_t)__builtin_amdgcn_readlane((int)v, (int)c2);
                        const uint32_t p2 = (uint32_t)__builtin_amdgcn_readlane((int)pos, (int)c2);
                        same += v2 == v;
                        before += v2 == v && p2 < pos;
                    }
                    const bool kth = lane < nc && cget<kGroup>(SZ, v) - same + before + 1 == k;
                    T = group_min_u32<64>(kth ? pos : 0xFFFFFFFFu);
                } else if (nc <= kSkimCand) {
                    // the same with the pairs of candidates dealt over the
                    // block's threads (both counts in one word)
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
                        if (cget<kGroup>(SZ, (uint32_t)e) - (seen >> 16) + (seen & 0xFFFFu) + 1 == k)
                            atomicMin(&s_xmin, (uint32_t)(e >> 32));
                    }
                    __syncthreads();
                    T = s_xmin;
                } else {
                    uint32_t none = 0;  // prefixes none and T: nothing fills, something does
                    while (T - none > 1) {
                        const uint32_t mid = none + (T - none) / 2;
                        move(at, mid);
                        at = mid;
                        bool g = false;
                        for (uint64_t t = tid; t < C.ex[mid]; t += kSkimBlock)
                            g |= cget<kGroup>(SZ, entry(t)) >= k;
                        ++tag;
                        if (__any(g) && (tid & 63u) == 0) s_found = tag;
                        __syncthreads();
                        if (s_found == tag) T = mid;
                        else none = mid;
                    }
                }
                if (nc <= kSkimCand) {  // T is a flat position: its pair's prefix
                    if (T - (uint32_t)ex < cnt) s_T = tid + 1;
                    __syncthreads();
                    T = s_T;
                }
                move(at, T);
                if (tid == 0) s_xmin = 0xFFFFFFFFu;
            }
            // does the committed prefix fit in the index pool?
            const uint64_t need = C.ex[T], pbase = s_pool;
            if (pbase + need > A.pool_cap) {
                for (uint64_t t = tid; t < need; t += kSkimBlock) csub<kGroup>(SZ, entry(t), 1u);
                if (tid == 0) {
                    A.ctl->flags |= kFlagPool;
                    A.ctl->need = pbase + need;
                    s_stop = 1;
                    s_ncand = 0;
                }
                __syncthreads();
                break;
            }
            // commit pairs [0, T): index entries in pair order
            for (uint64_t t = tid; t < need; t += kSkimBlock) st<kGroup>(A.pool + pbase + t, entry(t));
            if (tid < T && cnt) {
                st<kGroup>(A.idx + p, ((pbase + ex) << 32) | cnt);
                commit<kGroup>(ST, p);
            }
            if (filled) {
                // the nodes that just reached k are in pair T - 1's search;
                // the seed is the smallest of them
                __syncthreads();
                for (uint64_t t = C.ex[T - 1] + tid; t < need; t += kSkimBlock) {
                    const uint32_t v = entry(t);
                    if (cget<kGroup>(SZ, v) >= k) atomicMin(&s_xmin, v);
                }
                if (tid == T - 1) s_tau = pair_rank(A.seed, p);
                __syncthreads();
            }
            taken += T;
            batch = filled ? min((uint32_t)kSkimBlock, max(64u, 4 * taken)) : (uint32_t)kSkimBlock;
            if (filled) taken = 0;
            if (tid == 0) {
                if (filled) {
                    s_x = s_xmin == 0xFFFFFFFFu ? -1 : (int)s_xmin;
                    s_fill0 = C.ex[T - 1];
                    s_fill1 = need;
                }
                s_cursor = cursor + T;
                s_pool = pbase + need;
                s_ncand = 0;
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
                if (!ld<kGroup>(A.sel + v)) {
                    const unsigned long long key =
                        ((unsigned long long)cget<kGroup>(SZ, v) << 32) | (0xFFFFFFFFu - v);
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
            if (v != xs) csub<kGroup>(SZ, v, 1u);
        }
        uint32_t xsize = 0;
        if (tid == 0) {
            s_second = 0;
            xsize = cget<kGroup>(SZ, xs);
            csub<kGroup>(SZ, xs, xsize);
        }
        __syncthreads();
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
            if (v != xs) cadd<kGroup>(SZ, v, 1u);
        }
        if (tid == 0) {
            cadd<kGroup>(SZ, xs, xsize);
            rec_tau[it] = fill1 ? (uint64_t)s_tau : ~0ull;
            rec_second[it] = s_second;
        }
        }  // !resumed
        const uint32_t x = (uint32_t)s_x;
        // ------------------------------------------------- residual problem
        // Level-synchronous over all instances at once: a frontier of pairs
        // (64 v + i) in two halves of the queue area.  A pair is claimed by
        // the atomic that covers it.  One barrier a level: level L reads
        // counter L % 3, appends to (L + 1) % 3 and clears (L + 2) % 3.
        // Pairs of long out-lists are expanded by the whole block.  (10^6 nodes, levels of 1 to 4 thousand
        // pairs: 1024 pairs at a time with six barriers each 30 us a level.)
        // A level with more than `handoff` pairs (0: none) and the rest of
        // the search go to the whole grid (k_resid_level); the host then
        // completes the seed.
        uint32_t *F[2] = {A.front, A.front + (uint64_t)A.n * kPairStride};
        const uint32_t par0 = resumed ? s_rcur : 0u;  // buffer of local level 0
        if (tid == 0) {
            s_fcnt[1] = s_fcnt[2] = 0;
            s_hcnt[1] = s_hcnt[2] = 0;
            if (resumed) s_hcnt[0] = 0;
        }
        if (!resumed) {
            if (tid < 64) {  // the first wave holds every instance (l <= 64)
                const uint32_t px = x * kPairStride + tid;
                const uint64_t was = tid < A.ell ? cover<kGroup>(ST, px) : kCovered;
                const bool fresh = !(was & kCovered);
                const bool any = fresh && (was & (kHasEdges | kCommitted));
                const bool big = any && (was & kLong), add = any && !big;
                const uint64_t m = __ballot(add), mb = __ballot(big), below = (1ull << tid) - 1ull;
                const uint32_t e = px | (was & kCommitted ? kHasEntry : 0u);
                if (add) s_front[0][__popcll(m & below)] = e;
                if (big) s_long[0][__popcll(mb & below)] = e;  // l <= kBlockItems
                const uint64_t g = __ballot(fresh);
                if (tid == 0) {
                    s_fcnt[0] = (uint32_t)__popcll(m);
                    s_hcnt[0] = (uint32_t)__popcll(mb);
                    s_gain = (unsigned long long)__popcll(g);
                }
            }
        } else {
            // the grid left the pending level in the queue area
            for (uint32_t e = tid; e < s_fcnt[0] && e < kSkimLdsFront; e += kSkimBlock)
                s_front[par0][e] = F[par0][e];
        }
        bool handed = false;
        const uint64_t seed_edges = A.fptr[(uint64_t)x * kPairStride + kPairStride] -
                                    A.fptr[(uint64_t)x * kPairStride];
        for (uint32_t L = 0;; ++L) {
            __syncthreads();
            const uint32_t cur = (par0 + L) & 1u, c0 = L % 3, c1 = (L + 1) % 3, c2 = (L + 2) % 3;
            const uint32_t fc = s_fcnt[c0], nh = min(s_hcnt[c0], kBlockItems);
            if (fc == 0 && nh == 0) break;
            if (handoff &&
                (fc > handoff || (L == 0 && !resumed && seed_edges > kSkimHandoffEdges))) {
                // the grid reads the level from the queue area
                if (tid < nh) st<kGroup>(A.heavy + (uint64_t)kHeavyItems * cur + tid, s_long[cur][tid]);
                for (uint32_t e = tid; e < fc && e < kSkimLdsFront; e += kSkimBlock)
                    st<kGroup>(F[cur] + e, s_front[cur][e]);
                if (tid == 0) {
                    A.ctl->pend = 1;
                    A.ctl->px = x;
                    A.ctl->rcur = cur;
                    A.ctl->rsize[0] = fc;
                    A.ctl->rsize[16] = 0;
                    A.ctl->rsize[32] = 0;
                    A.ctl->hsize[0] = nh;
                    A.ctl->hsize[16] = A.ctl->hsize[32] = 0;
                    A.ctl->rgain = s_gain;
                }
                handed = true;
                break;
            }
            if (tid == 0) {
                s_fcnt[c2] = s_hcnt[c2] = 0;
            }
            auto fin = [&](uint64_t e) { return e < kSkimLdsFront ? s_front[cur][e] : ld<kGroup>(F[cur] + e); };
            auto push = [&](const uint64_t (&was)[kResidEdges], const uint32_t (&qw)[kResidEdges]) {
                uint64_t m[kResidEdges];
                uint32_t all = 0, fresh = 0, pos = 0;
                bool add[kResidEdges];
#pragma unroll
                for (int u = 0; u < kResidEdges; ++u) {
                    add[u] = !(was[u] & kCovered) && (was[u] & (kHasEdges | kCommitted));
                    fresh += (uint32_t)__popcll(__ballot(!(was[u] & kCovered)));
                    if (add[u] && (was[u] & kLong)) {
                        const uint32_t slot = atomicAdd(&s_hcnt[c1], 1u);
                        if (slot < kBlockItems) {
                            s_long[cur ^ 1u][slot] = qw[u] | (was[u] & kCommitted ? kHasEntry : 0u);
                            add[u] = false;
                        }
                    }
                    m[u] = __ballot(add[u]);
                    all += (uint32_t)__popcll(m[u]);
                }
                if (!fresh) return;
                if (lane_id() == 0) {
                    atomicAdd(&s_gain, (unsigned long long)fresh);
                    pos = atomicAdd(&s_fcnt[c1], all);
                }
                pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)pos);
#pragma unroll
                for (int u = 0; u < kResidEdges; ++u) {
                    const uint32_t j = pos + (uint32_t)__popcll(m[u] & ((1ull << lane_id()) - 1ull));
                    pos += (uint32_t)__popcll(m[u]);
                    if (add[u]) {
                        const uint32_t e = qw[u] | (was[u] & kCommitted ? kHasEntry : 0u);
                        if (j < kSkimLdsFront) s_front[cur ^ 1u][j] = e;
                        else st<kGroup>(F[cur ^ 1u] + j, e);
                    }
                }
            };
            const uint32_t wave = tid >> 6;
            if (fc <= kSkimBlock) {
                ResidWave<1> &W = reinterpret_cast<ResidWave<1> &>(s_u.wave[wave]);
                if (64 * wave < fc)
                    resid_wave<kGroup, 1>(A, SZ, ST, 64 * wave, fc, W, fin, push);
            } else {
                for (uint32_t base = 256 * wave; base < fc; base += 4 * kSkimBlock)
                    resid_wave<kGroup, 4>(A, SZ, ST, base, fc, s_u.wave[wave], fin, push);
            }
            for (uint32_t h = 0; h < nh; ++h) {
                const uint32_t q = s_long[cur][h], pq = q & ~kHasEntry;
                const uint64_t f0 = A.fptr[pq], deg = A.fptr[pq + 1] - f0;
                for (uint64_t b = 0; b < deg; b += kResidEdges * kSkimBlock) {
                    uint32_t qw[kResidEdges];
                    uint64_t was[kResidEdges];
#pragma unroll
                    for (int u = 0; u < kResidEdges; ++u) {
                        const uint64_t t = b + u * kSkimBlock + tid;
                        qw[u] = t < deg ? A.fadj[f0 + t] * kPairStride + pq % kPairStride : 0xFFFFFFFFu;
                    }
#pragma unroll
                    for (int u = 0; u < kResidEdges; ++u)
                        was[u] = qw[u] != 0xFFFFFFFFu ? cover<kGroup>(ST, qw[u]) : kCovered;
                    push(was, qw);
                }
                if (tid < 64) {
                    const bool mine = tid == 0 && (q & kHasEntry);
                    erase_entry<kGroup>(A, SZ, mine ? q : 0u, mine ? A.idx[pq] : 0ull);
                }
            }
        }
        if (handed) break;  // uniform
        __syncthreads();
        if (tid == 0) {
            st<kGroup>(A.sel + x, 1u);
            seeds[it] = x;
            gains[it] = s_gain;
            if (gain_d) gain_d[it] = (double)s_gain / (double)A.ell;
        }
        __syncthreads();
    }
    if constexpr (kLds) {
        __syncthreads();
        for (uint32_t w = tid; w < swords; w += kSkimBlock) st<kGroup>(A.size + w, s_size[w]);
        if constexpr (kLdsState)
            for (uint32_t w = tid; w < 4 * n; w += kSkimBlock) st<kGroup>(A.state + w, ST[w]);
    }
    if (tid == 0) {
        A.ctl->cursor = s_cursor;
        A.ctl->pool_used = s_pool;
        A.ctl->done = it;
    }
}

// Level L of a round of a residual search handed over by k_skim, on the whole
// grid: frontier buffer (rcur + L) & 1 of the queue area, sizes in global
// memory.  First the level's long pairs, their edges laid end to end and split
// evenly over every workgroup, kResidBlock pairs at a time; then the others.
// Both append to level L + 1.  A launch with nothing to do returns at once.
//
// What bounds it: small levels (most of them) the chain of accesses, 7 us;
// large ones the wave with the most edges.
__global__ void __launch_bounds__(kResidBlock) k_resid_level(SkArgs A, uint32_t L) {
    __shared__ FlatShared X;
    __shared__ ResidWave<4> W[kResidBlock / 64];
    __shared__ ResidStage S;
    const uint32_t tid = threadIdx.x, lane = lane_id();
    // (none of these words is written while a level reads it)
    const uint32_t pend = A.ctl->pend, cur = (A.ctl->rcur + L) & 1u;
    const uint64_t rs = A.ctl->rsize[16 * (L % 3)], hs = A.ctl->hsize[16 * (L % 3)];
    if (pend != 1) return;
    if (tid == 0) {
        S.n = S.gain = 0;
        if (blockIdx.x == 0) {
            A.ctl->rsize[16 * ((L + 2) % 3)] = 0;  // level L + 1 appends there
            A.ctl->hsize[16 * ((L + 2) % 3)] = 0;
            A.ctl->rgain += rs >> 32;
        }
    }
    const uint64_t fc = rs & 0xFFFFFFFFu;
    const uint32_t nh = hs < kHeavyItems ? (uint32_t)hs : kHeavyItems;
    if (fc == 0 && nh == 0) return;  // uniform
    __syncthreads();
    const uint64_t half = (uint64_t)A.n * kPairStride;
    const uint32_t *Fin = A.front + cur * half;
    uint32_t *Fout = A.front + (cur ^ 1u) * half;
    unsigned long long *next = &A.ctl->rsize[16 * ((L + 1) % 3)];
    unsigned long long *hnext = &A.ctl->hsize[16 * ((L + 1) % 3)];
    const uint32_t *hin = A.heavy + (uint64_t)kHeavyItems * cur;
    uint32_t *hout = A.heavy + (uint64_t)kHeavyItems * (cur ^ 1u);
    auto fin = [&](uint64_t e) { return Fin[e]; };
    auto push = [&](const uint64_t (&was)[kResidEdges], const uint32_t (&qw)[kResidEdges]) {
        uint64_t m[kResidEdges];
        uint32_t all = 0, fresh = 0, pos = 0;
        bool add[kResidEdges];
#pragma unroll
        for (int u = 0; u < kResidEdges; ++u) {
            add[u] = !(was[u] & kCovered) && (was[u] & (kHasEdges | kCommitted));
            fresh += (uint32_t)__popcll(__ballot(!(was[u] & kCovered)));
            if (add[u] && (was[u] & kLong)) {
                const unsigned long long slot = atomicAdd(hnext, 1ull);
                if (slot < kHeavyItems) {
                    hout[slot] = qw[u] | (was[u] & kCommitted ? kHasEntry : 0u);
                    add[u] = false;
                }
            }
            m[u] = __ballot(add[u]);
            all += (uint32_t)__popcll(m[u]);
        }
        if (!fresh) return;
        if (lane == 0) {
            atomicAdd(&S.gain, fresh);
            pos = atomicAdd(&S.n, all);
        }
        pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)pos);
#pragma unroll
        for (int u = 0; u < kResidEdges; ++u) {
            const uint32_t j = pos + (uint32_t)__popcll(m[u] & ((1ull << lane) - 1ull));
            pos += (uint32_t)__popcll(m[u]);
            if (add[u]) {
                const uint32_t e = qw[u] | (was[u] & kCommitted ? kHasEntry : 0u);
                if (j < 8 * kResidBlock) S.buf[j] = e;
                else Fout[(uint32_t)atomicAdd(next, 1ull)] = e;  // stage full
            }
        }
    };
    // the stage to level L + 1 (called by all threads, after a barrier)
    auto flush = [&]() {
        const uint32_t ns = min(S.n, 8u * kResidBlock);
        if (tid == 0 && S.gain)
            S.base = atomicAdd(next, ((unsigned long long)S.gain << 32) | ns) & 0xFFFFFFFFu;
        __syncthreads();
        const unsigned long long b = S.base;
        for (uint32_t j = tid; j < ns; j += kResidBlock) Fout[b + j] = S.buf[j];
        __syncthreads();
        if (tid == 0) S.n = S.gain = 0;
        __syncthreads();
    };
    // Where the lower half of the workgroups is enough for the others, the
    // upper half takes the long pairs: two chains side by side.
    const uint32_t lb0 = fc <= (uint64_t)gridDim.x / 2 * kResidBlock ? gridDim.x / 2 : 0u;
    const uint32_t lb = blockIdx.x - lb0, lbs = gridDim.x - lb0;
    for (uint32_t h0 = 0; h0 < nh && blockIdx.x >= lb0; h0 += kResidBlock) {
        uint64_t deg = 0, f0 = 0;
        uint32_t q = 0;
        if (h0 + tid < nh) {
            q = hin[h0 + tid];
            f0 = A.fptr[q & ~kHasEntry];
            deg = A.fptr[(q & ~kHasEntry) + 1] - f0;
        }
        uint64_t tot;
        const uint64_t e = block_excl_scan<kResidBlock>(deg, X.wsum, tot);
        X.ex[tid] = e;
        X.q[tid] = q % kPairStride;
        X.f0[tid] = f0;
        if (tid == 0) X.ex[kResidBlock] = tot;
        __syncthreads();
        // one workgroup erases the index entries
        if (lb == (h0 / kResidBlock) % lbs)
            erase_entry<kAgent>(A, A.size, q, q & kHasEntry ? A.idx[q & ~kHasEntry] : 0ull);
        const uint64_t a = tot * lb / lbs, b = tot * (lb + 1) / lbs;
        for (uint64_t base = a; base < b; base += kResidEdges * kResidBlock) {
            uint32_t qw[kResidEdges];
            bool in[kResidEdges];
            uint64_t was[kResidEdges];
#pragma unroll
            for (int u = 0; u < kResidEdges; ++u) {
                const uint64_t t = base + u * kResidBlock + tid;
                in[u] = t < b;
                qw[u] = 0;
                if (in[u]) {
                    const uint32_t r = run_of<kResidBlock>(X.ex, t);
                    qw[u] = A.fadj[X.f0[r] + (t - X.ex[r])] * kPairStride + X.q[r];
                }
            }
#pragma unroll
            for (int u = 0; u < kResidEdges; ++u)
                was[u] = in[u] ? cover<kAgent>(A.state, qw[u]) : kCovered;
            push(was, qw);
            __syncthreads();
            const bool full = S.n > 4 * kResidBlock;
            __syncthreads();  // every thread has read S.n: the test below is uniform
            if (full) flush();
        }
        __syncthreads();  // X is reused
    }
    // four pairs per lane where there is one for every lane of the grid
    const bool many = fc > (uint64_t)kResidGrid * kResidBlock;
    const uint64_t chunk = many ? 4 * kResidBlock : kResidBlock;
    for (uint64_t base = blockIdx.x * chunk; base < fc; base += gridDim.x * chunk) {
        const uint32_t wave = tid >> 6;
        if (many)
            resid_wave<kAgent, 4>(A, A.size, A.state, base + 256 * wave, fc, W[wave], fin, push);
        else
            resid_wave<kAgent, 1>(A, A.size, A.state, base + 64 * wave, fc,
                                  reinterpret_cast<ResidWave<1> &>(W[wave]), fin, push);
        __syncthreads();
        const bool full = S.n > 4 * kResidBlock;
        __syncthreads();
        if (full) flush();
    }
    __syncthreads();
    flush();
}

// The end of a round: a search that has ended completes its seed, one that has
// become small goes back to k_skim, any other goes on in the next round.
__global__ void k_resid_end(SkArgs A, uint32_t *seeds, uint64_t *gains, double *gain_d) {
    SkCtl *c = A.ctl;
    if (c->pend != 1) return;
    const uint32_t f = (uint32_t)c->rsize[0];
    if (c->hsize[0] == 0 && f == 0) {
        const uint32_t x = c->px, it = c->done;
        const unsigned long long g = c->rgain + (c->rsize[0] >> 32);
        A.sel[x] = 1u;
        seeds[it] = x;
        gains[it] = g;
        if (gain_d) gain_d[it] = (double)g / (double)A.ell;
        c->pend = 0;
        c->done = it + 1;
    } else if (c->hsize[0] == 0 && f <= kSkimHandBack) {
        c->pend = 2;
    }
}

// State words of a new run: every pair's out-list bits.
__global__ void k_state_init(uint32_t n, const uint64_t *fptr, uint64_t *state) {
    const uint64_t npairs = (uint64_t)n * kPairStride;
    for (uint64_t p = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; p < npairs;
         p += (uint64_t)gridDim.x * blockDim.x) {  // whole waves: 64 pairs are a node's
        const uint64_t deg = fptr[p + 1] - fptr[p];
        const uint64_t some = __ballot(deg > 0), more = __ballot(deg > kLongEdges);
        const uint32_t part = (uint32_t)(p % 64);
        if (part < 4)
            state[p / 64 * 4 + part] = ((some >> (16 * part)) & 0xFFFFu) << 32 |
                                       ((more >> (16 * part)) & 0xFFFFu) << 48;
    }
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
constexpr int kTailWaves = 4;
constexpr int kTailPairBlock = 64 * kTailWaves;
constexpr int kTailBlocks = kTailChunk + 15;       // 16-cell blocks of a that a chunk meets
constexpr int kTailPad = 18;
typedef double v4d __attribute__((ext_vector_type(4)));

__global__ void __launch_bounds__(kTailPairBlock) k_tail_pair(const double *in, double *out,
                                                              uint32_t bins, TailLevel L,
                                                              double *partial, uint32_t *arrived) {
    __shared__ double s_a[kTailBlocks * kTailPad];  // blocks of 16, padded: no bank conflicts
    __shared__ double s_b[16 * kTailChunk + 16];
    __shared__ double s_red[kTailWaves][kTailTile];
    __shared__ uint32_t s_last;
    const int64_t W = (int64_t)bins + 1;
    const int tid = (int)threadIdx.x, wave = tid / 64, lane = tid % 64;
    const int li = lane % 16, lk = lane / 16;
    for (uint64_t item = blockIdx.x; item < L.items; item += gridDim.x) {
        const TailItem work = tail_item(L, item);
        const uint64_t p = work.pair;
        uint32_t tile = work.tile;
        int more = work.more;
        if (p >= L.pairs) {  // the odd last row
            const int64_t j = (int64_t)tile * kTailTile + tid;
            if (j < W) out[p * W + j] = in[2 * p * W + j];
            continue;
        }
        for (;; tile = (uint32_t)more, more = -1) {
        const int64_t c0 = 16 * (int64_t)tile;
        const int64_t d0 = (int64_t)work.part * L.part;
        const int64_t d1 = d0 + L.part < c0 + 16 ? d0 + L.part : c0 + 16;
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
        if (work.nparts > 1) {
            // item numbers of a tile's parts are consecutive
            // (agent-scope stores and loads reach the memory all XCDs see, so
            // no fence has to write back or invalidate a whole cache; the
            // stores have arrived before the counter is touched)
            st<kAgent>(partial + item * kTailTile + tid, v);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0);
            __syncthreads();
            if (tid == 0) {
                uint32_t *cnt = arrived + p * L.tiles + tile;
                const uint32_t before = atomicAdd(cnt, 1u);
                s_last = before + 1 == work.nparts;
                if (s_last) atomicExch(cnt, 0u);  // ready for the next level
            }
            __syncthreads();
            if (!s_last) break;  // uniform
            const double *first = partial + (item - work.part) * kTailTile;
            v = 0.0;
            for (uint32_t q = 0; q < work.nparts; ++q)
                v += ld<kAgent>(first + (uint64_t)q * kTailTile + tid);
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
    for (uint32_t rows = s; rows > 1; rows = (rows + 1) / 2) {
        const TailLevel L = tail_level(rows, W);
        if (rows == 2) out = tail;
        k_tail_pair<<<(unsigned)std::min<uint64_t>(L.items, 1u << 20), kTailPairBlock, 0, hs>>>(
            in, out, bins, L, T.partial, T.arrived);
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
    bool running = false;     // a call is under way, or ended in an error
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

// The next step of the pairs' order by rank.  An allocation may fail anywhere
// in it and the state goes on being used: what the order holds, the rank it
// goes on from and the next step's length change together, once the step's
// pairs are in place.
void greedy_extend_order(skim_greedy_state *st, hipStream_t s) {
    SkArgs &A = st->args;
    const uint64_t left = A.nsrc - A.ordered;
    const bool whole = A.nsrc <= kOrderWhole;
    Arena T(s);
    uint64_t count = A.nsrc, rank_next = st->rank_next, order_step = st->order_step;
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
        if (count > left || (last && count != left)) {  // `order` has room for all ranks, once
            set_error("%llu pairs in a step of the rank order, %llu left",
                      (unsigned long long)count, (unsigned long long)left);
            throw Fail{SKIM_EDEVICE};
        }
        keys = T.alloc<uint64_t>(count ? count : 1);
        vals = T.alloc<uint32_t>(count ? count : 1);
        k_rank_take<<<kOrderGrid, kOrderBlock, 0, s>>>(A.n, A.ell, A.seed, r0, r1, counts,
                                                       totals + 1, keys, vals);
        SKIM_LAUNCH_CHECK();
        rank_next = r1 + 1;
        order_step *= 4;
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
    st->rank_next = rank_next;
    st->order_step = order_step;
}

skim_greedy_state *greedy_create(const skim_graph *g, uint32_t ell, uint32_t k, uint64_t seed,
                                        hipStream_t s) {
    SKIM_REQUIRE(ell >= 1 && ell <= 64, "l must be in [1, 64]");
    // sizes and batch counters are 16-bit halves of words
    SKIM_REQUIRE(k >= 2 && k <= 65535, "k must be in [2, 65535]");
    SKIM_REQUIRE(g != nullptr, "graph is NULL");
    if ((uint64_t)g->n > (1ull << 22)) {
        set_error("skim_greedy supports n <= 4194304 (its searches take 2.5 KiB per node, at 32-bit "
                  "offsets)");
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
    A.state = M.alloc<uint64_t>(npairs / 16);
    const uint64_t cwords = size_words(n);
    A.size = M.alloc<uint32_t>(cwords);
    A.sel = M.alloc<uint32_t>(n);
    A.idx = M.alloc<uint64_t>(npairs);
    A.heavy = M.alloc<uint32_t>(2 * (uint64_t)kHeavyItems);
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
    k_state_init<<<grid_for(npairs, 256, 8192), 256, 0, s>>>(n, A.fptr, A.state);
    SKIM_LAUNCH_CHECK();
    fill_u32(A.size, 0, cwords, s);
    fill_u32(A.sel, 0, n, s);
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
    const uint32_t before = st->selected;
    uint32_t done = 0;
    int growths = 0, rounds = 0;
    bool begin = true;
    // a call that failed (memory) left its count and its request behind
    if (st->running) fill_u32(&A.ctl->done, 0, 2, s);
    st->running = true;
    auto skim = [&] {
        auto kernel = A.n <= kSkimStateNodes ? k_skim<true, true>
                      : A.n <= kSkimLdsNodes ? k_skim<true, false>
                                             : k_skim<false, false>;
        kernel<<<1, kSkimBlock, 0, s>>>(A, s_goal, begin, kSkimHandoff, seeds, gains, gain_d,
                                        A.rec_tau + before, A.rec_second + before);
        SKIM_LAUNCH_CHECK();
        begin = false;
    };
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
        if (rounds == 0) skim();
        // once a search has gone to the grid, rounds of levels and the loop's
        // next launch are enqueued together: each finds out on the device
        // what there is to do (reading the control block between them left
        // the device idle 25 us each time)
        for (int r = 0; r < rounds; ++r) {
            for (uint32_t L = 0; L < kRoundLevels; ++L) {
                k_resid_level<<<kResidGrid, kResidBlock, 0, s>>>(A, L);
                SKIM_LAUNCH_CHECK();
            }
            k_resid_end<<<1, 1, 0, s>>>(A, seeds, gains, gain_d);
            SKIM_LAUNCH_CHECK();
            skim();
        }
        SkCtl c;
        read_back(&c, A.ctl, sizeof c, s);
        const bool moved = c.done > done || c.cursor > st->cursor;
        st->cursor = c.cursor;
        done = c.done;
        st->selected = before + done;
        rounds = 0;
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
            rounds = kRounds;
        } else if (done < s_goal && !moved) {
            set_error("SKIM stopped early");
            throw Fail{SKIM_EDEVICE};
        }
    }
    st->running = false;
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

// A saved state holds a word per pair, 1 if it is covered, and the index word
// of every committed pair that is not covered, 0 for the others.
// Made kImagePairs pairs at a time (a multiple of 64).
constexpr uint64_t kImagePairs = 1ull << 22;
__global__ void k_state_unpack(SkArgs A, uint64_t p0, uint64_t count, uint32_t *covered,
                               uint64_t *idx) {
    for (uint64_t t = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; t < count;
         t += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t p = p0 + t;
        const uint64_t w = A.state[p / 16] >> (p % 16);
        covered[t] = w & kCovered ? 1u : 0u;
        idx[t] = (w & (kCovered | kCommitted)) == kCommitted ? A.idx[p] : 0ull;
    }
}
__global__ void k_state_pack(SkArgs A, uint64_t p0, uint64_t count, const uint32_t *covered) {
    for (uint64_t w = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; w < count / 16;
         w += (uint64_t)gridDim.x * blockDim.x) {
        uint64_t bits = 0;
        for (uint32_t j = 0; j < 16; ++j)
            bits |= (covered[16 * w + j] ? kCovered << j : 0u) |
                    (A.idx[p0 + 16 * w + j] ? kCommitted << j : 0u);
        A.state[p0 / 16 + w] |= bits;
    }
}

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
        skim::Arena T(hs);
        const uint64_t chunk = std::min(npairs, skim::kImagePairs);
        uint32_t *covered = T.alloc<uint32_t>(chunk);
        uint64_t *idx = T.alloc<uint64_t>(chunk);
        for (uint64_t p0 = 0; p0 < npairs; p0 += chunk) {
            const uint64_t c1 = std::min(chunk, npairs - p0);
            skim::k_state_unpack<<<skim::grid_for(c1, 256, 8192), 256, 0, hs>>>(A, p0, c1, covered,
                                                                              idx);
            SKIM_LAUNCH_CHECK();
            SKIM_HIP(hipMemcpyAsync(b + L.covered + 4 * p0, covered, 4 * c1, hipMemcpyDeviceToHost, hs));
            SKIM_HIP(hipMemcpyAsync(b + L.idx + 8 * p0, idx, 8 * c1, hipMemcpyDeviceToHost, hs));
        }
        const struct {
            uint64_t off;
            const void *src;
            uint64_t len;
        } parts[] = {{L.size, A.size, cwords * 4},
                     {L.sel, A.sel, (uint64_t)state->n * 4},
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
        } parts[] = {{A.size, L.size, cwords * 4},
                     {A.sel, L.sel, (uint64_t)h.n * 4},
                     {A.idx, L.idx, npairs * 8},
                     {A.pool, L.pool, h.pool_used * 4},
                     {A.rec_tau, L.tau, h.selected * 8},
                     {A.rec_second, L.second, h.selected * 4}};
        for (const auto &pt : parts)
            if (pt.len)
                SKIM_HIP(hipMemcpyAsync(pt.dst, b + pt.off, pt.len, hipMemcpyHostToDevice, hs));
        skim::Arena T(hs);
        const uint64_t chunk = std::min(npairs, skim::kImagePairs);
        uint32_t *covered = T.alloc<uint32_t>(chunk);
        for (uint64_t p0 = 0; p0 < npairs; p0 += chunk) {
            const uint64_t c1 = std::min(chunk, npairs - p0);
            SKIM_HIP(hipMemcpyAsync(covered, b + L.covered + 4 * p0, 4 * c1, hipMemcpyHostToDevice, hs));
            skim::k_state_pack<<<skim::grid_for(c1 / 16, 256, 8192), 256, 0, hs>>>(A, p0, c1, covered);
            SKIM_LAUNCH_CHECK();
        }
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
