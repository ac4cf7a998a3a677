// Persistent search for runs of small levels (single root).
//
// A level whose frontier holds a few thousand vertices does almost no work,
// but launching its kernels (degree scan, expansion, bookkeeping) costs a
// dispatch gap of several microseconds each; a 4096 x 4096 grid has
// thousands of such levels.  One persistent kernel of a few dozen
// workgroups runs them back to back instead.
//
// Such levels are bound by the chain of dependent memory round trips, so the
// loop is built around that chain:
//   - one XCD: of the launch's workgroups only every eighth takes part, and
//     workgroups are dealt to the eight XCDs in turn, so the ones that do
//     share one L2.  They compare their XCC ids when they start: when all are
//     equal, claims and barrier words are atomics and stores of that L2
//     (workgroup scope), a fraction of the latency of the device-scope ones,
//     and no barrier writes back or invalidates the L2; otherwise the same
//     loop runs at device scope;
//   - the frontier stays in the LDS of the workgroup that found it.  The next
//     queue in memory is written only when the frontier is dealt out anew (a
//     workgroup's share overflowed or became a multiple of the mean) and when
//     the kernel hands the search back;
//   - one barrier per level, which orders nothing but the claims: a workgroup
//     arrives as soon as its claims have returned, then loads the row starts
//     and the first neighbours of the vertices it found, and only then waits.
//     Each workgroup arrives with one store to its own slot, which also holds
//     its share of the new frontier, and reads all slots with one load per
//     lane, so the sizes arrive with the barrier;
//   - graphs whose largest degree is at most kRowEdges (lattices) take one lane
//     per edge; others map edges to threads by binary search in the
//     share's degree prefix sum (Section 3.4), and check the level's edge
//     count and largest degree in a second set of slots.
// One search, against one device-scope counter barrier and queue reservation
// per level: 256 x 256 grid (378 levels) 2.1-2.7 -> 0.69 ms, 4096 x 4096 grid
// (5799 levels) 46.8 -> 22.8 ms; the loop's launches of an R-MAT 16 search
// 82 -> 43 us.
//
// On levels of few edges claims go straight to the atomicOr of Algorithm 3
// (a plain-read probe would add one dependent round trip).  Levels with more
// probe first, and collect the ids below kHotIds (under degree order the ones
// most edges point at) in LDS, to be claimed a bitmap word at a time.  Where
// edges do not meet, on symmetric graphs without hubs and with more ids than
// those, they claim directly at any size.  Winners write level and parent; the
// bitmap of the level before (vis_old) is left
// behind, the host brings it up to date before it next drives a level itself.
//
// The kernel hands the search back to the host when the next frontier, its
// edge count or its largest degree exceeds the limits the host passes, and
// ends the search when a frontier is empty.  Every wait is bounded.  The
// workgroups start together or not at all: one that has waited too long for
// the others (the GPU is held by other work) calls the launch off, and the
// host runs the level itself.  A wait inside the loop that does not end sets
// ctrl->err and every workgroup leaves.
#include "bfs_internal.h"
#include "wave_ops.h"

namespace bfsmi {

constexpr int kSW = 512;           // threads per workgroup (8 waves)
constexpr int kSmallEPT = 2;
constexpr int kSmallTile = kSW * kSmallEPT;
// Frontier entries per workgroup and pass.  (2048 would hold every frontier that
// the loop takes, and frontiers from 32K vertices on would not be dealt out
// again: 4,096 hubs of 15 leaves 178 -> 153 us.  But with 58 KB of LDS instead of 34
// the workgroups of concurrent searches wait for each other: twelve threads
// searching R-MAT 16 80 -> 165 us a search.)
constexpr int kSmallStage = 1024;
constexpr int kStagePer = kSmallStage / kSW;
constexpr int kRowEdges = 4;       // rows of at most this many edges: one lane per edge
constexpr int kRowStep = kSmallTile / kRowEdges;  // such rows per step
constexpr uint32_t kStartCap = 1u << 14;  // polls before a launch is called off
constexpr uint32_t kSpinCap = 1u << 23;
// Levels with more edges merge the hot ids' claims (at 2^9, 2^11, 2^13 and never:
// R-MAT 2^9 65, 65, 115, 115 us, 2^14 of edge factor 4 111, 112, 134, 607, 30 x 30
// x 30 lattice 267, 262, 276, 279).
constexpr int64_t kMergeEdges = 1 << 11;
// Lattices (their rows point at few ids a line: 512 x 512 from 2^11 edges on 1,475
// us, from 2^16 on 1,245) do from here on, or where a level points at half of
// the ids (ternary tree of 9,841 ids 152 -> 90 us).
constexpr int64_t kRowMergeEdges = 1 << 16;
constexpr int kHotIds = 1 << 16;  // ids below this are merged
// Edge counts saturate, per thread and per share, above every limit the host
// passes (at most 8192 edges per workgroup).
constexpr int64_t kDegSat = 1 << 22, kEdgeSat = 1 << 24;
static_assert((int64_t)kSmallMaxWGs * 8192 < kDegSat, "a saturated count is over the limit");

// Barrier words, one per workgroup, in two sets used in turn: a workgroup
// writes set k mod 2 again only after every other has arrived at barrier
// k + 1, which they do after reading set k mod 2.
struct SmallSlots {
    uint64_t cnt[2][kSmallMaxWGs];  // epoch << 32 | overflow << 31 | vertices found
    uint64_t deg[2][kSmallMaxWGs];  // epoch << 32 | a degree is over the limit << 31 | edges
};
static_assert(sizeof(SmallSlots) <= kSummaryMaxWords * 4, "the slots lie in the summary's words");

struct SmallLds {
    int32_t cum[kSmallStage + 1];
    int32_t uid[kSmallStage];
    int64_t base[kSmallStage];
    uint16_t map[kSmallTile];
    uint32_t hot[kHotIds / 32];  // merge levels: hot ids this workgroup's edges point at
    int32_t nv[2][kSmallStage];  // vertices found, this level's and the last one's
    int32_t wave[kSW / 64];
    int32_t dmax[kSW / 64];
    uint32_t cnt[2];   // vertices found at the level, by level mod 2
    // of the last barrier: total, bits (some flag bit set; some share above
    // twice the mean; the wait ended), sum before this workgroup
    int32_t sum, bits, pre;
};
constexpr int kBarAny = 1, kBarSkew = 2, kBarOk = 4;

template <bool L>
__device__ __forceinline__ uint32_t claim_or(uint32_t* p, uint32_t m)
{
    if constexpr (L)
        return __hip_atomic_fetch_or(p, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else
        return __hip_atomic_fetch_or(p, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <bool L, typename T>
__device__ __forceinline__ void scoped_store(T* p, T x)
{
    if constexpr (L)
        __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else
        __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The launch's result, visible to the workgroup that leaves last.
__device__ __forceinline__ void report(Ctrl* ctrl, int32_t done, int32_t qlen, int32_t level,
                                       int32_t steps, int64_t reached, int32_t levels)
{
    scoped_store<false>(&ctrl->done, done);
    scoped_store<false>(&ctrl->qlen, qlen);
    scoped_store<false>(&ctrl->level, level);
    scoped_store<false>(&ctrl->steps, steps);
    scoped_store<false>(&ctrl->reached, reached);
    scoped_store<false>(&ctrl->levels, levels);
}

// Queue entries are read past the L1: other workgroups write them during the
// launch, and no barrier invalidates it.  (Also applied to shares in LDS.)
__device__ __forceinline__ int32_t queue_load(const int32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits until all N slots carry the epoch, then sums their low 31 bits into
// S.sum and S.pre; S.bits as above (skew: a share of more than skew_min that
// is more than twice the mean).  Returns {sum, bits}, uniform.  Every thread
// calls it; the last wave, which has the least to load, polls.
__device__ __forceinline__ int2 wait_slots(const uint64_t* slots, uint32_t epoch, int N, int w,
                                           int32_t skew_min, SmallLds& S)
{
    if (threadIdx.x >= kSW - 64) {
        const int lane = __lane_id();
        uint64_t x = (uint64_t)epoch << 32;
        uint32_t spins = 0;
        bool ok = true;
        while (true) {
            // agent scope: read past the L1
            if (lane < N) x = __hip_atomic_load(slots + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (__all((uint32_t)(x >> 32) == epoch)) break;
            if (++spins > kSpinCap) {
                ok = false;
                break;
            }
        }
        const int32_t c = (int32_t)((uint32_t)x & 0x7fffffffu);
        const int32_t inc = wave_inclusive_scan_dpp(c);
        const int32_t sum = __builtin_amdgcn_readlane(inc, 63);
        const uint64_t any = __ballot(((uint32_t)x >> 31) != 0);
        const uint64_t skew = __ballot(c > skew_min && (int64_t)c * N > 2 * (int64_t)sum);
        if (lane == w) S.pre = inc - c;
        if (lane == 0) {
            S.sum = sum;
            S.bits = (any ? kBarAny : 0) | (skew ? kBarSkew : 0) | (ok ? kBarOk : 0);
        }
    }
    __syncthreads();
    return make_int2(__builtin_amdgcn_readfirstlane(S.sum), __builtin_amdgcn_readfirstlane(S.bits));
}

// Appends the winners among a wave's NE edges per lane to the workgroup's
// share; those that do not fit go to the queue in memory, behind one
// reservation per wave.
template <bool L, int NE>
__device__ __forceinline__ void keep_winners(const int32_t (&vv)[NE], const bool (&win)[NE],
                                             int32_t V, int32_t* nv, uint32_t* cnt, int32_t* __restrict__ Qn,
                                             uint32_t* __restrict__ spill, uint32_t spill0,
                                             Ctrl* __restrict__ ctrl)
{
    uint64_t mask[NE];
    uint32_t total = 0;
#pragma unroll
    for (int j = 0; j < NE; ++j) {
        mask[j] = __ballot(win[j]);
        total += (uint32_t)__popcll(mask[j]);
    }
    if (!total) return;  // uniform over the wave
    uint32_t pos0 = 0;
    if (__lane_id() == 0) pos0 = atomicAdd(cnt, total);
    pos0 = __builtin_amdgcn_readfirstlane(pos0);
    const uint32_t over0 = pos0 > kSmallStage ? pos0 : kSmallStage;  // first position that spills
    uint32_t q0 = 0;
    if (pos0 + total > over0) {
        if (__lane_id() == 0) q0 = atomicAdd(spill, pos0 + total - over0);
        q0 = __builtin_amdgcn_readfirstlane(q0) - spill0;
    }
    uint32_t base = pos0;
#pragma unroll
    for (int j = 0; j < NE; ++j) {
        if (win[j]) {
            const int32_t v = vv[j];
            const uint32_t pos = base + lanes_below(mask[j]);
            if (pos < kSmallStage) {
                nv[pos] = v;
            } else {
                const uint32_t q = q0 + (pos - over0);
                if (q < (uint32_t)V) scoped_store<L>(Qn + q, v);
                else scoped_store<false>(&ctrl->err, 5);
            }
        }
        base += (uint32_t)__popcll(mask[j]);
    }
}

// Where few probes meet (rows that may meet at a vertex, but no hubs seen), they
// read the bitmap through the L1: past it, a level of 250K edges took 60 us more
// (directed, 2^18 ids of mean degree 8: 350 -> 309 us; graphs with hubs lose 2 to 4 us
// by it).  Its words are dropped from the L1 at a merge level's end, by the wave
// that has the least to do while the others arrive: a later level must not take
// an id for unvisited, since it stores the parents of those.
__device__ __forceinline__ void drop_l1()
{
    if (threadIdx.x >= kSW - 64) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
}

// Claims of one step: the atomicOr on every edge.  At a merge level an edge
// first reads the bitmap; one to an unvisited hot id is noted in hot (the
// first of the workgroup stores the parent: whichever store remains, it names
// a frontier neighbour) and claimed by merge_hot.
// (Loads are unconditional, of valid ids, here and below: behind a branch
// the compiler waits for each before it issues the next.)
template <bool L, int NE>
__device__ __forceinline__ void claim_edges(const int32_t (&vv)[NE], const int32_t (&uu)[NE],
                                            const bool (&ok)[NE], bool merge, bool l1,
                                            uint32_t* __restrict__ vis,
                                            int32_t* __restrict__ parent, uint32_t* hot,
                                            bool (&win)[NE])
{
    uint32_t old[NE];
#pragma unroll
    for (int j = 0; j < NE; ++j) old[j] = ok[j] ? 0u : ~0u;
    if (merge) {
        if (l1) {  // (uniform)
#pragma unroll
            for (int j = 0; j < NE; ++j)
                old[j] |= __hip_atomic_load(vis + (vv[j] >> 5), __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_WAVEFRONT);
        } else {
#pragma unroll
            for (int j = 0; j < NE; ++j)
                old[j] |= __hip_atomic_load(vis + (vv[j] >> 5), __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
        }
#pragma unroll
        for (int j = 0; j < NE; ++j) {
            const uint32_t bit = 1u << (vv[j] & 31);
            if (!(old[j] & bit) && vv[j] < kHotIds) {
                old[j] = ~0u;
                if (!(atomicOr(&hot[vv[j] >> 5], bit) & bit) && parent) parent[vv[j]] = uu[j];
            }
        }
    }
#pragma unroll
    for (int j = 0; j < NE; ++j)
        if (!(old[j] & (1u << (vv[j] & 31))))
            old[j] = claim_or<L>(vis + (vv[j] >> 5), 1u << (vv[j] & 31));
#pragma unroll
    for (int j = 0; j < NE; ++j) win[j] = !(old[j] & (1u << (vv[j] & 31)));
}

// End of a merge level: the noted ids are claimed a bitmap word at a time,
// consecutive words by consecutive lanes.  Hub rows point at the same few
// lines of the bitmap, whose atomics an L2 takes one after the other: a level
// of R-MAT 12 with 32K edges (4 lines) took 58 us of single-bit claims.
template <bool L>
__device__ __forceinline__ void merge_hot(uint32_t* hot, int32_t lvl, int32_t V,
                                          uint32_t* __restrict__ vis, int32_t* __restrict__ level,
                                          int32_t* nv, uint32_t* cnt, int32_t* __restrict__ Qn,
                                          uint32_t* __restrict__ spill, uint32_t spill0,
                                          Ctrl* __restrict__ ctrl)
{
    constexpr int PER = kHotIds / 32 / kSW;
    uint32_t x[PER], old[PER];
#pragma unroll
    for (int m = 0; m < PER; ++m) {
        x[m] = hot[m * kSW + threadIdx.x];
        old[m] = 0;
        if (x[m]) old[m] = claim_or<L>(vis + m * kSW + threadIdx.x, x[m]);
    }
#pragma unroll
    for (int m = 0; m < PER; ++m) x[m] &= ~old[m];
#pragma unroll
    for (int m = 0; m < PER; ++m) {
        const int32_t c = __popc(x[m]);
        const int32_t inc = wave_inclusive_scan_dpp(c);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane(inc, 63);
        if (!total) continue;  // uniform over the wave
        uint32_t pos0 = 0, q0 = 0;
        if (__lane_id() == 0) pos0 = atomicAdd(cnt, total);
        pos0 = __builtin_amdgcn_readfirstlane(pos0);
        const uint32_t over0 = pos0 > kSmallStage ? pos0 : kSmallStage;
        if (pos0 + total > over0) {
            if (__lane_id() == 0) q0 = atomicAdd(spill, pos0 + total - over0);
            q0 = __builtin_amdgcn_readfirstlane(q0) - spill0;
        }
        uint32_t pos = pos0 + (uint32_t)(inc - c);
        for (uint32_t b = x[m]; b; b &= b - 1, ++pos) {
            const int32_t v = (m * kSW + (int32_t)threadIdx.x) * 32 + __builtin_ctz(b);
            if (pos < kSmallStage) {
                nv[pos] = v;
            } else {
                const uint32_t q = q0 + (pos - over0);
                if (q < (uint32_t)V) scoped_store<L>(Qn + q, v);
                else scoped_store<false>(&ctrl->err, 5);
            }
            level[v] = lvl;
        }
    }
}

// Maps the tile's slots of the staged share (n entries, R edges) to entries
// and loads their neighbours.
__device__ __forceinline__ void map_small_tile(SmallLds& S, int32_t n, int32_t R, int32_t e0,
                                               const int32_t* __restrict__ col,
                                               int32_t (&vv)[kSmallEPT], int32_t (&uu)[kSmallEPT],
                                               bool (&ok)[kSmallEPT])
{
    const int t = threadIdx.x;
    const int32_t n_e = R - e0 < kSmallTile ? R - e0 : kSmallTile;
    // slots sl0, sl0 + 1 of this thread: entry = max{i : cum[i] <= slot}
    const int32_t sl0 = e0 + t * kSmallEPT;
    if (t * kSmallEPT < n_e) {
        int32_t lo = 0;
        for (int32_t st = 1 << (31 - __builtin_clz(n)); st > 0; st >>= 1) {
            const int32_t x = lo + st;
            if (x < n && S.cum[x] <= sl0) lo = x;
        }
        int32_t i = lo;
#pragma unroll
        for (int j = 0; j < kSmallEPT; ++j) {
            const int32_t sl = sl0 + j;
            if (sl - e0 < n_e) {
                while (i + 1 < n && S.cum[i + 1] <= sl) ++i;
                S.map[sl - e0] = (uint16_t)i;
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSmallEPT; ++j) {
        const int32_t sl = t + j * kSW;
        ok[j] = sl < n_e;
        const int32_t sc = ok[j] ? sl : n_e - 1;
        const int32_t i = S.map[sc];
        uu[j] = S.uid[i];
        vv[j] = col[S.base[i] + e0 + sc];
    }
}

// Stages entries ids[0..n), n <= kSmallStage, kStagePer consecutive ones per thread:
// row starts, caller ids and the prefix sum of the degrees.  Returns the
// share's edges (saturated: over the limits the prefix sums mean nothing);
// S.dmax gets the largest degree of each wave.
__device__ __forceinline__ int32_t stage_share(SmallLds& S, const int32_t* __restrict__ ids, int32_t n,
                                               const int64_t* __restrict__ off,
                                               const int32_t* __restrict__ orig)
{
    const int t = threadIdx.x;
    if (n == 0) {  // uniform
        if (t < kSW / 64) S.dmax[t] = 0;
        __syncthreads();
        return 0;
    }
    int64_t a[kStagePer], sum = 0;
    int32_t d[kStagePer], id[kStagePer];
    int32_t mx = 0;
#pragma unroll
    for (int m = 0; m < kStagePer; ++m) {
        const int32_t i = t * kStagePer + m;
        const int32_t u = queue_load(ids + (i < n ? i : n - 1));
        a[m] = off[u];
        const int64_t dd = off[u + 1] - a[m];
        d[m] = i < n ? (int32_t)(dd < kDegSat ? dd : kDegSat) : 0;
        id[m] = orig ? orig[u] : u;
    }
#pragma unroll
    for (int m = 0; m < kStagePer; ++m) {
        sum += d[m];
        mx = d[m] > mx ? d[m] : mx;
    }
    const int32_t tot = (int32_t)(sum < kDegSat ? sum : kDegSat);
    const int32_t inc = wave_inclusive_scan_dpp(tot);
    const uint64_t big = __ballot(mx > 0);
    if (big)  // uniform over the wave
        for (int o = 32; o >= 1; o >>= 1) {
            const int32_t m2 = __shfl_xor(mx, o, 64);
            mx = m2 > mx ? m2 : mx;
        }
    if ((t & 63) == 63) S.wave[t >> 6] = inc;
    if ((t & 63) == 0) S.dmax[t >> 6] = mx;
    __syncthreads();
    int32_t c = inc - tot, R = 0;
#pragma unroll
    for (int k = 0; k < kSW / 64; ++k) {
        const int32_t x = S.wave[k];
        if (k < (t >> 6)) c += x;
        R += x;
    }
#pragma unroll
    for (int m = 0; m < kStagePer; ++m) {
        const int32_t i = t * kStagePer + m;
        if (i < n) {
            S.cum[i] = c;
            S.uid[i] = id[m];
            S.base[i] = a[m] - c;
        }
        c += d[m];
    }
    if (t == 0) S.cum[n] = R;
    __syncthreads();
    return R;
}

// Edges and largest degree of this workgroup's slice of Q, as a deg slot's
// low half (every thread gets it).
__device__ __forceinline__ uint32_t slice_limits(SmallLds& S, const int32_t* __restrict__ Q,
                                                 int64_t k0, int64_t k1,
                                                 const int64_t* __restrict__ off, int32_t dlimit)
{
    const int t = threadIdx.x;
    int64_t sum = 0;
    int32_t over = 0;
    for (int64_t k = k0 + t; k < k1; k += kSW) {
        const int32_t u = queue_load(Q + k);
        const int64_t d = off[u + 1] - off[u];
        sum += d;
        over |= d > dlimit;
    }
    int32_t s = (int32_t)(sum < kDegSat ? sum : kDegSat);
    s = __builtin_amdgcn_readlane(wave_inclusive_scan_dpp(s), 63);
    const uint64_t any = __ballot(over);
    if ((t & 63) == 0) {
        S.wave[t >> 6] = s;
        S.dmax[t >> 6] = any != 0;
    }
    __syncthreads();
    int64_t tot = 0;
    uint32_t o = 0;
#pragma unroll
    for (int k = 0; k < kSW / 64; ++k) {
        tot += S.wave[k];
        o |= (uint32_t)S.dmax[k];
    }
    __syncthreads();
    return (uint32_t)(tot < kEdgeSat ? tot : kEdgeSat) | (o << 31);
}

// The levels; every workgroup returns from it exactly once.  deg slot set 1
// holds epoch 1, the limits of the first frontier (Qa[0 .. qlen0)).  ROWS: one
// lane per edge, in a body of its own (what the other form does between two
// levels cost the 256 x 256 grid 3% as branches of one body: 620 -> 641 us, apart
// 609).
template <bool L, bool ROWS>
__device__ __forceinline__ void small_levels_body(
    SmallLds& S, int32_t V, const int64_t* __restrict__ off, const int32_t* __restrict__ col,
    const int32_t* __restrict__ orig, uint32_t* __restrict__ vis,
    int32_t* __restrict__ Qa, int32_t* __restrict__ Qb, int32_t* __restrict__ level,
    int32_t* __restrict__ parent, SmallSync* __restrict__ sy, SmallSlots* __restrict__ slots,
    Ctrl* __restrict__ ctrl, int N, int w, int32_t qlen0, int32_t lvl0, int32_t qlimit,
    int64_t rlimit, int32_t dlimit, int32_t maxdeg, HubRule hub)
{
    const int t = threadIdx.x;
    uint32_t ep_cnt = 0, ep_deg = 1;
    int32_t qlen = qlen0, lvl = lvl0, step = 0, par = 0, code = 0;
    int64_t my_edges = 0, reached = 0;

    int2 bar = wait_slots(slots->deg[1], 1, N, w, 0, S);
    if (!(bar.y & kBarOk)) {
        if (t == 0) scoped_store<false>(&ctrl->err, 4);
        return;
    }
    if (bar.x > rlimit || (bar.y & kBarAny)) {
        if (w == 0 && t == 0) report(ctrl, 2, qlen0, lvl0, 0, 0, 0);
        return;
    }
    // No hubs, and ids outside the hot ones: if the graph is symmetric, no id is
    // pointed at much more often than others either, and claims do not queue
    // (2^18 ids of mean degree 64 497 -> 269 us, 2^20 810 -> 629, 128 x 128 x 128
    // lattice 3.37 -> 2.79 ms; 40 x 40 x 40 lattice, all ids hot, merged 8% faster).
    const bool plain = !ROWS && V > kHotIds && maxdeg <= hub.degree;
    const int64_t merge_edges = plain && hub.symmetric ? INT64_MAX : kMergeEdges;
    const bool l1 = L && plain;
    bool merge = bar.x > merge_edges;
    if (t < 2) S.cnt[t] = 0;
    __syncthreads();
    uint32_t spill0 = 0; // sy->spill before this level: it only grows within a launch
    bool local = false;  // the frontier lies in the shares, else in the queue
    int32_t n = 0;       // this workgroup's share
    int buf = 0;         // nv[buf]: this level's share
    // a step's edges; the share's first step is loaded ahead of the barrier
    int32_t tv[kSmallEPT] = {}, tu[kSmallEPT] = {};
    bool tok[kSmallEPT] = {};
    int32_t R = 0;
    // the last step's winners, whose outputs are stored behind the next loads
    int32_t ov[kSmallEPT], ou[kSmallEPT];
    bool own[kSmallEPT] = {};
    auto store_outputs = [&](int32_t depth) {
#pragma unroll
        for (int j = 0; j < kSmallEPT; ++j) {
            if (own[j]) {
                level[ov[j]] = depth;
                if (parent) parent[ov[j]] = ou[j];
            }
            own[j] = false;
        }
    };

    // rows i0 .. i0 + kRowStep - 1 of the share nv, one lane per edge
    auto load_rows = [&](const int32_t* nv, int32_t i0) {
        const int32_t e = t % kRowEdges;
        int64_t a[kSmallEPT], b[kSmallEPT];
        bool any = false;
#pragma unroll
        for (int j = 0; j < kSmallEPT; ++j) {
            const int32_t i = i0 + j * (kSW / kRowEdges) + t / kRowEdges;
            tok[j] = i < n;
            tv[j] = tok[j] ? nv[i] : 0;
            any |= tok[j];
        }
        if (!__any(any)) return;
#pragma unroll
        for (int j = 0; j < kSmallEPT; ++j) {
            a[j] = off[tv[j]];
            b[j] = off[tv[j] + 1];
            tu[j] = orig && parent ? orig[tv[j]] : tv[j];
        }
        any = false;
#pragma unroll
        for (int j = 0; j < kSmallEPT; ++j) {
            tok[j] = tok[j] && a[j] + e < b[j];
            any |= tok[j];
        }
        if (!__any(any)) return;  // (some edge exists: col[0] is one)
#pragma unroll
        for (int j = 0; j < kSmallEPT; ++j) tv[j] = col[tok[j] ? a[j] + e : 0];
    };

    while (true) {
        int32_t* __restrict__ Qn = par ? Qa : Qb;
        uint32_t* cnt = &S.cnt[step & 1];
        if (merge) {
            for (int i = t; i < kHotIds / 32; i += kSW) S.hot[i] = 0;
            __syncthreads();
        }
        int32_t* nv_in = S.nv[buf];
        int32_t* nv_out = S.nv[buf ^ 1];
        auto tile_step = [&]() {
            store_outputs(lvl);
            claim_edges<L, kSmallEPT>(tv, tu, tok, merge, l1, vis, parent, S.hot, own);
            keep_winners<L, kSmallEPT>(tv, own, V, nv_out, cnt, Qn, &sy->spill, spill0, ctrl);
#pragma unroll
            for (int j = 0; j < kSmallEPT; ++j) {
                ov[j] = tv[j];
                ou[j] = tu[j];
            }
        };
        if (ROWS && local) {
            for (int32_t i0 = 0; i0 < n; i0 += kRowStep) {
                if (i0 > 0) load_rows(nv_in, i0);
#pragma unroll
                for (int j = 0; j < kSmallEPT; ++j) my_edges += tok[j] ? 1 : 0;
                tile_step();
            }
        } else if (local) {
            if (t == 0) my_edges += R;
            for (int32_t e0 = 0; e0 < R; e0 += kSmallTile) {
                if (e0 > 0) {
                    __syncthreads();  // the map is reused
                    map_small_tile(S, n, R, e0, col, tv, tu, tok);
                }
                tile_step();
            }
        } else {
            const int32_t* __restrict__ Q = par ? Qb : Qa;
            // a frontier that one stage holds is split by edges (every
            // workgroup stages all of it), a larger one by entries
            const bool split = qlen <= kSmallStage;
            const int64_t k0 = split ? 0 : (int64_t)qlen * w / N;
            const int64_t k1 = split ? qlen : (int64_t)qlen * (w + 1) / N;
            for (int64_t s0 = k0; s0 < k1; s0 += kSmallStage) {
                const int32_t ns = (int32_t)(k1 - s0 < kSmallStage ? k1 - s0 : kSmallStage);
                const int32_t Rs = stage_share(S, Q + s0, ns, off, orig);
                const int32_t e_lo = split ? (int32_t)((int64_t)Rs * w / N) : 0;
                const int32_t e_hi = split ? (int32_t)((int64_t)Rs * (w + 1) / N) : Rs;
                if (t == 0) my_edges += e_hi - e_lo;
                for (int32_t e0 = e_lo; e0 < e_hi; e0 += kSmallTile) {
                    map_small_tile(S, ns, e_hi, e0, col, tv, tu, tok);
                    tile_step();
                    __syncthreads();  // the map and the stage are reused
                }
            }
        }
        if (merge) {
            __syncthreads();
            merge_hot<L>(S.hot, lvl, V, vis, level, nv_out, cnt, Qn, &sy->spill, spill0, ctrl);
        }
        __syncthreads();
        // arrive: every claim of this workgroup has returned
        const uint32_t c = __builtin_amdgcn_readfirstlane(*cnt);
        const uint32_t flag = c > (uint32_t)kSmallStage ? 1u : 0u;
        n = flag ? kSmallStage : (int32_t)c;
        buf ^= 1;
        ++ep_cnt;
        if (t == 0)
            scoped_store<L>(&slots->cnt[ep_cnt & 1][w],
                          ((uint64_t)ep_cnt << 32) | (flag << 31) | (uint32_t)n);
        if (t == kSW - 1) S.cnt[(step & 1) ^ 1] = 0;  // the next level's, behind a barrier
        // the share's rows and first neighbours, while the others arrive
        if (ROWS) {
            load_rows(S.nv[buf], 0);
        } else {
            R = stage_share(S, S.nv[buf], n, off, orig);
            ++ep_deg;
            if (t == 0) {
                int32_t mx = S.dmax[0];
                for (int k = 1; k < kSW / 64; ++k) mx = S.dmax[k] > mx ? S.dmax[k] : mx;
                const uint32_t sat = R > kEdgeSat ? (uint32_t)kEdgeSat : (uint32_t)R;
                scoped_store<L>(&slots->deg[ep_deg & 1][w],
                              ((uint64_t)ep_deg << 32) | (mx > dlimit ? 1u << 31 : 0u) | sat);
            }
            if (R > 0 && R <= rlimit) map_small_tile(S, n, R, 0, col, tv, tu, tok);
        }
        if (merge && l1) drop_l1();
        store_outputs(lvl);
        bar = wait_slots(slots->cnt[ep_cnt & 1], ep_cnt, N, w, kRowStep, S);
        if (!(bar.y & kBarOk)) {
            code = 3;
            break;
        }
        const bool over = (bar.y & kBarAny) != 0;
        bool deal = over || (ROWS && (bar.y & kBarSkew));
        int32_t qn = bar.x, spilled = 0;
        if (over) {
            // (the next spill is behind the barrier of the dealing below)
            const uint32_t s1 = __builtin_amdgcn_readfirstlane(
                __hip_atomic_load(&sy->spill, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            spilled = (int32_t)(s1 - spill0);
            spill0 = s1;
            qn += spilled;  // at most V
        }
        ++step;
        ++lvl;
        par ^= 1;
        reached += qn;
        qlen = qn;
        if (qn == 0) {
            code = 1;
            break;
        }
        bool back = qn > qlimit;
        int32_t pre = -1;
        if (!back && !over) {
            if (ROWS) {
                const int64_t r = (int64_t)qn * maxdeg;  // at least the level's edges
                merge = r > kRowMergeEdges || (r > kMergeEdges && 2 * r > V);
            } else {
                pre = S.pre;
                __syncthreads();  // S.pre has been read
                bar = wait_slots(slots->deg[ep_deg & 1], ep_deg, N, w, kSmallTile, S);
                if (!(bar.y & kBarOk)) {
                    code = 3;
                    break;
                }
                back = bar.x > rlimit || (bar.y & kBarAny);
                deal = (bar.y & kBarSkew) != 0;
                merge = bar.x > merge_edges;
            }
        }
        if (back || deal) {
            // the whole frontier to the queue: the spilled entries are there
            int32_t* __restrict__ Qx = par ? Qb : Qa;
            if (pre < 0) pre = S.pre;
            for (int32_t i = t; i < n; i += kSW) {
                const int64_t q = (int64_t)spilled + pre + i;
                if (q < V) scoped_store<L>(Qx + q, S.nv[buf][i]);
                else scoped_store<false>(&ctrl->err, 5);
            }
            if (back) {
                code = 2;
                break;
            }
            // the stores (the spilled entries' too) have reached the L2, or
            // with device scope the other XCDs: no cache is written back
            wait_stores();
            __syncthreads();
            ++ep_cnt;
            if (t == 0) scoped_store<L>(&slots->cnt[ep_cnt & 1][w], (uint64_t)ep_cnt << 32);
            bar = wait_slots(slots->cnt[ep_cnt & 1], ep_cnt, N, w, 0, S);
            if (!(bar.y & kBarOk)) {
                code = 3;
                break;
            }
            if (over) {
                // the spilled entries' degrees have not been looked at
                const int64_t k0 = (int64_t)qlen * w / N, k1 = (int64_t)qlen * (w + 1) / N;
                const uint32_t lim = slice_limits(S, Qx, k0, k1, off, dlimit);
                ++ep_deg;
                if (t == 0)
                    scoped_store<L>(&slots->deg[ep_deg & 1][w], ((uint64_t)ep_deg << 32) | lim);
                bar = wait_slots(slots->deg[ep_deg & 1], ep_deg, N, w, 0, S);
                if (!(bar.y & kBarOk)) {
                    code = 3;
                    break;
                }
                if (bar.x > rlimit || (bar.y & kBarAny)) {
                    code = 2;
                    break;
                }
                merge = bar.x > merge_edges;
            }
            local = false;
        } else {
            local = true;
        }
    }
    if (code == 3) {
        if (t == 0) scoped_store<false>(&ctrl->err, 4);
        return;
    }
    int64_t e = my_edges;
    for (int o = 32; o >= 1; o >>= 1) e += __shfl_xor(e, o, 64);
    if ((t & 63) == 0 && e)
        atomicAdd(reinterpret_cast<unsigned long long*>(&sy->edges), (unsigned long long)e);
    if (w == 0 && t == 0)
        report(ctrl, code, qlen, lvl, step, reached, code == 1 ? step - 1 : step);
}

__device__ __forceinline__ int arrivals(uint64_t a)
{
    int n = 0;
#pragma unroll
    for (int x = 0; x < kXcdSlices; ++x) n += (int)((a >> (7 * x)) & 127u);
    return n;
}

// Workgroups b with b mod 8 == cls take part; the launch leaves its sync
// block as it found it (zero): the workgroup that leaves last stores the edge
// total, clears the block and publishes the control block to the host.
__global__ __launch_bounds__(kSW) void k_small_levels(
    int32_t V, const int64_t* __restrict__ off, const int32_t* __restrict__ col,
    const int32_t* __restrict__ orig, uint32_t* __restrict__ vis,
    int32_t* __restrict__ Qa, int32_t* __restrict__ Qb, int32_t* __restrict__ level,
    int32_t* __restrict__ parent, SmallSync* __restrict__ sy, SmallSlots* __restrict__ slots,
    Ctrl* __restrict__ ctrl, Ctrl* __restrict__ h_ctrl, uint64_t seq, int32_t cls, int32_t qlen0, int32_t lvl0, int32_t qlimit,
    int64_t rlimit, int32_t dlimit, int32_t maxdeg, HubRule hub)
{
    if ((int)(blockIdx.x & (kXcdSlices - 1)) != cls) return;
    __shared__ SmallLds S;
    __shared__ int s_go;  // 0 called off, 1 device scope, 2 one XCD
    const int N = (int)(gridDim.x / kXcdSlices);
    const int w = (int)(blockIdx.x / kXcdSlices);
    const int t = threadIdx.x;
    // qlen0 < 0: launched right behind a host-driven level, whose next
    // frontier size is in ctrl; an empty frontier ends the search and one
    // above the limit goes back to the host, both before any level
    bool run = !(ctrl->err & kErrCsr);
    if (maxdeg < 0) maxdeg = ctrl->maxdeg;
    if (qlen0 < 0) {
        qlen0 = (int32_t)(ctrl->qn_count + (uint32_t)(ctrl->pack[-1 - qlen0] & kPackMask));
        if (w == 0 && t == 0) scoped_store<false>(&ctrl->front_n, (uint32_t)qlen0);
        if (qlen0 == 0 || qlen0 > qlimit) run = false;
    }
    auto not_run = [&]() { report(ctrl, qlen0 == 0 ? 1 : 2, qlen0, lvl0, 0, 0, 0); };
    if (run) {
        const uint32_t lim = slice_limits(S, Qa, (int64_t)qlen0 * w / N, (int64_t)qlen0 * (w + 1) / N,
                                          off, dlimit);
        if (t == 0) {
            scoped_store<false>(&slots->cnt[0][w], (uint64_t)0);
            scoped_store<false>(&slots->cnt[1][w], (uint64_t)0);
            scoped_store<false>(&slots->deg[0][w], (uint64_t)0);
            scoped_store<false>(&slots->deg[1][w], ((uint64_t)1 << 32) | lim);
            // the slots have reached the other XCDs before this arrival does
            wait_stores();
            // one 7-bit count of arrivals per XCC; the sign bit calls off
            const uint32_t xcc = __builtin_amdgcn_s_getreg((2 << 11) | 20);  // XCC_ID[2:0]
            const uint64_t one = 1ull << (7 * xcc);
            uint64_t a = __hip_atomic_fetch_add(&sy->arrive, one, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT) + one;
            uint32_t spins = 0;
            while (!(a >> 63) && arrivals(a) < N) {
                if (++spins > kStartCap) {
                    uint64_t seen = a;
                    if (__hip_atomic_compare_exchange_strong(&sy->arrive, &seen, a | (1ull << 63),
                                                             __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT))
                        not_run();
                }
                a = __hip_atomic_load(&sy->arrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            s_go = (a >> 63) ? 0 : (a == one * (uint64_t)N ? 2 : 1);
        }
        __syncthreads();
        // rows that take one lane per edge: the limits on edges and degrees cannot
        // be exceeded by a frontier that fits the workgroups' shares
        const bool rows = maxdeg <= kRowEdges && maxdeg <= dlimit &&
                          (int64_t)N * kSmallStage * maxdeg <= rlimit;
#define BFS_SMALL_BODY(L, ROWS)                                                                   \
    small_levels_body<L, ROWS>(S, V, off, col, orig, vis, Qa, Qb, level, parent, sy, slots, ctrl, \
                               N, w, qlen0, lvl0, qlimit, rlimit, dlimit, maxdeg, hub)
        if (s_go == 2) {
            if (rows) BFS_SMALL_BODY(true, true);
            else BFS_SMALL_BODY(true, false);
        } else if (s_go == 1) {
            if (rows) BFS_SMALL_BODY(false, true);
            else BFS_SMALL_BODY(false, false);
        }
#undef BFS_SMALL_BODY
    } else if (w == 0 && t == 0) {
        not_run();
    }
    wait_stores();  // edge counts and result
    __syncthreads();
    if (t < 64) {
        uint32_t k = 0;
        if (t == 0)
            k = __hip_atomic_fetch_add(&sy->leave, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        k = __builtin_amdgcn_readfirstlane(k);
        if ((int)k != N - 1) return;
        const int64_t edges =
            __hip_atomic_load(&sy->edges, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (t == 0) {
            ctrl->r_total = edges;
            if (__hip_atomic_load(&ctrl->steps, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > 0) {
                // a scan of the frontier these levels started from is spent
                ctrl->pack[0] = ctrl->pack[1] = 0;
                ctrl->dropped[0] = ctrl->dropped[1] = 0;
            }
            sy->arrive = 0;
            sy->spill = 0;
            sy->edges = 0;
            sy->leave = 0;
        }
        if (h_ctrl) {
            // the mirror: a lane per 8 bytes, then the sequence number
            constexpr int n8 = offsetof(Ctrl, seq) / 8;
            static_assert(n8 <= 64, "one lane per word");
            if (t < n8) {
                uint64_t x = __hip_atomic_load(reinterpret_cast<const uint64_t*>(ctrl) + t,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (t == offsetof(Ctrl, r_total) / 8) x = (uint64_t)edges;
                reinterpret_cast<uint64_t*>(h_ctrl)[t] = x;
            }
            __threadfence_system();
            if (t == 0)
                __hip_atomic_store(&h_ctrl->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

int small_loop_blocks()
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_small_levels, kSW, 0) != hipSuccess)
        return 0;
    return n;
}

hipError_t launch_small_levels(hipStream_t s, int wgs, int cls, int32_t V, const int64_t* off,
                               const int32_t* col, const int32_t* orig, uint32_t* vis,
                               int32_t* Qa, int32_t* Qb, int32_t* level,
                               int32_t* parent, SmallSync* sy, uint32_t* slot_words, Ctrl* ctrl,
                               Ctrl* h_ctrl, uint64_t seq, int32_t qlen, int32_t lvl, int32_t qlimit, int64_t rlimit,
                               int32_t dlimit, int32_t maxdeg, HubRule hub)
{
    // An ordinary launch: the workgroups that take part are few enough to be
    // resident at once, and a cooperative launch would make the runtime stop
    // overlapping later kernels of other streams.
    if (wgs < 1 || wgs > kSmallMaxWGs) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_small_levels, dim3(wgs * kXcdSlices), dim3(kSW), 0, s, V, off, col, orig,
                       vis, Qa, Qb, level, parent, sy,
                       reinterpret_cast<SmallSlots*>(slot_words), ctrl, h_ctrl, seq, cls, qlen,
                       lvl, qlimit, rlimit, dlimit, maxdeg, hub);
    return hipGetLastError();
}

}  // namespace bfsmi
