// Persistent multi-source levels for serving batches on deep graphs.
//
// On a grid-like graph a serving batch runs thousands of levels whose union
// frontier holds a few thousand vertices.  As separate launches each level
// is seven kernels (degree scan, expansion, front clear, finalize, advance),
// and on a busy GPU every one of them waits behind other graphs' kernels in
// the shared hardware queues.  This kernel runs up to max_levels such levels
// in one launch of a few dozen workgroups, one barrier per level.
//
// A level's work is the expansion of the paper's Section 3.4 on lane masks:
// per edge u -> v the lanes new to v are f = mask(u) & ~seen[v], ORed into
// v's marks with a returning atomic, and the thread that turns the marks from
// zero to non-zero keeps v as a candidate (so each vertex is kept once); then
// each candidate is finalized: new = marks & ~seen, seen |= new, marks = 0,
// and each new lane b gets depth level - lane_start[b] in its int16 result
// row (caller ids).
//
// The finalize of one level and the expansion of the next run in the same
// phase, so only one barrier separates levels.  Marks and candidates come in
// two parities (sn[].next and front[]): a phase finalizes one parity while
// its expansion fills the other, so a thread that finalizes v writes only v's
// own words of the parity it reads, and the seen masks it updates are read
// elsewhere only as a filter (a stale seen lets a spurious candidate through,
// which its finalize then drops).
//
// Such levels are bound by the chain of dependent memory round trips, so, as
// in the single-root loop (smallloop.hip):
//   - the workgroups that take part share one XCD (every eighth of the launch;
//     they compare their XCC ids when they start): marks are ORed with atomics
//     of that L2, shared words are read past the L1, and no barrier writes
//     back or invalidates the L2;
//   - candidates stay in the LDS of the workgroup that found them; the lists
//     in memory take only those that do not fit, or all when the candidates
//     are dealt out anew (a share overflowed or is a multiple of the mean);
//   - a workgroup arrives at the barrier with one store to its own slot, which
//     also holds its candidate count, and loads the rows of its candidates
//     while it waits; it reads all slots with one load per lane;
//   - graphs whose largest degree is at most kMsRowEdges (lattices) take one
//     lane per row and load the neighbours before the barrier too, so the
//     candidates' marks and the neighbours' seen masks are one round trip.
//     Others map edges to threads by binary search in the share's degree
//     prefix sum and put the level's edge count and largest degree in the
//     slots.
// A 512 x 512 grid served alone, against one agent-scope counter barrier and
// list reservations per wave (and host rounds of 2, 8, 32 levels): 1 query
// (836 levels) 13.2 -> 3.5 ms, 6 queries 16.4 -> 5.2, 48 queries 29.0 -> 15.0;
// a 1000 x 1000 grid, 32 queries 62.7 -> 39.9 ms.
//
// The kernel starts from the state the level kernels leave (frontier in Qa,
// lane masks in front) and leaves the same state when it stops: the round's
// last phase only finalizes, writing the frontier to Qa and its masks to
// front.  The per-level bookkeeping is that of the separate launches
// (level, alive lanes, reached, done), so the host's round logic does not
// change.  The kernel stops when the batch is done, after max_levels levels,
// or before expanding a frontier whose candidates (an upper bound on it),
// their edges or their largest degree exceed the limits; the host then
// runs that level with the ordinary kernels.  Every wait is bounded.  The
// workgroups start together or not at all: one that has waited too long for
// the others, or finds them on more than one XCD, makes the launch run no
// level, and the host runs the round.  A wait inside the loop that does not
// end sets ctrl->err and every workgroup leaves.
#include "bfs_internal.h"
#include "wave_ops.h"

namespace bfsmi {

constexpr int kMsW = 512;                // threads per workgroup
constexpr int kMsShare = 1024;           // candidates a workgroup keeps in LDS
constexpr int kMsPass = kMsW;            // candidates per pass, one per thread
constexpr int kMsEPT = 4;                // edges per thread per pass
constexpr int kMsTile = kMsW * kMsEPT;
constexpr int kMsRowEdges = 4;           // rows of at most this many edges: a lane per row
constexpr int kMsSkewMin = 256;          // shares up to this size are left alone
constexpr uint32_t kMsStartCap = 1u << 14;  // polls before a launch is called off
constexpr uint32_t kMsSpinCap = 1u << 23;
constexpr int32_t kMsDegSat = 1 << 14;   // degrees saturate here in the sums, above the host's limit
constexpr uint32_t kMsEdgeSat = 1u << 25;  // ... and a share's edges in its slot

struct MsLds {
    int32_t cum[kMsPass + 1];
    uint64_t f[kMsPass];
    int64_t base[kMsPass];
    uint16_t map[kMsTile];
    int32_t nv[2][kMsShare];  // candidates, by parity
    int32_t wave[kMsW / 64];
    int16_t* out[64];
    int32_t start[64];
    uint32_t cnt[2];      // candidates found (those in memory included), by parity
    uint32_t found;       // some vertex got new lanes in this phase
    uint32_t bad;         // a guard tripped or a depth overflowed
    unsigned long long edges;  // of this workgroup's candidates
    int32_t mdeg;              // their largest degree
    uint32_t q0;          // flush: where this share goes in the list
    // of the last barrier
    int32_t sum, esum, bits;
};
constexpr int kMsDeal = 1, kMsFound = 2, kMsBad = 4, kMsOver = 8, kMsOk = 16;
// slot word 0: epoch << 32 | share overflowed << 31 | found << 30 | bad << 29 |
// candidates; word 1: epoch << 32 | a degree over the limit << 31 | edges
constexpr uint32_t kMsCount = (1u << 29) - 1;

template <typename T>
__device__ __forceinline__ T ms_load(const T* p)  // past the L1
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T>
__device__ __forceinline__ void ms_store_agent(T* p, T x)
{
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Words that other workgroups of the XCD read behind a barrier.
template <typename T>
__device__ __forceinline__ void ms_store(T* p, T x)
{
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__device__ __forceinline__ void ms_bad(MsLds& S, int32_t* flag, int32_t x)
{
    ms_store_agent(flag, x);
    S.bad = 1;
}

// Slots of set epoch & 1: N words 0, then N words 1.
__device__ __forceinline__ uint64_t* ms_slots(uint64_t* slots, uint32_t epoch, int N)
{
    return slots + (epoch & 1u) * 2 * N;
}

// Waits until all slots carry the epoch; sums and flags go to S.  Every
// thread calls it; the last wave, which has the least to load, polls (word 0
// on its lower half, word 1 on its upper).
template <bool ROWS>
__device__ __forceinline__ void ms_wait(uint64_t* slots, uint32_t epoch, int N, MsLds& S)
{
    if (threadIdx.x >= kMsW - 64) {
        const int lane = __lane_id();
        const int k = lane & 31;
        const bool mine = k < N && (lane < 32 || !ROWS);
        const uint64_t* p = ms_slots(slots, epoch, N) + (lane < 32 ? 0 : N) + (mine ? k : 0);
        uint64_t x = (uint64_t)epoch << 32;
        uint32_t spins = 0;
        bool ok = true;
        while (true) {
            if (mine) x = ms_load(p);
            if (__all((uint32_t)(x >> 32) == epoch)) break;
            if (++spins > kMsSpinCap) {
                ok = false;
                break;
            }
        }
        const uint32_t lo = (uint32_t)x;
        const int32_t c = mine && lane < 32 ? (int32_t)(lo & kMsCount) : 0;
        const int32_t sum = __builtin_amdgcn_readlane(wave_inclusive_scan_dpp(c), 63);
        int32_t esum = 0;
        if (!ROWS) {
            const int32_t e = mine && lane >= 32 ? (int32_t)(lo & 0x7fffffffu) : 0;
            esum = __builtin_amdgcn_readlane(wave_inclusive_scan_dpp(e), 63);
        }
        const uint64_t top = __ballot(mine && (lo >> 31));
        const uint64_t found = __ballot(mine && lane < 32 && ((lo >> 30) & 1u));
        const uint64_t bad = __ballot(mine && lane < 32 && ((lo >> 29) & 1u));
        const uint64_t skew = __ballot(c > kMsSkewMin && (int64_t)c * N > 2 * (int64_t)sum);
        if (lane == 0) {
            S.sum = sum;
            S.esum = esum;
            S.bits = ((uint32_t)top || skew ? kMsDeal : 0) | (found ? kMsFound : 0) |
                     (bad ? kMsBad : 0) | (top >> 32 ? kMsOver : 0) | (ok ? kMsOk : 0);
        }
    }
    __syncthreads();
}

// Appends the candidates among a wave's NE edges per lane to the workgroup's
// share; those that do not fit go to the list in memory.
template <bool ROWS, int NE>
__device__ __forceinline__ void ms_append(MsLds& S, const int32_t (&vv)[NE], const bool (&first)[NE],
                                          int par, int32_t V, const int64_t* __restrict__ off,
                                          int32_t* __restrict__ list, uint32_t* list_n,
                                          Ctrl* __restrict__ ctrl)
{
    uint64_t mask[NE];
    uint32_t total = 0;
#pragma unroll
    for (int j = 0; j < NE; ++j) {
        mask[j] = __ballot(first[j]);
        total += (uint32_t)__popcll(mask[j]);
    }
    if (!total) return;  // uniform over the wave
    uint32_t pos0 = 0, q0 = 0;
    if (__lane_id() == 0) pos0 = atomicAdd(&S.cnt[par], total);
    pos0 = __builtin_amdgcn_readfirstlane(pos0);
    const uint32_t over0 = pos0 > kMsShare ? pos0 : kMsShare;  // first position that spills
    if (pos0 + total > over0) {
        if (__lane_id() == 0)
            q0 = __hip_atomic_fetch_add(list_n, pos0 + total - over0, __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_WORKGROUP);
        q0 = __builtin_amdgcn_readfirstlane(q0);
    }
    uint32_t base = pos0;
#pragma unroll
    for (int j = 0; j < NE; ++j) {
        if (first[j]) {
            const uint32_t pos = base + lanes_below(mask[j]);
            if (pos < kMsShare) {
                S.nv[par][pos] = vv[j];
            } else {
                const uint32_t q = q0 + (pos - over0);
                if (q < (uint32_t)V) ms_store(list + q, vv[j]);
                else ms_bad(S, &ctrl->err, 7);
                if (!ROWS) {
                    const int64_t dd = off[vv[j] + 1] - off[vv[j]];
                    const int32_t d = (int32_t)(dd < kMsDegSat ? dd : kMsDegSat);
                    atomicAdd(&S.edges, (unsigned long long)d);
                    atomicMax(&S.mdeg, d);
                }
            }
        }
        base += (uint32_t)__popcll(mask[j]);
    }
}

// A thread's NE edges: the lanes nb new to x go into its marks of parity tp;
// first: they were the first.  (All atomics are issued before one is waited
// for.)
template <int NE>
__device__ __forceinline__ void ms_mark(const uint64_t (&nb)[NE], const int32_t (&x)[NE], int tp,
                                        SeenNext* sn, uint64_t* front, bool (&first)[NE])
{
    uint64_t old[NE];
#pragma unroll
    for (int k = 0; k < NE; ++k) old[k] = ~0ull;
#pragma unroll
    for (int k = 0; k < NE; ++k)
        if (nb[k])
            old[k] = __hip_atomic_fetch_or(tp ? front + x[k] : &sn[x[k]].next, nb[k],
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
    for (int k = 0; k < NE; ++k) first[k] = old[k] == 0;
}

// The levels; every workgroup returns from it exactly once.
template <bool ROWS>
__device__ __forceinline__ void ms_levels_body(
    MsLds& S, int32_t V, const int64_t* __restrict__ off, const int32_t* __restrict__ col,
    const int32_t* __restrict__ orig, SeenNext* sn, uint64_t* front, int32_t* Qa, int32_t* Qb,
    int32_t* found, uint64_t* slots, MsSync* sy, Ctrl* ctrl, int N, int w, int32_t qlen0,
    int32_t lvl0, int32_t max_levels, int32_t qlimit, int64_t rlimit, int32_t dlimit)
{
    const int t = threadIdx.x;
    // this thread's entry of the pass: vertex (-1: none), caller id, row and
    // its first neighbours
    int32_t v, vo = 0, d, cv[kMsRowEdges];
    int64_t a = 0;
    // loads entries 0 .. n-1 of a share in LDS (list null) or in memory
    // (loads are unconditional, of valid ids: behind a branch the compiler
    // waits for each before it issues the next)
    auto fetch = [&](const int32_t* share, const int32_t* list, int32_t n) {
        v = -1;
        if (t < n) v = list ? ms_load(list + t) : share[t];
        if (v >= V) {
            ms_bad(S, &ctrl->err, 9);
            v = -1;
        }
        d = 0;
#pragma unroll
        for (int k = 0; k < kMsRowEdges; ++k) cv[k] = 0;
        if (!__any(v >= 0)) return;
        const int32_t u = v < 0 ? 0 : v;
        a = off[u];
        const int64_t a1 = off[u + 1];
        vo = orig ? orig[u] : u;
        d = v < 0 ? 0 : (int32_t)(a1 - a);
        if (ROWS && __any(d > 0))  // (then col[0] is a neighbour)
#pragma unroll
            for (int k = 0; k < kMsRowEdges; ++k) cv[k] = col[k < d ? a + k : 0];
    };
    // expands the pass's n entries with lane masks nw into the marks of
    // parity tp; ROWS: seen holds the neighbours' seen masks
    auto expand = [&](uint64_t nw, const uint64_t (&seen)[kMsRowEdges], int32_t n, int tp,
                      int32_t* list, uint32_t* list_n) {
        if constexpr (ROWS) {
            if (!__any(nw != 0)) return;
            bool first[kMsRowEdges];
            uint64_t nb[kMsRowEdges];
#pragma unroll
            for (int k = 0; k < kMsRowEdges; ++k) nb[k] = k < d ? nw & ~seen[k] : 0ull;
            ms_mark(nb, cv, tp, sn, front, first);
            ms_append<ROWS>(S, cv, first, tp, V, off, list, list_n, ctrl);
        } else {
            const int32_t tot = nw ? d : 0;
            const int32_t inc = wave_inclusive_scan_dpp(tot);
            if ((t & 63) == 63) S.wave[t >> 6] = inc;
            __syncthreads();
            int32_t c = inc - tot, R = 0;
#pragma unroll
            for (int k = 0; k < kMsW / 64; ++k) {
                const int32_t x = S.wave[k];
                if (k < (t >> 6)) c += x;
                R += x;
            }
            if (t < n) {
                S.cum[t] = c;
                S.f[t] = nw;
                S.base[t] = a - c;
            }
            if (t == 0) S.cum[n] = R;
            __syncthreads();
            for (int32_t e0 = 0; e0 < R; e0 += kMsTile) {
                const int32_t n_e = R - e0 < kMsTile ? R - e0 : kMsTile;
                const int32_t sl0 = e0 + t * kMsEPT;
                if (t * kMsEPT < n_e) {
                    int32_t lo = 0;
                    for (int32_t st = 1 << (31 - __builtin_clz(n)); st > 0; st >>= 1) {
                        const int32_t x = lo + st;
                        if (x < n && S.cum[x] <= sl0) lo = x;
                    }
                    int32_t i = lo;
#pragma unroll
                    for (int j = 0; j < kMsEPT; ++j) {
                        const int32_t sl = sl0 + j;
                        if (sl - e0 < n_e) {
                            while (i + 1 < n && S.cum[i + 1] <= sl) ++i;
                            S.map[sl - e0] = (uint16_t)i;
                        }
                    }
                }
                __syncthreads();
                if (__any(t < n_e)) {
                    int32_t vv[kMsEPT];
                    uint64_t fm[kMsEPT], have[kMsEPT];
                    bool first[kMsEPT];
#pragma unroll
                    for (int j = 0; j < kMsEPT; ++j) {
                        const int32_t sl = t + j * kMsW;
                        const bool ok = sl < n_e;
                        const int32_t sc = ok ? sl : n_e - 1;
                        const int32_t i = S.map[sc];
                        fm[j] = ok ? S.f[i] : 0ull;
                        vv[j] = col[S.base[i] + e0 + sc];
                    }
                    // stale masks only let more threads issue the atomic
#pragma unroll
                    for (int j = 0; j < kMsEPT; ++j)
                        have[j] = ms_load(&sn[vv[j]].seen) | ms_load(&sn[vv[j]].next) |
                                  ms_load(front + vv[j]);
#pragma unroll
                    for (int j = 0; j < kMsEPT; ++j) fm[j] &= ~have[j];
                    ms_mark(fm, vv, tp, sn, front, first);
                    ms_append<ROWS>(S, vv, first, tp, V, off, list, list_n, ctrl);
                }
                __syncthreads();
            }
        }
    };

    uint32_t epoch = 0;
    // arrives at the next barrier; called by all threads behind a
    // __syncthreads that follows each wave's vmcnt(0)
    auto arrive = [&](uint32_t w0, uint32_t w1) {
        ++epoch;
        if (t == 0) {
            uint64_t* p = ms_slots(slots, epoch, N) + w;
            ms_store(p, (uint64_t)epoch << 32 | w0);
            if (!ROWS) ms_store(p + N, (uint64_t)epoch << 32 | w1);
        }
    };
    auto settle = [&]() {
        wait_stores();
        __syncthreads();
    };
    auto limits = [&]() {
        return (uint32_t)(S.edges < kMsEdgeSat ? S.edges : kMsEdgeSat) |
               (S.mdeg > dlimit ? 1u << 31 : 0u);
    };
    // adds the fetched entries' degrees to S.edges, S.mdeg
    auto add_degrees = [&]() {
        int32_t s = d < kMsDegSat ? d : kMsDegSat, mx = d;
        if (!__any(mx > 0)) return;
        s = __builtin_amdgcn_readlane(wave_inclusive_scan_dpp(s), 63);
        for (int o = 32; o >= 1; o >>= 1) {
            const int32_t m2 = __shfl_xor(mx, o, 64);
            mx = m2 > mx ? m2 : mx;
        }
        if ((t & 63) == 0) {
            atomicAdd(&S.edges, (unsigned long long)s);
            atomicMax(&S.mdeg, mx);
        }
    };
    // the last pass's new vertices, whose results are stored behind the loads
    // for the next phase
    uint64_t onw = 0;
    int32_t ovo = 0;
    auto store_results = [&](int32_t dl) {
        for (; onw; onw &= onw - 1) {
            const int k = __builtin_ctzll(onw);
            const int32_t dd = dl - S.start[k];
            if (dd > 32767) ms_bad(S, &ctrl->overflow, 1);
            else if (S.out[k]) S.out[k][ovo] = (int16_t)dd;  // null: retired lane
        }
    };
    // the end of a phase: publishes this share's size and limits, loads its
    // rows and waits for the others
    auto next_phase = [&](int par, int32_t dl) {
        settle();
        const uint32_t c = S.cnt[par];
        const int32_t n = (int32_t)(c < (uint32_t)kMsShare ? c : (uint32_t)kMsShare);
        const uint32_t w0 = (c & kMsCount) | (c > (uint32_t)kMsShare ? 1u << 31 : 0u) |
                            (S.found ? 1u << 30 : 0u) | (S.bad ? 1u << 29 : 0u);
        uint32_t w1 = 0;
        if (ROWS) {
            arrive(w0, 0u);
            fetch(S.nv[par], nullptr, n);
        } else {
            // the first pass's entries last: the next phase starts with them
            for (int32_t s0 = (n - 1) / kMsPass * kMsPass; s0 >= 0; s0 -= kMsPass) {
                fetch(S.nv[par] + s0, nullptr, n - s0);
                add_degrees();
            }
            __syncthreads();
            w1 = limits();
            arrive(w0, w1);
        }
        if (t == 0) {
            S.cnt[par ^ 1] = 0;
            S.found = 0;
            S.edges = 0;
            S.mdeg = 0;
        }
        store_results(dl);
        ms_wait<ROWS>(slots, epoch, N, S);
        return n;
    };
    auto fail = [&]() {
        if (t == 0) ms_store_agent(&ctrl->err, 6);
    };

    // the entry frontier's limits
    const int64_t k0 = (int64_t)qlen0 * w / N, k1 = (int64_t)qlen0 * (w + 1) / N;
    if (!ROWS) {
        for (int64_t s0 = k0; s0 < k1; s0 += kMsPass) {
            const int32_t n = (int32_t)(k1 - s0 < kMsPass ? k1 - s0 : kMsPass);
            fetch(nullptr, Qa + s0, n);
            add_degrees();
        }
        __syncthreads();
        arrive(0u, limits());
        if (t == 0) {
            S.edges = 0;
            S.mdeg = 0;
        }
        ms_wait<ROWS>(slots, epoch, N, S);
        if (!(S.bits & kMsOk)) return fail();
        if (S.esum > rlimit || (S.bits & kMsOver)) return;  // no level run
    }

    // ---- phase 0: expand the entry frontier (Qa, lane masks in front, which
    // are cleared) into marks 0 (sn.next), candidates into share 0
    for (int64_t s0 = k0; s0 < k1; s0 += kMsPass) {
        const int32_t n = (int32_t)(k1 - s0 < kMsPass ? k1 - s0 : kMsPass);
        fetch(nullptr, Qa + s0, n);
        uint64_t nw = 0, seen[kMsRowEdges];
        if (v >= 0) {
            nw = ms_load(front + v);
            ms_store(front + v, (uint64_t)0);  // this workgroup is the only reader of v's mask
        }
        if (ROWS)
#pragma unroll
            for (int k = 0; k < kMsRowEdges; ++k) seen[k] = ms_load(&sn[cv[k]].seen);
        expand(nw, seen, n, 0, found, &sy->fn[0]);
    }
    int32_t n = next_phase(0, lvl0);
    if (!(S.bits & kMsOk)) return fail();

    // ---- phase j >= 1: finalize the candidates of expansion j (found at
    // depth level lvl0 + j - 1) and, unless this is the round's last phase,
    // expand the new frontier at once (expansion j + 1).  Marks and shares
    // alternate by parity: phase j reads those of parity (j - 1) & 1 (every
    // candidate is kept there once, and its marks are cleared here) while
    // its expansion fills those of parity j & 1, cleared in phase j - 1.
    int32_t steps = 0;
    int64_t reached = 0;
    for (int32_t j = 1; !(S.bits & kMsBad); ++j) {
        const int pc = (j - 1) % 3, cs = j % 3;
        const int sp = (j - 1) & 1;
        int32_t* Lin = sp ? Qb : found;
        int32_t* Lout = sp ? found : Qb;
        const int32_t fn = S.sum;
        const bool last = j >= max_levels || fn > qlimit ||
                          (!ROWS && (S.esum > rlimit || (S.bits & kMsOver)));
        const bool deal = (S.bits & kMsDeal) != 0;
        if (w == 0 && t == 0)  // last read before the previous barrier
            ms_store(&sy->fn[(j + 1) % 3], 0u);
        int64_t f0 = 0, f1 = n;
        if (deal) {
            // the share behind what has spilled, then equal slices for all
            if (t == 0)
                S.q0 = n ? __hip_atomic_fetch_add(&sy->fn[pc], (uint32_t)n, __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_WORKGROUP) : 0u;
            __syncthreads();
            for (int32_t i = t; i < n; i += kMsW) {
                const uint32_t q = S.q0 + (uint32_t)i;
                if (q < (uint32_t)V) ms_store(Lin + q, S.nv[sp][i]);
                else ms_bad(S, &ctrl->err, 8);
            }
            settle();
            arrive(0u, 0u);
            ms_wait<ROWS>(slots, epoch, N, S);
            if (!(S.bits & kMsOk)) return fail();
            f0 = (int64_t)fn * w / N;
            f1 = (int64_t)fn * (w + 1) / N;
        }
        const int32_t dl = lvl0 + j - 1;
        for (int64_t s0 = f0; s0 < f1; s0 += kMsPass) {
            const int32_t ns = (int32_t)(f1 - s0 < kMsPass ? f1 - s0 : kMsPass);
            if (deal) fetch(nullptr, Lin + s0, ns);
            else if (s0 > 0) fetch(S.nv[sp] + s0, nullptr, ns);
            uint64_t nw = 0, seen[kMsRowEdges];
            if (__any(v >= 0)) {
                const int32_t u = v < 0 ? 0 : v;
                const uint64_t had = ms_load(&sn[u].seen);
                const uint64_t marks = sp ? ms_load(front + u) : ms_load(&sn[u].next);
                if (ROWS && !last)
#pragma unroll
                    for (int k = 0; k < kMsRowEdges; ++k) seen[k] = ms_load(&sn[cv[k]].seen);
                if (v >= 0) {
                    nw = marks & ~had;
                    // v's own slot only: other threads OR into the marks of
                    // the other parity meanwhile
                    if (sp) {
                        if (nw) ms_store(&sn[v].seen, had | nw);
                        ms_store(front + v, last ? nw : (uint64_t)0);
                    } else {
                        sn[v] = SeenNext{had | nw, 0ull};  // (one 16-byte store)
                        if (last) ms_store(front + v, nw);
                    }
                }
                if (nw) S.found = 1;
            }
            if (!last) expand(nw, seen, ns, j & 1, Lout, &sy->fn[cs]);
            store_results(dl);  // of the pass before
            onw = nw;
            ovo = vo;
            reached += nw ? 1 : 0;
            if (last) {
                store_results(dl);
                // the new frontier goes to Qa, the form the level kernels take
                const uint64_t mask = __ballot(nw != 0);
                if (mask) {
                    uint64_t alive = nw;
                    for (int o = 32; o >= 1; o >>= 1) alive |= __shfl_xor(alive, o, 64);
                    uint32_t base = 0;
                    if (__lane_id() == 0) {
                        base = atomicAdd(&sy->qn, (uint32_t)__popcll(mask));
                        atomicOr(reinterpret_cast<unsigned long long*>(&sy->alive),
                                 (unsigned long long)alive);
                    }
                    base = __builtin_amdgcn_readfirstlane(base);
                    if (nw) {
                        const uint32_t pos = base + lanes_below(mask);
                        if (pos < (uint32_t)V) Qa[pos] = v;
                        else ms_bad(S, &ctrl->err, 8);
                    }
                }
            }
        }
        steps = j;
        if (last) break;
        n = next_phase(j & 1, dl);
        if (!(S.bits & kMsOk)) return fail();
        if (!(S.bits & kMsFound)) break;  // the batch has ended
    }
    for (int o = 32; o >= 1; o >>= 1) reached += __shfl_xor(reached, o, 64);
    if ((t & 63) == 0 && reached)
        atomicAdd(reinterpret_cast<unsigned long long*>(&sy->reached), (unsigned long long)reached);
    if (w == 0 && t == 0) ms_store_agent(&sy->steps, steps);
}

__device__ __forceinline__ int ms_arrivals(uint64_t a)
{
    int n = 0;
#pragma unroll
    for (int x = 0; x < kXcdSlices; ++x) n += (int)((a >> (7 * x)) & 127u);
    return n;
}

static_assert(sizeof(Ctrl) % 8 == 0 && sizeof(Ctrl) <= 512, "mirrored by a wave, 8 bytes a lane");

// Workgroups b with b mod 8 == cls take part.  The launch leaves its sync
// block as it found it (zero) and mirrors the control block into pinned host
// memory, so a round needs no clearing and no copy of its own: the workgroup
// that leaves last (after every other has stopped using the sync block) does
// both, and the level bookkeeping that the separate advance does.
template <bool ROWS>
__global__ __launch_bounds__(kMsW) void k_ms_small_levels(
    int32_t V, const int64_t* __restrict__ off, const int32_t* __restrict__ col,
    const int32_t* __restrict__ orig, SeenNext* sn, uint64_t* front, int32_t* Qa, int32_t* Qb,
    int32_t* found, int16_t* const* __restrict__ lane_out, const int32_t* __restrict__ lane_start,
    MsSync* sy, uint64_t* slots, Ctrl* ctrl, Ctrl* __restrict__ h_ctrl, int32_t cls,
    int32_t max_levels, int32_t qlimit, int64_t rlimit, int32_t dlimit)
{
    if ((int)(blockIdx.x & (kXcdSlices - 1)) != cls) return;
    __shared__ MsLds S;
    __shared__ int s_go;  // the workgroups share one XCD
    const int N = (int)(gridDim.x / kXcdSlices);
    const int w = (int)(blockIdx.x / kXcdSlices);
    const int t = threadIdx.x;
    // ctrl changes only once every workgroup has left
    const int32_t qlen0 = ctrl->qlen, lvl0 = ctrl->level;
    if (!ctrl->done && max_levels >= 1 && qlen0 <= qlimit) {  // else no level
        if (t < 64) {
            S.out[t] = lane_out[t];
            S.start[t] = lane_start[t];
        }
        if (t == 0) {
            S.cnt[0] = S.cnt[1] = 0;
            S.found = S.bad = 0;
            S.edges = 0;
            S.mdeg = 0;
            for (int k = 0; k < 4; ++k) ms_store_agent(slots + k * N + w, (uint64_t)0);
            // the slots have reached the other XCDs before this arrival does
            wait_stores();
            // one 7-bit count of arrivals per XCC; the sign bit calls off
            const uint32_t xcc = __builtin_amdgcn_s_getreg((2 << 11) | 20);  // XCC_ID[2:0]
            const uint64_t one = 1ull << (7 * xcc);
            uint64_t a = __hip_atomic_fetch_add(&sy->arrive, one, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT) + one;
            uint32_t spins = 0;
            while (!(a >> 63) && ms_arrivals(a) < N) {
                if (++spins > kMsStartCap) {
                    uint64_t seen = a;
                    (void)__hip_atomic_compare_exchange_strong(&sy->arrive, &seen,
                                                               a | (1ull << 63), __ATOMIC_RELAXED,
                                                               __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_AGENT);
                }
                a = __hip_atomic_load(&sy->arrive, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            s_go = a == one * (uint64_t)N;
        }
        __syncthreads();
        if (s_go)
            ms_levels_body<ROWS>(S, V, off, col, orig, sn, front, Qa, Qb, found, slots, sy, ctrl,
                                 N, w, qlen0, lvl0, max_levels, qlimit, rlimit, dlimit);
    }
    wait_stores();  // what this wave reports
    __syncthreads();
    if (t >= 64) return;
    uint32_t k = 0;
    if (t == 0)
        k = __hip_atomic_fetch_add(&sy->leave, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    k = __builtin_amdgcn_readfirstlane(k);
    if ((int)k != N - 1) return;
    if (t == 0) {
        const int32_t steps = ms_load(&sy->steps);
        ctrl->steps = steps;
        if (steps > 0) {
            const uint32_t qn = ms_load(&sy->qn);
            const int32_t err = ms_load(&ctrl->err), ovf = ms_load(&ctrl->overflow);
            ctrl->last_alive = ms_load(&sy->alive);
            ctrl->alive = 0;
            ctrl->reached += ms_load(&sy->reached);
            ctrl->levels += qn ? steps : steps - 1;
            ctrl->level = lvl0 + steps;
            ctrl->qlen = (int32_t)qn;
            ctrl->qn_count = 0;
            ctrl->sparse = (int32_t)qn <= ctrl->sparse_limit;
            ctrl->pull = 0;  // chosen for a frontier that is gone
            ctrl->no_push = 0;
            ctrl->done = qn == 0 || qn > (uint32_t)V || ovf || err ? 1 : 0;
        }
        *sy = MsSync{};
    }
    if (h_ctrl) {
        wait_stores();
        if (t < (int)(sizeof(Ctrl) / 8))
            reinterpret_cast<uint64_t*>(h_ctrl)[t] =
                ms_load(reinterpret_cast<const uint64_t*>(ctrl) + t);
        __threadfence_system();
    }
}

int ms_small_loop_blocks()
{
    int n = 0, m = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_ms_small_levels<false>, kMsW, 0) !=
            hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&m, k_ms_small_levels<true>, kMsW, 0) !=
            hipSuccess)
        return 0;
    return n < m ? n : m;
}

hipError_t launch_ms_small_levels(hipStream_t s, int wgs, int cls, int32_t V, const int64_t* off,
                                  const int32_t* col, const int32_t* orig, SeenNext* sn,
                                  uint64_t* front, int32_t* Qa, int32_t* Qb, int32_t* found,
                                  int16_t* const* lane_out, const int32_t* lane_start,
                                  MsSync* sy, uint64_t* slots, Ctrl* ctrl, Ctrl* h_ctrl,
                                  int32_t max_levels, int32_t qlimit, int64_t rlimit,
                                  int32_t dlimit, int32_t maxdeg)
{
    // an ordinary launch: the workgroups that take part are few enough to be
    // resident at once, and a cooperative launch would make the runtime stop
    // overlapping later kernels of other streams
    if (wgs < 1 || wgs > kMsMaxWGs) return hipErrorInvalidValue;
    if (V < kMsMinV) wgs = 1;  // the slots fit the smallest region
    const bool rows = maxdeg <= kMsRowEdges && maxdeg <= dlimit &&
                      (int64_t)qlimit * kMsRowEdges <= rlimit;
    hipLaunchKernelGGL(rows ? k_ms_small_levels<true> : k_ms_small_levels<false>,
                       dim3(wgs * kXcdSlices), dim3(kMsW), 0, s, V, off, col, orig, sn, front, Qa,
                       Qb, found, lane_out, lane_start, sy, slots, ctrl, h_ctrl, cls, max_levels,
                       qlimit, rlimit, dlimit);
    return hipGetLastError();
}

}  // namespace bfsmi
