// Multi-source batch search: up to 64 independent searches in one pass.
//
// Lane b of a 64-bit mask per vertex belongs to root b.  seen[v] holds the
// lanes that reached v, front[v] the lanes for which v is in this level's
// frontier, next[v] the lanes that found v during this level; seen and next
// sit side by side (SeenNext), so one 16-byte load tests both.  A level is
// the paper's frontier expansion (Section 3.4) run once over the union
// frontier {v : front[v] != 0}: the same degree scan and edge -> thread
// mapping, with the visited test and claim done on whole masks,
//   next[v] |= front[u] & ~(seen[v] | next[v])   (64-bit atomic OR, no
//   return value, skipped when no lane is new),
// then a finalize pass turns next into the new frontier (new = next & ~seen),
// writes level L into row b of the output for every new lane b, and
// compacts the union frontier.  Lanes never interact, so each row equals the
// single-root search from its root.
//
// When the union frontier is small (at most V/64 vertices of a graph above
// 2^18: deep, narrow searches such as grids), the expansion also marks each vertex it finds in
// a touched bitmap, the old frontier's masks are cleared through the queue,
// and the finalize pass only does work for touched vertices, so a level
// costs O(frontier + V/32) instead of O(V).
//
// Every launch reads its sizes from ctrl and returns at once when
// ctrl->done is set, so a fixed sequence of levels can be captured in a
// hipGraph and replayed until the frontier is empty.
#include "bfs_internal.h"
#include "tile_map.h"
#include "wave_ops.h"

namespace bfsmi {

// Largest union frontier of a sparse level (see the file comment).  On small
// graphs no level is: a finalize that writes every vertex's frontier mask costs
// less there than the launch that clears the old ones and the atomics that
// mark what was found (5 roots, plain graph of 50,021 vertices, with the
// finalize's smaller chunks 280 -> 219 us; 64 roots, R-MAT 16 352 -> 322).  Sparse
// against dense at 2^18 vertices: 5 roots of a plain R-MAT 335 / 318 us, a 512 x 512
// grid by level kernels 19.3 / 18.4 ms; sparse levels pay from 2^21 on, on deep
// graphs (1448 x 1448 51.7 / 57.9 ms, a binary tree of 2^23 ids 2.21 / 2.29; R-MAT 23
// 4.40 / 4.33).
constexpr int32_t kMsDenseV = 1 << 18;
__host__ __device__ constexpr int32_t ms_sparse_limit(int32_t V)
{
    return V <= kMsDenseV ? -1 : V / 64;
}

__global__ __launch_bounds__(kWG) void k_ms_clear(int32_t V, int32_t n_roots,
                                                  SeenNext* __restrict__ sn,
                                                  uint64_t* __restrict__ front,
                                                  uint32_t* __restrict__ touched,
                                                  int8_t* __restrict__ out8, int vec)
{
    const int64_t stride = (int64_t)gridDim.x * kWG;
    const int64_t tid = (int64_t)blockIdx.x * kWG + threadIdx.x;
    for (int64_t v = tid; v < V; v += stride) {
        sn[v] = SeenNext{0ull, 0ull};
        front[v] = 0;
    }
    for (int64_t w = tid; w < ((int64_t)V + 31) / 32; w += stride) touched[w] = 0;
    const int64_t nbytes = (int64_t)n_roots * V;
    int64_t done = 0;
    if (vec) {
        int4* o4 = reinterpret_cast<int4*>(out8);
        const int4 m1 = make_int4(-1, -1, -1, -1);
        for (int64_t i = tid; i < nbytes / 16; i += stride) o4[i] = m1;
        done = nbytes / 16 * 16;
    }
    for (int64_t i = done + tid; i < nbytes; i += stride) out8[i] = -1;
}

// out8: the rows the level kernels write (ctrl->out8); null when they record
// the levels as planes instead.
__global__ __launch_bounds__(kWG) void k_ms_roots(int32_t V, int32_t n_roots,
                                                  const int32_t* __restrict__ roots,
                                                  const int32_t* __restrict__ rank,
                                                  SeenNext* __restrict__ sn,
                                                  uint64_t* __restrict__ front,
                                                  int8_t* __restrict__ out8,
                                                  int32_t* __restrict__ Q,
                                                  Ctrl* __restrict__ ctrl)
{
    __shared__ int32_t s_x[64];
    __shared__ int32_t s_n;
    const int b = threadIdx.x;
    if (b == 0) s_n = 0;
    if (b < n_roots) {
        const int32_t r = roots[b];
        s_x[b] = rank ? rank[r] : r;
        if (out8) out8[(int64_t)b * V + r] = 0;
    }
    __syncthreads();
    if (b < n_roots) {
        const int32_t x = s_x[b];
        uint64_t lanes = 0;
        bool first = true;
        for (int c = 0; c < n_roots; ++c) {
            if (s_x[c] == x) {
                lanes |= 1ull << c;
                if (c < b) first = false;
            }
        }
        if (first) {
            sn[x].seen = lanes;
            front[x] = lanes;
            Q[atomicAdd(&s_n, 1)] = x;
        }
    }
    __syncthreads();
    if (b == 0) {
        ctrl->qlen = s_n;
        ctrl->qn_count = 0;
        ctrl->level = 1;
        ctrl->done = 0;
        ctrl->err = 0;
        ctrl->overflow = 0;
        ctrl->r = 0;
        ctrl->ntiles = 0;
        ctrl->r_total = 0;
        ctrl->reached = s_n;
        ctrl->levels = 1;
        ctrl->alive = 0;
        ctrl->last_alive = 0;
        ctrl->out8 = out8;
        ctrl->full_prefix = 0;
        ctrl->fp_cand = 0x7fffffff;
        ctrl->skipped = 0;
        ctrl->next_deg = 0;
        ctrl->pull = 0;
        ctrl->no_push = 0;
        ctrl->pack[0] = ctrl->pack[1] = 0;
        ctrl->dropped[0] = ctrl->dropped[1] = 0;
        ctrl->sparse_limit = ms_sparse_limit(V);
        ctrl->sparse = s_n <= ctrl->sparse_limit;
    }
}

hipError_t launch_ms_init(hipStream_t s, int grid, int32_t V, const int32_t* roots_dev,
                          int32_t n_roots, const int32_t* rank, SeenNext* sn, uint64_t* front,
                          uint32_t* touched, int8_t* out8, int32_t* Q, Ctrl* ctrl)
{
    if (grid < 1) grid = 1;
    const int vec = ((uintptr_t)out8 % 16) == 0;
    hipLaunchKernelGGL(k_ms_clear, dim3(grid), dim3(kWG), 0, s, V, out8 ? n_roots : 0, sn, front,
                       touched, out8, vec);
    hipLaunchKernelGGL(k_ms_roots, dim3(1), dim3(64), 0, s, V, n_roots, roots_dev, rank, sn, front,
                       out8, Q, ctrl);
    return hipGetLastError();
}

// Level planes (degree order).  The levels of a batch are at most 127 and
// usually below 8, so the level kernels record a level by its binary digits:
// plane k holds, per vertex, the lanes whose level has bit k set, and a level
// costs one 8-byte OR per set bit and vertex that got new lanes instead of
// one byte store per lane.  The finalize of level 2^k writes plane k for
// every vertex, so the planes need no clearing.
//
// At the end the caller's rows are written once from the planes: out8[b][c] =
// the bits of lane b in the planes of x = rank[c] where lane b has seen x,
// else -1.  A thread takes four caller ids; after a 4 x 4 byte transpose of
// their masks, one shift and one mask give a bit of all four ids for a lane,
// so a lane's four bytes cost a dozen instructions and one 4-byte store (256
// contiguous bytes per wave and row).  The kernel is bound by those stores:
// R-MAT 22, 64 roots (268 MB of rows) 117 us; rows stored by
// internal id level by level and reordered byte by byte took 670 us, and
// 384 us of finalize against 268.  Ids go to workgroups in runs of
// 4096 (the relabelling's unit, one contiguous internal range per degree
// class), so the gathers reuse lines.
constexpr int kReorderChunk = 4096;

// T[g] byte i = byte g of w[i].
__device__ __forceinline__ void transpose_bytes(const uint32_t (&w)[4], uint32_t* T)
{
    const uint32_t a0 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u);
    const uint32_t a1 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
    const uint32_t b0 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
    const uint32_t b1 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
    T[0] = __builtin_amdgcn_perm(b0, a0, 0x05040100u);
    T[1] = __builtin_amdgcn_perm(b0, a0, 0x07060302u);
    T[2] = __builtin_amdgcn_perm(b1, a1, 0x05040100u);
    T[3] = __builtin_amdgcn_perm(b1, a1, 0x07060302u);
}

__device__ __forceinline__ void transpose_masks(const uint64_t (&m)[4], uint32_t (&T)[8])
{
    const uint32_t lo[4] = {(uint32_t)m[0], (uint32_t)m[1], (uint32_t)m[2], (uint32_t)m[3]};
    const uint32_t hi[4] = {(uint32_t)(m[0] >> 32), (uint32_t)(m[1] >> 32), (uint32_t)(m[2] >> 32),
                            (uint32_t)(m[3] >> 32)};
    transpose_bytes(lo, T);
    transpose_bytes(hi, T + 4);
}

// VEC: the thread's ids are four consecutive ones (4-byte stores; V and out8
// multiples of 4), else they are kWG apart (byte stores).
template <int NP, bool VEC>
__global__ __launch_bounds__(kWG) void k_ms_rows(int32_t V, int32_t n_roots,
                                                 const int32_t* __restrict__ rank,
                                                 const SeenNext* __restrict__ sn,
                                                 const uint64_t* __restrict__ planes,
                                                 int8_t* __restrict__ out8)
{
    const int64_t nchunks = ((int64_t)V + kReorderChunk - 1) / kReorderChunk;
    for (int64_t ch = blockIdx.x; ch < nchunks; ch += gridDim.x) {
        for (int j = 0; j < kReorderChunk / (4 * kWG); ++j) {
            const int64_t c0 = ch * kReorderChunk + j * 4 * kWG + (VEC ? 4 : 1) * threadIdx.x;
            constexpr int step = VEC ? 1 : kWG;
            if (c0 >= V) continue;
            int32_t x[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t c = c0 + i * step;
                x[i] = rank[c < V ? c : c0];
            }
            uint64_t m[4];
            uint32_t S[8], P[NP][8];
#pragma unroll
            for (int i = 0; i < 4; ++i) m[i] = sn[x[i]].seen;
            transpose_masks(m, S);
#pragma unroll
            for (int k = 0; k < NP; ++k) {
#pragma unroll
                for (int i = 0; i < 4; ++i) m[i] = planes[(int64_t)k * V + x[i]];
                transpose_masks(m, P[k]);
            }
            int8_t* o = out8 + c0;
#pragma unroll
            for (int g = 0; g < 8; ++g) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    if (8 * g + i < n_roots) {  // uniform
                        const uint32_t not_seen = ~(S[g] >> i) & 0x01010101u;
                        uint32_t lv = (not_seen << 8) - not_seen;  // 0xff where not seen
#pragma unroll
                        for (int k = 0; k < NP; ++k) lv |= ((P[k][g] >> i) & 0x01010101u) << k;
                        if (VEC) {
                            *reinterpret_cast<uint32_t*>(o) = lv;
                        } else {
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                if (c0 + q * step < V) o[q * step] = (int8_t)(lv >> (8 * q));
                        }
                        o += V;
                    }
                }
            }
        }
    }
}

hipError_t launch_ms_rows(hipStream_t s, int grid, int32_t V, int32_t n_roots, int32_t max_level,
                          const int32_t* rank, const SeenNext* sn, const uint64_t* planes,
                          int8_t* out8)
{
    const int64_t nchunks = ((int64_t)V + kReorderChunk - 1) / kReorderChunk;
    if (grid > nchunks) grid = (int)nchunks;
    if (grid < 1) grid = 1;
    // planes written: those of the powers of two up to the last level run
    int np = 1;
    while (np < kMsPlanes && (2 << (np - 1)) <= max_level) ++np;
    const bool vec = V % 4 == 0 && (uintptr_t)out8 % 4 == 0;
#define BFS_ROWS_CASE(N)                                                                          \
    case N:                                                                                      \
        if (vec)                                                                                 \
            hipLaunchKernelGGL((k_ms_rows<N, true>), dim3(grid), dim3(kWG), 0, s, V, n_roots, rank, \
                               sn, planes, out8);                                                \
        else                                                                                     \
            hipLaunchKernelGGL((k_ms_rows<N, false>), dim3(grid), dim3(kWG), 0, s, V, n_roots,     \
                               rank, sn, planes, out8);                                          \
        break;
    switch (np) {
        BFS_ROWS_CASE(1)
        BFS_ROWS_CASE(2)
        BFS_ROWS_CASE(3)
        BFS_ROWS_CASE(4)
        BFS_ROWS_CASE(5)
        BFS_ROWS_CASE(6)
        BFS_ROWS_CASE(7)
    default:
        return hipErrorInvalidValue;
    }
#undef BFS_ROWS_CASE
    return hipGetLastError();
}

// The level's degree scan in one launch (as k_list_scan of the single-root
// search): a workgroup reserves its entries and edges with one atomic on
// ctrl->pack[par], so entries lie in the order in which workgroups come.  The
// row prefix skip and the rows whose lanes are all searched from the unseen
// side as in k_scan_reduce.  A workgroup and pass takes 256 entries, 2048 of a
// queue that gives every workgroup more.  A level whose lanes are all searched
// from the unseen side is not scanned at all (ctrl->no_push; 45 us at each of
// two levels of R-MAT 22, 64 roots).
// With FUSE, the finalize writes the entries itself, for graphs whose next
// scan needs nothing that is known only after it (no prefix skip, no pull
// levels): one launch less, and no second pass over the queue.
// Against reduce, top and down as three launches a level and a read-back every
// 4 levels instead of 8: 5 roots on a plain graph of 50,021 vertices 364 ->
// 280 us, 64 roots on R-MAT 16 439 -> 346, R-MAT 22 2,480 -> 2,270.
struct MsScan {
    int64_t* rowstart;
    int32_t* uidv;
    int64_t* cumul;
    int32_t* tile_k;
    int tile_sh, par;
    int64_t max_edges;
};

template <int NI>
__device__ __forceinline__ void ms_scan_chunk(const int32_t* __restrict__ Q, int64_t q0, int32_t n,
                                              const int64_t* __restrict__ off,
                                              const int32_t* __restrict__ sk, uint64_t pull,
                                              const uint64_t* __restrict__ front, const MsScan& o,
                                              int32_t V, Ctrl* __restrict__ ctrl, uint32_t* s_wave,
                                              uint32_t* s_c, uint64_t* s_base, uint32_t& dropped)
{
    const int t = threadIdx.x;
    int32_t u[NI];
    int64_t a[NI];
    uint32_t d[NI], sum = 0;
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int32_t i = t * NI + j;
        u[j] = Q[q0 + (i < n ? i : n - 1)];
    }
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        a[j] = off[u[j]];
        d[j] = (uint32_t)(off[u[j] + 1] - a[j]);
    }
    if (sk) {
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int32_t x = sk[u[j]];
            a[j] += x;
            d[j] -= (uint32_t)x;
            dropped += t * NI + j < n ? (uint32_t)x : 0u;
        }
    }
    if (pull) {
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            if (!(front[u[j]] & ~pull)) {
                dropped += t * NI + j < n ? d[j] : 0u;
                d[j] = 0;
            }
        }
    }
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        if (t * NI + j >= n) d[j] = 0;
        sum += d[j];
    }
    uint32_t tot;
    uint32_t c = wg_exclusive_scan_dpp(sum, &tot, s_wave);
    if (t == 0)
        *s_base = atomicAdd(reinterpret_cast<unsigned long long*>(&ctrl->pack[o.par]),
                            ((unsigned long long)tot << kPackBits) | (unsigned long long)n);
    __syncthreads();
    const int32_t p0 = (int32_t)(*s_base & kPackMask);
    const int64_t c0 = (int64_t)(*s_base >> kPackBits);
    if ((int64_t)p0 + n > V || c0 + tot > o.max_edges) {
        ctrl->err = 1;  // more than the graph holds: refuse
        return;
    }
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int32_t i = t * NI + j;
        if (i < n) {
            s_c[i] = c;
            o.cumul[p0 + i] = c0 + c;
            o.rowstart[p0 + i] = a[j];
            o.uidv[p0 + i] = u[j];
        }
        c += d[j];
    }
    __syncthreads();
    write_tile_heads(s_c, n, tot, p0, c0, o.tile_sh, o.tile_k);
}

__global__ __launch_bounds__(kWG) void k_ms_scan(const int32_t* __restrict__ Q,
                                                 const int64_t* __restrict__ off, MsScan out,
                                                 Ctrl* __restrict__ ctrl,
                                                 const int32_t* __restrict__ skip, int32_t V,
                                                 const uint64_t* __restrict__ front)
{
    __shared__ uint32_t s_wave[kWG / 64];
    __shared__ uint32_t s_c[kWG * 8];
    __shared__ uint64_t s_base;
    if (ctrl->done || ctrl->no_push) return;
    const int32_t qlen = ctrl->qlen;
    const int32_t* sk = nullptr;
    if (skip) {
        const int32_t fp = ctrl->full_prefix;
        int lv = -1;
#pragma unroll
        for (int i = 0; i < kSkipLevels; ++i)
            if (fp >= (1 << (kSkipLow + i))) lv = i;
        if (lv >= 0) sk = skip + (int64_t)lv * V;
    }
    const uint64_t pull = front ? ctrl->pull : 0ull;
    const bool wide = qlen > (int64_t)gridDim.x * kWG;
    const int32_t chunk = wide ? kWG * 8 : kWG;
    int64_t dropped = 0;
    for (int64_t q0 = (int64_t)blockIdx.x * chunk; q0 < qlen; q0 += (int64_t)gridDim.x * chunk) {
        const int32_t n = (int32_t)(qlen - q0 < chunk ? qlen - q0 : chunk);
        uint32_t dr = 0;
        if (wide)
            ms_scan_chunk<8>(Q, q0, n, off, sk, pull, front, out, V, ctrl, s_wave, s_c, &s_base, dr);
        else
            ms_scan_chunk<1>(Q, q0, n, off, sk, pull, front, out, V, ctrl, s_wave, s_c, &s_base, dr);
        dropped += dr;
        __syncthreads();  // s_c, s_base are rewritten by the next chunk
    }
    if (sk || pull) {
        for (int o = 32; o >= 1; o >>= 1) dropped += __shfl_xor(dropped, o, 64);
        __shared__ int64_t s_drop[kWG / 64];
        if (__lane_id() == 0) s_drop[threadIdx.x >> 6] = dropped;
        __syncthreads();
        if (threadIdx.x == 0) {
            int64_t x = 0;
            for (int w = 0; w < kWG / 64; ++w) x += s_drop[w];
            if (x) atomicAdd(reinterpret_cast<unsigned long long*>(&ctrl->dropped[out.par]),
                             (unsigned long long)x);
        }
    }
}

template <int EPT>
__global__ __launch_bounds__(kWG) void k_ms_expand(const int64_t* __restrict__ rowstart,
                                                   const int32_t* __restrict__ uidv,
                                                   const int64_t* __restrict__ cumul,
                                                   const int32_t* __restrict__ tile_k,
                                                   const int32_t* __restrict__ col,
                                                   const uint64_t* __restrict__ front,
                                                   SeenNext* __restrict__ sn,
                                                   uint32_t* __restrict__ touched,
                                                   const Ctrl* __restrict__ ctrl, int par)
{
    __shared__ TileLds<EPT> L;
    if (ctrl->done || ctrl->err) return;
    const bool sparse = ctrl->sparse != 0;
    const uint64_t push = ~ctrl->pull;
    // par >= 0: scanned in one launch, edges and entries in ctrl->pack[par]
    const uint64_t pack = par >= 0 ? ctrl->pack[par] : 0ull;
    const int64_t r = par >= 0 ? (int64_t)(pack >> kPackBits) : ctrl->r;
    const int32_t ntiles = par >= 0 ? (int32_t)((r + kWG * EPT - 1) / (kWG * EPT)) : ctrl->ntiles;
    const int32_t k_last = par >= 0 ? (int32_t)(pack & kPackMask) - 1 : -1;
    StageRegs<EPT> cur = fetch_stage<EPT>(blockIdx.x, ntiles, cumul, rowstart, uidv, tile_k, k_last);
    for (int32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        int32_t uu[EPT], vv[EPT];
        bool ok[EPT];
        int64_t ee[EPT];
        map_tile<EPT>(L, cur, r, cumul, rowstart, uidv, col, uu, vv, ok, ee);
        cur = fetch_stage<EPT>(tile + gridDim.x, ntiles, cumul, rowstart, uidv, tile_k, k_last);
        // one 16-byte load gives both masks of the target: lanes that have
        // seen it, and lanes already recorded for the next level (a stale
        // pair only lets more threads issue the atomic)
        uint64_t f[EPT], have[EPT];
#pragma unroll
        for (int j = 0; j < EPT; ++j) f[j] = ok[j] ? front[uu[j]] & push : 0ull;
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            have[j] = ~0ull;
            if (f[j]) {
                const SeenNext p = sn[vv[j]];
                have[j] = p.seen | p.next;
            }
        }
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const uint64_t nb = f[j] & ~have[j];
            if (nb) {
                (void)__hip_atomic_fetch_or(&sn[vv[j]].next, nb, __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT);
                if (sparse)
                    (void)__hip_atomic_fetch_or(touched + (vv[j] >> 5), 1u << (vv[j] & 31),
                                                __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
    }
}

// Vertices per thread and chunk in the finalize: two on small graphs, whose
// chunks would else keep a tenth of the chip busy (eight against two, 5 and 64
// roots of a plain R-MAT: 2^14 222 / 181, 343 / 236 us, 2^17 291 / 257, 590 / 476;
// the curves cross between 2^18, 320 / 301, and 2^19, 471 / 492).
constexpr int kFinItems = 8, kFinItemsSmall = 2;
constexpr int32_t kFinSmallV = 1 << 17;

__device__ __forceinline__ uint64_t wave_or64(uint64_t x)
{
    for (int d = 1; d < 64; d <<= 1) x |= __shfl_xor(x, d, 64);
    return x;
}

// OUT16 = false: batch output, the level planes (degree order), or without
//                them int8 rows ctrl->out8[b][v] = level.
// OUT16 = true : serving output, lane b writes level - lane_start[b] into
//                its own int16 buffer lane_out[b] (caller ids).
template <bool OUT16, bool FUSE, int IT>
__global__ __launch_bounds__(kWG) void k_ms_finalize(int32_t V, const int32_t* __restrict__ orig,
                                                     SeenNext* __restrict__ sn,
                                                     uint64_t* __restrict__ front,
                                                     uint32_t* __restrict__ touched,
                                                     int32_t* __restrict__ Qn,
                                                     int16_t* const* __restrict__ lane_out,
                                                     const int32_t* __restrict__ lane_start,
                                                     Ctrl* __restrict__ ctrl,
                                                     const int64_t* __restrict__ deg_off,
                                                     uint64_t* __restrict__ planes, MsScan next)
{
    __shared__ uint32_t s_c[FUSE ? kWG * IT : 1];
    __shared__ uint64_t s_wave2[kWG / 64], s_pack;
    __shared__ int16_t* s_out[64];
    __shared__ int32_t s_start[64];
    __shared__ uint32_t s_wave[kWG / 64];
    __shared__ uint32_t s_base;
    __shared__ uint64_t s_alive[kWG / 64];
    __shared__ int64_t s_dsum[kWG / 64];
    if (ctrl->done) return;
    const int32_t lvl = ctrl->level;
    const bool sparse = ctrl->sparse != 0;
    int8_t* __restrict__ out8 = ctrl->out8;
    if (OUT16) {
        // the lane tables, once per workgroup
        if (threadIdx.x < 64) {
            s_out[threadIdx.x] = lane_out[threadIdx.x];
            s_start[threadIdx.x] = lane_start[threadIdx.x];
        }
        __syncthreads();
    }
    // A workgroup takes chunks of kWG * IT vertices; each chunk reserves its
    // queue slots with one atomicAdd (a per-wave add on the one counter
    // would serialise tens of thousands of atomics per level).
    constexpr int64_t chunk = (int64_t)kWG * IT;
    // level planes: the new lanes go to the planes of the level's set bits;
    // level 2^k writes plane k whole
    const bool plane_out = !OUT16 && planes && lvl <= 127;
    const bool whole = (lvl & (lvl - 1)) == 0;
    uint64_t alive = 0;
    int64_t dsum = 0;  // degrees of this thread's new union frontier entries
    for (int64_t c0 = (int64_t)blockIdx.x * chunk; c0 < V; c0 += (int64_t)gridDim.x * chunk) {
        uint64_t nw[IT];
        uint32_t cnt = 0;
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            const int64_t v = c0 + j * kWG + threadIdx.x;
            nw[j] = 0;
            bool hit = v < V;
            if (sparse && v < V) {
                // the 32 lanes of a word read it before its first lane clears it
                const uint32_t tw = touched[v >> 5];
                hit = (tw >> (v & 31)) & 1u;
                if ((v & 31) == 0 && tw) touched[v >> 5] = 0;
            }
            if (hit) {
                const SeenNext p = sn[v];
                if (p.next) {
                    nw[j] = p.next & ~p.seen;
                    sn[v] = SeenNext{p.seen | nw[j], 0ull};
                }
                front[v] = nw[j];
            }
            if (plane_out && v < V && (whole || nw[j])) {
                for (int32_t bits = lvl; bits; bits &= bits - 1) {
                    uint64_t* pl = planes + (int64_t)__builtin_ctz(bits) * V + v;
                    *pl = whole ? nw[j] : (*pl | nw[j]);
                }
            }
            cnt += nw[j] ? 1u : 0u;
        }
        uint32_t tot, ex, pos;
        if constexpr (FUSE) {
            // the next level's scan: rows and edge numbers of the new entries
            int64_t a[IT], a1[IT];
            uint64_t both = cnt;
#pragma unroll
            for (int j = 0; j < IT; ++j) {
                const int64_t v = c0 + j * kWG + threadIdx.x;
                a[j] = a1[j] = 0;
                if (nw[j]) {
                    a[j] = deg_off[v];
                    a1[j] = deg_off[v + 1];
                }
            }
#pragma unroll
            for (int j = 0; j < IT; ++j) both += (uint64_t)(a1[j] - a[j]) << kPackBits;
            uint64_t all;
            const uint64_t before = wg_exclusive_scan<uint64_t>(both, &all, s_wave2);
            tot = (uint32_t)(all & kPackMask);
            if (tot == 0) continue;  // uniform: no queue slots, no outputs
            if (threadIdx.x == 0)
                s_pack = atomicAdd(reinterpret_cast<unsigned long long*>(&ctrl->pack[next.par]),
                                   (unsigned long long)all);
            __syncthreads();
            const uint32_t p0 = (uint32_t)(s_pack & kPackMask);
            const int64_t e0 = (int64_t)(s_pack >> kPackBits);
            ex = (uint32_t)(before & kPackMask);
            pos = p0 + ex;
            if ((int64_t)p0 + tot <= V && e0 + (int64_t)(all >> kPackBits) <= next.max_edges) {
                uint32_t c = (uint32_t)(before >> kPackBits), i = ex;
#pragma unroll
                for (int j = 0; j < IT; ++j) {
                    if (!nw[j]) continue;
                    s_c[i] = c;
                    next.cumul[p0 + i] = e0 + c;
                    next.rowstart[p0 + i] = a[j];
                    next.uidv[p0 + i] = (int32_t)(c0 + j * kWG + threadIdx.x);
                    c += (uint32_t)(a1[j] - a[j]);
                    ++i;
                }
                __syncthreads();
                write_tile_heads(s_c, (int32_t)tot, (uint32_t)(all >> kPackBits), (int32_t)p0, e0,
                                 next.tile_sh, next.tile_k);
            } else {
                ctrl->err = 1;  // more than the graph holds: refuse
            }
        } else {
            ex = wg_exclusive_scan<uint32_t>(cnt, &tot, s_wave);
            if (tot == 0) continue;  // uniform: no queue slots, no outputs
            if (threadIdx.x == 0) s_base = atomicAdd(&ctrl->qn_count, tot);
            __syncthreads();
            pos = s_base + ex;
        }
#pragma unroll
        for (int j = 0; j < IT; ++j) {
            if (!nw[j]) continue;
            const int64_t v = c0 + j * kWG + threadIdx.x;
            if (pos < (uint32_t)V) Qn[pos] = (int32_t)v;
            else ctrl->err = 4;
            ++pos;
            if (!FUSE && deg_off) dsum += deg_off[v + 1] - deg_off[v];
            // each vertex writes only the lanes that reached it now
            if (OUT16) {
                const int64_t vo = orig ? orig[v] : v;
                for (uint64_t m = nw[j]; m; m &= m - 1) {
                    const int b = __builtin_ctzll(m);
                    const int32_t d = lvl - s_start[b];
                    if (d > 32767) ctrl->overflow = 1;
                    else if (s_out[b]) s_out[b][vo] = (int16_t)d;  // null: retired lane
                }
            } else if (lvl > 127) {
                ctrl->overflow = 1;
            }
            alive |= nw[j];
        }
        if (!OUT16 && !planes && lvl <= 127) {
            // lane b of a wave's vertices is one contiguous
            // (masked) store, lanes taken in the same order by every thread
#pragma unroll
            for (int j = 0; j < IT; ++j) {
                const int64_t v = c0 + j * kWG + threadIdx.x;
                for (uint64_t m = wave_or64(nw[j]); m; m &= m - 1) {
                    const int b = __builtin_ctzll(m);
                    if ((nw[j] >> b) & 1ull) out8[(int64_t)b * V + v] = (int8_t)lvl;
                }
            }
        }
        __syncthreads();  // s_base is rewritten by the next chunk
    }
    // one update of the level's lanes and degree sum per workgroup
    alive = wave_or64(alive);
    if (!FUSE && deg_off)
        for (int d = 32; d >= 1; d >>= 1) dsum += __shfl_xor(dsum, d, 64);
    if (__lane_id() == 0) {
        s_alive[threadIdx.x >> 6] = alive;
        s_dsum[threadIdx.x >> 6] = dsum;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t a = 0;
        int64_t ds = 0;
        for (int w = 0; w < kWG / 64; ++w) {
            a |= s_alive[w];
            ds += s_dsum[w];
        }
        if (a) atomicOr((unsigned long long*)&ctrl->alive, (unsigned long long)a);
        if (ds) atomicAdd((unsigned long long*)&ctrl->next_deg, (unsigned long long)ds);
    }
}

// Pull levels (symmetric, degree-ordered graphs).  At the dense levels of a
// small-world graph the expansion above is bound by its 64-bit atomics and
// 16-byte probes.  A lane of ctrl->pull is searched the other way round: a
// vertex that has not seen it ORs the frontier masks of its own row and
// takes the lanes it wants (the CSR equals its transpose, so the row lists
// the in-edges), stopping once every wanted lane is found.  The only writes
// are one mask per vertex that found something, without atomics (hub rows
// aside), and the rows of vertices that have seen every such lane are not
// read.  The lanes taken and the level's result are the expansion's.
//
// Rows are split by id range, which under degree order is by degree: rows of
// kPullHub edges or more are cut into kPullUnit-edge pieces, one wave each
// (their finds meet in sn[].next with an atomic OR); a wave takes one row of
// kPullMid edges or more, four rows of kPullLow or more, sixteen shorter ones.
constexpr int kPullUnit = 2048;

template <int CTRL>
__device__ __forceinline__ uint64_t dpp_or64(uint64_t x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), CTRL, 0xf, 0xf, true);
    return x | ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo;
}

// OR over aligned groups of G lanes (whole groups are active).
template <int G>
__device__ __forceinline__ uint64_t group_or64(uint64_t x)
{
    if (G >= 16) {
        x = dpp_or64<0x128>(x);  // row_ror:8
        x = dpp_or64<0x124>(x);  // row_ror:4
    }
    x = dpp_or64<0x4e>(x);  // quad_perm [2,3,0,1]
    x = dpp_or64<0xb1>(x);  // quad_perm [1,0,3,2]
    if (G == 64) {
        uint64_t y = 0;
#pragma unroll
        for (int r = 0; r < 64; r += 16) {
            const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, r);
            const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(x >> 32), r);
            y |= ((uint64_t)hi << 32) | lo;
        }
        x = y;
    }
    return x;
}

// The frontier lanes of edges [e, b) that want still lacks, read by a group
// of G lanes (lane l of it), 4 edges per lane and step, until none is left.
template <int G>
__device__ __forceinline__ uint64_t pull_edges(int64_t e, int64_t b, int l, uint64_t want,
                                               const int32_t* __restrict__ col,
                                               const uint64_t* __restrict__ front)
{
    uint64_t acc = 0;
    for (; e < b && (want & ~acc); e += 4 * G) {
        int32_t u[4];
        uint64_t f[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t i = e + k * G + l;
            u[k] = i < b ? col[i] : -1;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) f[k] = u[k] >= 0 ? front[u[k]] : 0ull;
        acc = group_or64<G>(acc | f[0] | f[1] | f[2] | f[3]);
    }
    return acc & want;
}

// One group of G lanes per row of [v0, v1), 64 / G rows per wave.
template <int G>
__device__ __forceinline__ void pull_rows(int64_t v0, int64_t v1, uint64_t pull,
                                          const int64_t* __restrict__ off,
                                          const int32_t* __restrict__ col,
                                          const uint64_t* __restrict__ front,
                                          SeenNext* __restrict__ sn)
{
    const int lane = __lane_id();
    const int64_t v = v0 + lane / G;
    if (v >= v1) return;  // whole groups
    const SeenNext p = sn[v];
    const uint64_t want = pull & ~p.seen;
    if (!want) return;
    const uint64_t got = pull_edges<G>(off[v], off[v + 1], lane % G, want, col, front);
    if (got && lane % G == 0) sn[v].next = p.next | got;
}

// After a level's expansion: the pull lanes, or at a sparse level (which has
// none) the old frontier's masks are cleared through the queue (after the
// expansion has read them, before the finalize writes new ones).
__global__ __launch_bounds__(kWG) void k_ms_pull(const int32_t* __restrict__ Q, PullRows R,
                                                 const int64_t* __restrict__ off,
                                                 const int32_t* __restrict__ col,
                                                 uint64_t* __restrict__ front,
                                                 SeenNext* __restrict__ sn,
                                                 const Ctrl* __restrict__ ctrl)
{
    if (ctrl->done) return;
    if (ctrl->sparse) {
        const int32_t qlen = ctrl->qlen;
        const int64_t stride = (int64_t)gridDim.x * kWG;
        for (int64_t k = (int64_t)blockIdx.x * kWG + threadIdx.x; k < qlen; k += stride)
            front[Q[k]] = 0;
        return;
    }
    const uint64_t pull = ctrl->pull;
    if (!pull) return;
    const int64_t e_hub = off[R.n_hub];
    const int64_t u0 = (e_hub + kPullUnit - 1) / kPullUnit;      // hub pieces
    const int64_t u1 = u0 + (R.n_wave - R.n_hub);                // one row each
    const int64_t u2 = u1 + ((int64_t)R.n_mid - R.n_wave + 3) / 4;
    const int64_t u3 = u2 + ((int64_t)R.n_act - R.n_mid + 15) / 16;
    const int64_t nwaves = (int64_t)gridDim.x * (kWG / 64);
    for (int64_t unit = (int64_t)(threadIdx.x >> 6) * gridDim.x + blockIdx.x; unit < u3;
         unit += nwaves) {
        if (unit >= u2) {
            const int64_t v = R.n_mid + (unit - u2) * 16;
            pull_rows<4>(v, R.n_act, pull, off, col, front, sn);
        } else if (unit >= u1) {
            const int64_t v = R.n_wave + (unit - u1) * 4;
            pull_rows<16>(v, R.n_mid, pull, off, col, front, sn);
        } else if (unit >= u0) {
            const int64_t v = R.n_hub + (unit - u0);
            pull_rows<64>(v, v + 1, pull, off, col, front, sn);
        } else {
            int64_t e = unit * kPullUnit;
            const int64_t end = e + kPullUnit < e_hub ? e + kPullUnit : e_hub;
            int32_t lo = 0, hi = R.n_hub - 1;  // the row holding edge e
            while (lo < hi) {
                const int32_t mid = (lo + hi + 1) >> 1;
                if (off[mid] <= e) lo = mid;
                else hi = mid - 1;
            }
            for (int32_t v = lo; e < end; ++v) {
                const int64_t b = off[v + 1] < end ? off[v + 1] : end;
                const SeenNext p = sn[v];
                const uint64_t want = pull & ~(p.seen | p.next);
                if (want) {
                    const uint64_t got = pull_edges<64>(e, b, __lane_id(), want, col, front);
                    if (got && __lane_id() == 0)
                        (void)__hip_atomic_fetch_or(&sn[v].next, got, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
                }
                e = b;
            }
        }
    }
}

// After a level's finalize: the first id, from the current prefix on, that
// some lane still searching (found vertices this level) has not seen.  Each
// workgroup takes 2048-id chunks in order and stops once a smaller candidate
// is known; k_ms_advance moves ctrl->full_prefix there (the prefix only
// grows: seen masks grow and the set of searching lanes shrinks).
constexpr int kPrefixChunk = kWG * 8;

__global__ __launch_bounds__(kWG) void k_ms_prefix(int32_t V, const SeenNext* __restrict__ sn,
                                                   Ctrl* __restrict__ ctrl)
{
    __shared__ int32_t s_min, s_known;
    if (ctrl->done) return;
    const uint64_t live = ctrl->alive;
    if (live == 0) return;  // the batch ends at this level
    const int32_t p0 = ctrl->full_prefix;
    for (int64_t c0 = (int64_t)p0 + (int64_t)blockIdx.x * kPrefixChunk; c0 < V;
         c0 += (int64_t)gridDim.x * kPrefixChunk) {
        if (threadIdx.x == 0) {
            s_min = 0x7fffffff;
            s_known = __hip_atomic_load(&ctrl->fp_cand, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        __syncthreads();
        if (c0 >= s_known) break;  // uniform (one read, shared through LDS)
#pragma unroll
        for (int j = 0; j < kPrefixChunk / kWG; ++j) {
            const int64_t x = c0 + j * kWG + threadIdx.x;
            if (x < V && (sn[x].seen & live) != live) atomicMin(&s_min, (int32_t)x);
        }
        __syncthreads();
        const int32_t m = s_min;
        if (m != 0x7fffffff) {
            if (threadIdx.x == 0) atomicMin(&ctrl->fp_cand, m);
            break;  // uniform
        }
        __syncthreads();  // s_min is reset for the next chunk
    }
}

// One wave.  nnz > 0: the next level may search lanes from the unseen side.
// It does when its union frontier points at more than 1/kPullShare of the
// edges (below that the push costs less than reading the rows: the levels of
// R-MAT 22 on either side of the line push in 25 and 840 us and pull in 50 and
// 350 us); the lanes are those that have seen at least kPullHubsSeen of the 64
// highest-degree vertices.  A lane that has not is still on its way to them:
// its frontier is cheap to expand, while searched the other way it would keep
// every vertex reading its whole row.  R-MAT 22, 64 roots, per batch: 1 of 64
// 3.34-3.42 ms, 8 3.20-3.26, 32 3.46, all 64 4.07, no pull levels 4.85-4.88.
constexpr int64_t kPullShare = 8;
constexpr int kPullHubsSeen = 8;

__global__ __launch_bounds__(64) void k_ms_advance(Ctrl* __restrict__ ctrl, int32_t V, int prefix,
                                                   const SeenNext* __restrict__ sn, int64_t nnz,
                                                   int par, int fused)
{
    if (ctrl->done) return;
    uint64_t core = 0;
    if (nnz > 0 && ctrl->next_deg * kPullShare > nnz) {
        // thread b: how many of those vertices lane b has seen
        const uint64_t s = threadIdx.x < V ? sn[threadIdx.x].seen : 0ull;
        int n = 0;
        for (int x = 0; x < 64; ++x) n += (int)((__shfl(s, x, 64) >> threadIdx.x) & 1ull);
        core = __ballot(n >= kPullHubsSeen);
    }
    if (threadIdx.x != 0) return;
    if (prefix) {
        // no candidate: every id from the old prefix on is seen by all live lanes
        const int32_t c = ctrl->fp_cand;
        ctrl->full_prefix = c < V ? c : V;
        ctrl->fp_cand = 0x7fffffff;
    }
    if (par >= 0) {  // the level's scan is spent
        ctrl->r_total += (int64_t)(ctrl->pack[par] >> kPackBits);
        ctrl->skipped += ctrl->dropped[par];
        ctrl->pack[par] = 0;
        ctrl->dropped[par] = 0;
    }
    const uint32_t q = fused ? (uint32_t)(ctrl->pack[par ^ 1] & kPackMask) : ctrl->qn_count;
    ctrl->sparse = (int32_t)q <= ctrl->sparse_limit;
    ctrl->last_alive = ctrl->alive;  // lanes that found vertices this level
    ctrl->pull = ctrl->sparse ? 0ull : core & ctrl->alive;
    // the whole frontier is searched from the unseen side: its scan would only
    // count the edges it drops, which are all of the frontier's
    ctrl->no_push = par >= 0 && ctrl->pull != 0 && !(ctrl->alive & ~ctrl->pull);
    if (ctrl->no_push) ctrl->skipped += ctrl->next_deg;
    ctrl->next_deg = 0;
    ctrl->alive = 0;
    ctrl->reached += q;
    ctrl->qlen = (int32_t)q;
    ctrl->qn_count = 0;
    if (q) ctrl->levels += 1;
    ctrl->level += 1;
    ctrl->done = (q == 0 || ctrl->overflow || ctrl->err) ? 1 : 0;
}

template <int EPT>
static void ms_expand_launch(hipStream_t s, int grid, const int64_t* rowstart, const int32_t* uidv,
                             const int64_t* cumul, const int32_t* tile_k, const int32_t* col,
                             const uint64_t* front, SeenNext* sn, uint32_t* touched,
                             const Ctrl* ctrl, int par)
{
    hipLaunchKernelGGL(k_ms_expand<EPT>, dim3(grid), dim3(kWG), 0, s, rowstart, uidv, cumul, tile_k,
                       col, front, sn, touched, ctrl, par);
}

int ms_expand_blocks_per_cu(int ept)
{
    int n = 0;
    hipError_t e = hipErrorInvalidValue;
    switch (ept) {
    case 1: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_ms_expand<1>, kWG, 0); break;
    case 2: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_ms_expand<2>, kWG, 0); break;
    case 4: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_ms_expand<4>, kWG, 0); break;
    case 8: e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k_ms_expand<8>, kWG, 0); break;
    default: break;
    }
    if (e != hipSuccess || n < 1) n = 1;
    return n;
}

hipError_t launch_ms_level(hipStream_t s, int scan_grid, int expand_grid, int fin_grid, int ept,
                           int32_t V, int64_t tile_cap, const int64_t* off, const int32_t* col,
                           const int32_t* orig, const int32_t* Q, int32_t* Qn, int32_t* deg,
                           int64_t* rowstart, int32_t* uidv, int64_t* bsum, int64_t* cumul,
                           int32_t* tile_k, SeenNext* sn, uint64_t* front, uint32_t* touched,
                           int16_t* const* lane_out, const int32_t* lane_start, Ctrl* ctrl,
                           const PullRows& pull, bool one, int level, bool last,
                           uint64_t* planes, const int32_t* skip, int prefix_grid)
{
    const bool prefix = skip != nullptr && prefix_grid > 0;
    const int64_t pull_nnz = pull.n_act > 0 ? pull.nnz : 0;
    const int64_t max_edges = (tile_cap - 1) * kMinTile;
    const bool can_fuse = one && !prefix && pull_nnz == 0;
    const int par = one ? level & 1 : -1;
    MsScan out{rowstart, uidv, cumul, tile_k, log2_tile(kWG * ept), par, max_edges};
    if (one && !(can_fuse && level > 0)) {
        hipLaunchKernelGGL(k_ms_scan, dim3(scan_grid < 1 ? 1 : scan_grid), dim3(kWG), 0, s, Q, off,
                           out, ctrl, prefix ? skip : nullptr, V, pull_nnz > 0 ? front : nullptr);
    } else if (!one) {
        const hipError_t e = launch_scan_dev(s, scan_grid, Q, off, nullptr, deg, rowstart, uidv, bsum,
                                             cumul, tile_k, tile_cap, kWG * ept, ctrl,
                                             prefix ? skip : nullptr, V,
                                             pull_nnz > 0 ? front : nullptr);
        if (e != hipSuccess) return e;
    }
    const bool fuse = can_fuse && !last;
    out.par ^= 1;
    if (expand_grid < 1) expand_grid = 1;
    switch (ept) {
    case 1: ms_expand_launch<1>(s, expand_grid, rowstart, uidv, cumul, tile_k, col, front, sn, touched, ctrl, par); break;
    case 2: ms_expand_launch<2>(s, expand_grid, rowstart, uidv, cumul, tile_k, col, front, sn, touched, ctrl, par); break;
    case 4: ms_expand_launch<4>(s, expand_grid, rowstart, uidv, cumul, tile_k, col, front, sn, touched, ctrl, par); break;
    case 8: ms_expand_launch<8>(s, expand_grid, rowstart, uidv, cumul, tile_k, col, front, sn, touched, ctrl, par); break;
    default: return hipErrorInvalidValue;
    }
    if (fin_grid < 1) fin_grid = 1;
    if (pull_nnz > 0 || V > kMsDenseV)  // else it has no lanes to search and nothing to clear
        hipLaunchKernelGGL(k_ms_pull, dim3(pull_nnz > 0 ? expand_grid : scan_grid), dim3(kWG), 0,
                           s, Q, pull, off, col, front, sn, ctrl);
    constexpr int L8 = kFinItems, L2 = kFinItemsSmall;
    const bool small = V <= kFinSmallV;
    const auto finalize =
        lane_out ? (fuse ? (small ? k_ms_finalize<true, true, L2> : k_ms_finalize<true, true, L8>)
                         : (small ? k_ms_finalize<true, false, L2> : k_ms_finalize<true, false, L8>))
                 : (fuse ? (small ? k_ms_finalize<false, true, L2> : k_ms_finalize<false, true, L8>)
                         : (small ? k_ms_finalize<false, false, L2> : k_ms_finalize<false, false, L8>));
    if (small) {  // a chunk per workgroup
        const int64_t chunks = ((int64_t)V + kWG * L2 - 1) / (kWG * L2);
        if (fin_grid < chunks) fin_grid = (int)chunks;
    }
    hipLaunchKernelGGL(finalize, dim3(fin_grid), dim3(kWG), 0, s, V, orig, sn, front, touched, Qn,
                       lane_out, lane_start, ctrl, fuse || pull_nnz > 0 ? off : nullptr, planes, out);
    if (prefix)
        hipLaunchKernelGGL(k_ms_prefix, dim3(prefix_grid), dim3(kWG), 0, s, V, sn, ctrl);
    hipLaunchKernelGGL(k_ms_advance, dim3(1), dim3(64), 0, s, ctrl, V, prefix ? 1 : 0, sn, pull_nnz,
                       par, fuse ? 1 : 0);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Serving: lanes join a running batch at a level boundary and retire when a
// level finds nothing for them.

__global__ __launch_bounds__(kWG) void k_srv_reset(int32_t V, SeenNext* __restrict__ sn,
                                                   uint64_t* __restrict__ front,
                                                   uint32_t* __restrict__ touched,
                                                   Ctrl* __restrict__ ctrl)
{
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t v = (int64_t)blockIdx.x * kWG + threadIdx.x; v < V; v += stride) {
        sn[v] = SeenNext{0ull, 0ull};
        front[v] = 0;
    }
    for (int64_t w = (int64_t)blockIdx.x * kWG + threadIdx.x; w < ((int64_t)V + 31) / 32; w += stride)
        touched[w] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctrl->qlen = 0;
        ctrl->qn_count = 0;
        ctrl->level = 1;
        ctrl->done = 1;  // nothing to expand until a lane joins
        ctrl->err = 0;
        ctrl->overflow = 0;
        ctrl->r = 0;
        ctrl->ntiles = 0;
        ctrl->r_total = 0;
        ctrl->reached = 0;
        ctrl->levels = 0;
        ctrl->alive = 0;
        ctrl->last_alive = 0;
        ctrl->out8 = nullptr;
        ctrl->next_deg = 0;
        ctrl->pull = 0;
        ctrl->no_push = 0;
        ctrl->pack[0] = ctrl->pack[1] = 0;
        ctrl->dropped[0] = ctrl->dropped[1] = 0;
        ctrl->sparse_limit = ms_sparse_limit(V);
        ctrl->sparse = 0 <= ctrl->sparse_limit;
    }
}

// Clear the retired lanes' bits from every vertex's seen mask.
__global__ __launch_bounds__(kWG) void k_srv_clear(int32_t V, SeenNext* __restrict__ sn,
                                                   uint64_t mask)
{
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t v = (int64_t)blockIdx.x * kWG + threadIdx.x; v < V; v += stride) {
        const uint64_t x = sn[v].seen;
        if (x & mask) sn[v].seen = x & ~mask;
    }
}

__global__ __launch_bounds__(kWG) void k_fill16(int16_t* __restrict__ p, int64_t n, int16_t val)
{
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < n; i += stride) p[i] = val;
}

// dst[i] = src[i] widened to int32, and *maxp = max(*maxp, max src[i]):
// delivery of a serving result into a device buffer of the caller.
__global__ __launch_bounds__(kWG) void k_widen16(const int16_t* __restrict__ src,
                                                 int32_t* __restrict__ dst, int64_t n,
                                                 int32_t* __restrict__ maxp)
{
    const int64_t stride = (int64_t)gridDim.x * kWG;
    int32_t m = -1;
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < n; i += stride) {
        const int32_t x = src[i];
        dst[i] = x;
        m = x > m ? x : m;
    }
    for (int d = 32; d >= 1; d >>= 1) {
        const int32_t o = __shfl_xor(m, d, 64);
        m = o > m ? o : m;
    }
    if ((threadIdx.x & 63) == 0 && m >= 0) atomicMax(maxp, m);
}

// Lane join_lane[i] starts a search from join_root[i] (caller id).  Its
// root gets depth 0; its first expansion is the next level, so
// lane_start = level - 1.  Roots not yet in the union frontier are appended.
__global__ void k_srv_join(int32_t V, int32_t n_join, const int32_t* __restrict__ join,
                           const int32_t* __restrict__ rank, SeenNext* __restrict__ sn,
                           uint64_t* __restrict__ front, int16_t* const* __restrict__ lane_out,
                           int32_t* __restrict__ lane_start, int32_t* __restrict__ Q,
                           Ctrl* __restrict__ ctrl)
{
    // join[2 * i] = root, join[2 * i + 1] = lane; one wave, n_join <= 64
    __shared__ int32_t s_app;
    const int i = threadIdx.x;
    if (i == 0) s_app = 0;
    __syncthreads();
    const int32_t qlen = ctrl->qlen;
    if (i < n_join) {
        const int32_t r = join[2 * i];
        const int32_t b = join[2 * i + 1];
        const int32_t x = rank ? rank[r] : r;
        const uint64_t bit = 1ull << b;
        atomicOr((unsigned long long*)&sn[x].seen, (unsigned long long)bit);
        const uint64_t old = atomicOr((unsigned long long*)&front[x], (unsigned long long)bit);
        lane_out[b][r] = 0;
        lane_start[b] = ctrl->level - 1;
        if (old == 0) {
            const int32_t pos = qlen + atomicAdd(&s_app, 1);
            if (pos < V) Q[pos] = x;
            else ctrl->err = 5;
        }
    }
    __syncthreads();
    if (i == 0) {
        ctrl->qlen = qlen + s_app;
        ctrl->sparse = ctrl->qlen <= ctrl->sparse_limit;
        ctrl->no_push = 0;  // the new lanes push
        ctrl->done = 0;
    }
}

hipError_t launch_srv_reset(hipStream_t s, int grid, int32_t V, SeenNext* sn, uint64_t* front,
                            uint32_t* touched, Ctrl* ctrl)
{
    hipLaunchKernelGGL(k_srv_reset, dim3(grid), dim3(kWG), 0, s, V, sn, front, touched, ctrl);
    return hipGetLastError();
}

hipError_t launch_srv_clear(hipStream_t s, int grid, int32_t V, SeenNext* sn, uint64_t mask)
{
    hipLaunchKernelGGL(k_srv_clear, dim3(grid), dim3(kWG), 0, s, V, sn, mask);
    return hipGetLastError();
}

hipError_t launch_fill16(hipStream_t s, int grid, int16_t* p, int64_t n, int16_t val)
{
    hipLaunchKernelGGL(k_fill16, dim3(grid), dim3(kWG), 0, s, p, n, val);
    return hipGetLastError();
}

hipError_t launch_widen16(hipStream_t s, int grid, const int16_t* src, int32_t* dst, int64_t n,
                          int32_t* maxp)
{
    hipLaunchKernelGGL(k_widen16, dim3(grid), dim3(kWG), 0, s, src, dst, n, maxp);
    return hipGetLastError();
}

hipError_t launch_srv_join(hipStream_t s, int32_t V, int32_t n_join, const int32_t* join,
                           const int32_t* rank, SeenNext* sn, uint64_t* front,
                           int16_t* const* lane_out, int32_t* lane_start, int32_t* Q, Ctrl* ctrl)
{
    hipLaunchKernelGGL(k_srv_join, dim3(1), dim3(64), 0, s, V, n_join, join, rank, sn, front,
                       lane_out, lane_start, Q, ctrl);
    return hipGetLastError();
}

}  // namespace bfsmi
