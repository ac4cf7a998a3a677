// Bottom-up steps of the direction-optimizing search (the variant the paper
// discusses among related work: a level is searched from the unvisited
// vertices, each looking for one neighbour in the frontier, instead of from
// the frontier's edges), and the symmetry check that guards it.
//
// A bottom-up step for depth lvl runs over every vertex id that has a
// neighbour (under degree order the ids below the count of such vertices).  An unvisited
// vertex scans its row in stored order and stops at the first neighbour that
// was visited when the step began; that neighbour is its parent.  At the
// start of the step the visited set is exactly the vertices of depth
// <= lvl - 1, and an unvisited vertex (depth >= lvl) has no neighbour of
// depth <= lvl - 2 in a symmetric graph, so any visited neighbour lies in
// the frontier (depth lvl - 1): probing the visited bitmap is the frontier
// test.  Under degree order each row lists its lowest ids (the hubs) first.
//
// The visited bitmap is read from vis_old, a copy taken when the step
// begins and not written during it; the new bits go to vis, each wave
// writing the two words of its own 64 vertices.  Afterwards vis & ~vis_old is
// the next frontier, as after a top-down level in bitmap form.
#include <algorithm>

#include "bfs_internal.h"
#include "wave_ops.h"

namespace bfsmi {

// vis_old := vis (the snapshot the step probes); clears the step's counters.
__global__ __launch_bounds__(kWG) void k_bu_begin(int32_t W, const uint32_t* __restrict__ vis,
                                                  uint32_t* __restrict__ vis_old, int32_t lvl,
                                                  Ctrl* __restrict__ ctrl)
{
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t i = (int64_t)blockIdx.x * kWG + threadIdx.x; i < W; i += stride) {
        const uint32_t x = vis[i];
        if (vis_old[i] != x) vis_old[i] = x;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctrl->qn_count = 0;
        ctrl->bitmap_out = 1;  // a switch back converts vis & ~vis_old to a queue
        ctrl->level = lvl;
        ctrl->bu_found = 0;
        ctrl->bu_deg = 0;
        ctrl->bu_edges = 0;
        ctrl->next_deg = 0;
    }
}

// One wave per 64 consecutive vertex ids (two bitmap words), a lane per vertex,
// walking its row kBuU neighbours at a time.  The step is bound by the chain
// of dependent loads (bitmap word, row offsets, neighbours, their bitmap
// words), so a wave works on four units at once: it loads the bitmap words of
// the third unit ahead, the offsets of the second and the first neighbours of
// the next before it probes the current one's.  Bits of the lowest kBuHot
// ids, which under degree order are the ones that rows list first, are probed
// in LDS; two workgroups of 1024 threads a CU share its 160 KB.  The
// three steps of an R-MAT 24 search (8.9M ids with a neighbour), against
// unpipelined lanes, probes in memory and three atomics a wave: 509 + 350 +
// 300 -> 202 + 80 + 38 us.  (16-byte loads of four neighbours, long rows one a
// wave and the last rows of a wave by all its lanes were no faster.)
constexpr int kBuWG = 1024;
constexpr int kBuHot = 1 << 19;
constexpr int kBuU = 4;

__global__ __launch_bounds__(kBuWG, 8) void k_bottom_up(int32_t V, int32_t V_scan, int32_t W,
                                                        const int64_t* __restrict__ off,
                                                        const int32_t* __restrict__ col,
                                                        const int32_t* __restrict__ orig,
                                                        uint32_t* __restrict__ vis,
                                                        const uint32_t* __restrict__ snap,
                                                        int32_t* __restrict__ level,
                                                        int32_t* __restrict__ parent, int32_t lvl,
                                                        Ctrl* __restrict__ ctrl)
{
    constexpr int U = kBuU;
    __shared__ uint32_t s_hot[kBuHot / 32];
    const int lane = __lane_id();
    const int32_t nhot = W < kBuHot / 32 ? W : kBuHot / 32;
    for (int i = threadIdx.x; i < nhot; i += kBuWG) s_hot[i] = snap[i];
    __syncthreads();
    const int32_t hot = nhot * 32;  // ids below it are probed in LDS
    const int64_t nwaves = (int64_t)gridDim.x * (kBuWG / 64);
    const int64_t nunits = ((int64_t)V_scan + 63) / 64;
    uint32_t found_n = 0;
    int64_t found_deg = 0, examined = 0;
    // unit's bitmap word of this lane (all ones past the end)
    auto load_word = [&](int64_t unit) {
        const int64_t v = unit * 64 + lane;
        return v < V_scan ? snap[v >> 5] : ~0u;
    };
    // row [a, b) of this lane's vertex, empty where it is visited (loads are
    // unconditional, of valid ids, here and below: behind a branch the compiler
    // waits for each before it issues the next)
    auto load_row = [&](int64_t unit, uint32_t word, int64_t& a, int64_t& b) {
        const bool open = !((word >> (lane & 31)) & 1u);
        a = b = 0;
        if (!__any(open)) return;
        const int64_t v = open ? unit * 64 + lane : 0;
        const int64_t x = off[v], y = off[v + 1];
        a = open ? x : 0;
        b = open ? y : 0;
    };
    auto load_block = [&](int64_t e, int64_t b, int32_t (&u)[U]) {
        if (!__any(e < b)) return;
#pragma unroll
        for (int k = 0; k < U; ++k) u[k] = col[e + k < b ? e + k : 0];
    };
    int64_t unit = (int64_t)blockIdx.x * (kBuWG / 64) + (threadIdx.x >> 6);
    uint32_t w0 = load_word(unit), w1 = load_word(unit + nwaves), w2 = load_word(unit + 2 * nwaves);
    int64_t a0, b0, a1, b1, a2, b2;
    int32_t u0[U], u1[U];
    load_row(unit, w0, a0, b0);
    load_row(unit + nwaves, w1, a1, b1);
    load_block(a0, b0, u0);
    for (; unit < nunits; unit += nwaves) {
        const uint32_t w3 = load_word(unit + 3 * nwaves);
        load_row(unit + 2 * nwaves, w2, a2, b2);
        load_block(a1, b1, u1);
        int32_t par = -1;
        for (int64_t e = a0;; e += U) {
            if (e > a0) load_block(par < 0 ? e : b0, b0, u0);
            if (par < 0 && e < b0) {
                // ids in LDS, then the others
                uint32_t hit = 0, cold = 0;
#pragma unroll
                for (int k = 0; k < U; ++k) {
                    const bool in = e + k < b0;
                    const bool lds = in && u0[k] < hot;
                    const uint32_t w = s_hot[lds ? u0[k] >> 5 : 0];
                    const bool h = lds && ((w >> (u0[k] & 31)) & 1u);
                    hit |= (h ? 1u : 0u) << k;
                    cold |= (in && !lds ? 1u : 0u) << k;
                }
                // an id outside LDS counts if it comes before the first hit
                if (hit) cold &= (hit & (0u - hit)) - 1u;
                if (cold) {
                    uint32_t w[U];
#pragma unroll
                    for (int k = 0; k < U; ++k) w[k] = snap[((cold >> k) & 1u) ? u0[k] >> 5 : 0];
#pragma unroll
                    for (int k = 0; k < U; ++k)
                        if ((cold >> k) & 1u) hit |= ((w[k] >> (u0[k] & 31)) & 1u) << k;
                }
                const int first = hit ? __builtin_ctz(hit) : U;
#pragma unroll
                for (int k = 0; k < U; ++k)
                    if (k == first) par = u0[k];
                examined += hit ? first + 1 : (b0 - e < U ? b0 - e : U);
            }
            if (!__any(par < 0 && e + U < b0)) break;
        }
        const bool got = par >= 0;
        const int64_t v = unit * 64 + lane;
        const uint64_t mask = __ballot(got);
        if (got) {
            level[v] = lvl;
            if (parent) parent[v] = orig ? orig[par] : par;
            found_deg += b0 - a0;
        }
        found_n += got ? 1u : 0u;
        const uint32_t lo = (uint32_t)mask, hi = (uint32_t)(mask >> 32);
        if (lane == 0 && lo) vis[unit * 2] = w0 | lo;
        if (lane == 32 && hi) vis[unit * 2 + 1] = w0 | hi;
        w0 = w1;
        w1 = w2;
        w2 = w3;
        a0 = a1;
        b0 = b1;
        a1 = a2;
        b1 = b2;
#pragma unroll
        for (int k = 0; k < U; ++k) u0[k] = u1[k];
    }
    // one update per workgroup: the atomics on a counter take 12 ns each, one
    // after the other (8192 waves made them 300 us of every step)
    for (int d = 32; d >= 1; d >>= 1) {
        found_n += __shfl_xor(found_n, d, 64);
        found_deg += __shfl_xor(found_deg, d, 64);
        examined += __shfl_xor(examined, d, 64);
    }
    __shared__ int64_t s_sum[3][kBuWG / 64];
    if (lane == 0) {
        s_sum[0][threadIdx.x >> 6] = found_n;
        s_sum[1][threadIdx.x >> 6] = found_deg;
        s_sum[2][threadIdx.x >> 6] = examined;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        int64_t x = 0;
        for (int k = 0; k < kBuWG / 64; ++k) x += s_sum[threadIdx.x][k];
        if (x && threadIdx.x == 0) atomicAdd(&ctrl->bu_found, (uint32_t)x);
        if (x && threadIdx.x == 1)
            atomicAdd((unsigned long long*)&ctrl->bu_deg, (unsigned long long)x);
        if (x && threadIdx.x == 2)
            atomicAdd((unsigned long long*)&ctrl->bu_edges, (unsigned long long)x);
    }
}

// Vertices of at least each of four degrees (creation time: under degree
// order they are exactly the internal ids below each count; a bottom-up step
// need not look at ids without a neighbour, which no search can reach).
__global__ __launch_bounds__(kWG) void k_count_degrees(int32_t V, const int64_t* __restrict__ off,
                                                       const uint32_t* __restrict__ xo,
                                                       uint32_t* __restrict__ out,
                                                       unsigned long long* __restrict__ slices)
{
    __shared__ unsigned long long s_n[4 + kXcdSlices];
    if (threadIdx.x < 4 + kXcdSlices) s_n[threadIdx.x] = 0;
    __syncthreads();
    uint32_t n[4] = {0, 0, 0, 0};
    int64_t x[kXcdSlices] = {};
    const int64_t stride = (int64_t)gridDim.x * kWG;
    for (int64_t v = (int64_t)blockIdx.x * kWG + threadIdx.x; v < V; v += stride) {
        const int64_t d = off[v + 1] - off[v];
        n[0] += d >= 1 ? 1u : 0u;
        n[1] += d >= kPullLow ? 1u : 0u;
        n[2] += d >= kPullMid ? 1u : 0u;
        n[3] += d >= kPullHub ? 1u : 0u;
        const uint32_t* st = xo + v * kXcdSlices;
#pragma unroll
        for (int s = 0; s < kXcdSlices; ++s)
            x[s] += (s + 1 < kXcdSlices ? (int64_t)st[s + 1] : d) - (int64_t)st[s];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (n[i]) atomicAdd(&s_n[i], (unsigned long long)n[i]);
#pragma unroll
    for (int s = 0; s < kXcdSlices; ++s)
        if (x[s]) atomicAdd(&s_n[4 + s], (unsigned long long)x[s]);
    __syncthreads();
    const int t = threadIdx.x;
    if (t < 4 && s_n[t]) atomicAdd(&out[t], (uint32_t)s_n[t]);
    if (t >= 4 && t < 4 + kXcdSlices && s_n[t]) atomicAdd(&slices[t - 4], s_n[t]);
}

hipError_t launch_count_degrees(hipStream_t s, int grid, int32_t V, const int64_t* off,
                                const uint32_t* xo, uint32_t* out, unsigned long long* slices)
{
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(k_count_degrees, dim3(grid), dim3(kWG), 0, s, V, off, xo, out,
                       slices);
    return hipGetLastError();
}

hipError_t launch_bottom_up(hipStream_t s, int grid, int num_cus, int32_t V, int32_t V_scan,
                            int32_t W, const int64_t* off, const int32_t* col, const int32_t* orig,
                            uint32_t* vis, uint32_t* vis_old, int32_t* level, int32_t* parent,
                            int32_t lvl, Ctrl* ctrl)
{
    if (grid < 1) grid = 1;
    const int64_t wgrid = std::min<int64_t>(grid, ((int64_t)W + kWG - 1) / kWG);
    hipLaunchKernelGGL(k_bu_begin, dim3((unsigned)std::max<int64_t>(wgrid, 1)), dim3(kWG), 0, s, W,
                       vis, vis_old, lvl, ctrl);
    if (V_scan < 0 || V_scan > V) V_scan = V;
    const int64_t units = ((int64_t)V_scan + 63) / 64;
    const int64_t bgrid = std::min<int64_t>(2 * (int64_t)num_cus, (units + kBuWG / 64 - 1) / (kBuWG / 64));
    hipLaunchKernelGGL(k_bottom_up, dim3((unsigned)std::max<int64_t>(bgrid, 1)), dim3(kBuWG), 0, s,
                       V, V_scan, W, off, col, orig, vis, vis_old, level, parent, lvl, ctrl);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Symmetry check at graph creation: the CSR is symmetric iff its edge
// multiset equals its reverse.  Both multisets are summarised by wrapping
// 64-bit sums of a mixed hash of (u, v) and of (v, u), two independent
// hashes each; equal sums are taken as symmetric (a non-symmetric CSR passes
// only if both pairs of 64-bit sums collide).  The mixing function is the
// SplitMix64 finaliser (Steele, Lea and Flood, 2014).

__device__ __forceinline__ uint64_t mix64(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

__global__ __launch_bounds__(kWG) void k_symmetry_sums(int32_t V, const int64_t* __restrict__ off,
                                                       const int32_t* __restrict__ col,
                                                       unsigned long long* __restrict__ sums)
{
    const int lane = __lane_id();
    const int64_t nwaves = (int64_t)gridDim.x * (kWG / 64);
    uint64_t f1 = 0, f2 = 0, r1 = 0, r2 = 0;
    for (int64_t u = (int64_t)blockIdx.x * (kWG / 64) + (threadIdx.x >> 6); u < V; u += nwaves) {
        const int64_t a = off[u], b = off[u + 1];
        for (int64_t e = a + lane; e < b; e += 64) {
            const uint64_t v = (uint32_t)col[e];
            const uint64_t fw = ((uint64_t)u << 32) | v, rv = (v << 32) | (uint64_t)u;
            f1 += mix64(fw);
            r1 += mix64(rv);
            f2 += mix64(fw ^ 0x5851f42d4c957f2dull);
            r2 += mix64(rv ^ 0x5851f42d4c957f2dull);
        }
    }
    for (int d = 32; d >= 1; d >>= 1) {
        f1 += __shfl_xor(f1, d, 64);
        f2 += __shfl_xor(f2, d, 64);
        r1 += __shfl_xor(r1, d, 64);
        r2 += __shfl_xor(r2, d, 64);
    }
    if (lane == 0) {
        atomicAdd(&sums[0], (unsigned long long)f1);
        atomicAdd(&sums[1], (unsigned long long)f2);
        atomicAdd(&sums[2], (unsigned long long)r1);
        atomicAdd(&sums[3], (unsigned long long)r2);
    }
}

hipError_t launch_symmetry_sums(hipStream_t s, int grid, int32_t V, const int64_t* off,
                                const int32_t* col, unsigned long long* sums)
{
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(k_symmetry_sums, dim3(grid), dim3(kWG), 0, s, V, off, col, sums);
    return hipGetLastError();
}

}  // namespace bfsmi
