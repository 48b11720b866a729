// Directed pre-processing (Section 2.4): the in-CSR, the strongly connected
// components, and the reach bounds alpha(v) <= r(v) <= omega(v) from the
// weighted DAG of SCCs, w(C) = |C|, arcs taken as a set:
//     alpha(C) = w(C) + max over successors D of alpha(D)   (w(C) for a sink)
//     omega(C) = w(C) + sum over successors D of omega(D),  capped at n,
// evaluated in reverse topological order (a component once all of its
// successors are known).
//
// Optional refinement (end of Section 2.4, graph flag BC_BIG_SCC): the
// largest component T (largest w; among equals the one holding the smallest
// node id) takes its exact reach rT = |R(T)| from one breadth-first search
// instead of the recurrence, so alpha(T) = omega(T) = rT and the exact value
// flows into every component that reaches T.  Such a component C also gets
// the upper bound rT + omega'(C), where omega' is the same recurrence over
// the components outside R(T) only (what C reaches outside R(T) is exactly
// what it reaches in the DAG without R(T)); omega(C) is the smaller bound.
//
// SCCs are found on the GPU without recursion:
//   1. trim: a node with no remaining in-arc or no remaining out-arc is a
//      singleton SCC (repeated a few times);
//   2. forward-backward: the SCC of a high-degree pivot is the intersection
//      of its forward and backward reachable sets (finds the giant SCC);
//   3. colouring rounds on what is left: colour(v) = largest id that reaches
//      v (max-propagation along arcs); a node whose colour is its own id is a
//      root, and the SCC of root c is the set of nodes of colour c that reach
//      c through nodes of colour c.  Every round removes at least the SCC of
//      the largest remaining id.
#include <hipcub/hipcub.hpp>

#include "arcs.h"
#include "bc_internal.h"

namespace bc {

namespace {

constexpr int kBlk = 256;

inline unsigned grid_for(int64_t work, int64_t cap = 8192) {
    int64_t b = (work + kBlk - 1) / kBlk;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

#define GSTRIDE_LOOP(i, N)                                                      \
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (N);   \
         i += (int64_t)gridDim.x * blockDim.x)

__device__ inline int32_t ld_rel(const int32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// In-degrees and the in-CSR, one arc per thread (in-degrees over the grid, the
// rows of the in-CSR's arcs recovered tile by tile, see arcs.h).  Bound by the atomics on the targets' counters; with one
// thread per row the longest row set the time (R-MAT scale 18, 3.9M arcs:
// in-degrees 4376 -> 208 us, filling 6295 -> 222 us).
__global__ __launch_bounds__(kArcBlk) void k_indeg(int64_t m, const int32_t* __restrict__ col,
                                                   int32_t* __restrict__ icnt) {
    GSTRIDE_LOOP(e, m) atomicAdd(&icnt[col[e]], 1);
}

__global__ void k_close(int32_t* rp, int32_t n, const int32_t* cnt) {
    if (blockIdx.x == 0 && threadIdx.x == 0) rp[n] = n > 0 ? rp[n - 1] + cnt[n - 1] : 0;
}

__global__ __launch_bounds__(kArcBlk) void k_fill_in(int32_t n, int64_t m, const int32_t* __restrict__ rp,
                                                     const int32_t* __restrict__ col, const int32_t* __restrict__ irp,
                                                     int32_t* __restrict__ fill, int32_t* __restrict__ icol) {
    __shared__ ArcRowLds L;
    const int32_t e0 = tile_first(blockIdx.x), len = tile_arcs(e0, m);
    block_arc_rows(rp, n, e0, len, L);
    tile_each<kArcBlk>(threadIdx.x, len, [&](int32_t i) {
        const int32_t w = col[e0 + i];
        icol[irp[w] + atomicAdd(&fill[w], 1)] = L.row[i];
    });
}

__global__ void k_fill_i32(int64_t n, int32_t* p, int32_t v) {
    GSTRIDE_LOOP(i, n) p[i] = v;
}

// trim: active v (comp < 0) without an active out-neighbour or without an
// active in-neighbour becomes its own SCC
__global__ void k_trim(int32_t n, const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                       const int32_t* __restrict__ irp, const int32_t* __restrict__ icol, int32_t* comp,
                       int32_t* changed) {
    GSTRIDE_LOOP(v, n) {
        if (ld_rel(&comp[v]) >= 0) continue;
        bool out = false, in = false;
        for (int32_t i = rp[v]; i < rp[v + 1] && !out; ++i) {
            int32_t w = col[i];
            out = (w != (int32_t)v) && ld_rel(&comp[w]) < 0;
        }
        for (int32_t i = irp[v]; i < irp[v + 1] && !in; ++i) {
            int32_t w = icol[i];
            in = (w != (int32_t)v) && ld_rel(&comp[w]) < 0;
        }
        if (!out || !in) {
            __hip_atomic_store(&comp[v], (int32_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *changed = 1;
        }
    }
}

__global__ void k_pivot(int32_t n, const int32_t* __restrict__ rp, const int32_t* __restrict__ irp,
                        const int32_t* __restrict__ comp, unsigned long long* best) {
    unsigned long long mx = 0;
    GSTRIDE_LOOP(v, n) {
        if (comp[v] >= 0) continue;
        uint64_t a = (uint64_t)(rp[v + 1] - rp[v]), b = (uint64_t)(irp[v + 1] - irp[v]);
        uint64_t sc = a * b;
        if (sc > 0x7FFFFFFFull) sc = 0x7FFFFFFFull;
        mx = max(mx, (unsigned long long)((sc << 32) | (uint32_t)v));
    }
    block_extreme64(mx, best);
}

// A level of a breadth-first search restricted to active nodes: mark bit
// `bit` in mark[], true for a node that this arc marked first.  The plain
// read skips the atomic for nodes marked at an earlier level.
struct ReachOp {
    const int32_t* comp;
    uint32_t* mark;
    uint32_t bit;
    __device__ bool operator()(int32_t w, uint32_t) const {
        if (comp[w] >= 0 || (mark[w] & bit)) return false;
        return !(atomicOr(&mark[w], bit) & bit);
    }
};

__global__ void k_fwbw_assign(int32_t n, const uint32_t* __restrict__ mark, int32_t* comp, int32_t pivot) {
    GSTRIDE_LOOP(v, n) {
        if (comp[v] < 0 && mark[v] == 3u) comp[v] = pivot;
    }
}

__global__ void k_color_init(int32_t n, const int32_t* __restrict__ comp, int32_t* color) {
    GSTRIDE_LOOP(v, n) color[v] = comp[v] < 0 ? (int32_t)v : -1;
}

// colour(w) = max colour of active in-neighbours (read as they change)
__global__ void k_color_prop(int32_t n, const int32_t* __restrict__ irp, const int32_t* __restrict__ icol,
                             const int32_t* __restrict__ comp, int32_t* color, int32_t* changed) {
    GSTRIDE_LOOP(w, n) {
        if (comp[w] >= 0) continue;
        int32_t c = ld_rel(&color[w]), c0 = c;
        for (int32_t e = irp[w]; e < irp[w + 1]; ++e) {
            int32_t u = icol[e];
            if (comp[u] >= 0) continue;
            int32_t cu = ld_rel(&color[u]);
            if (cu > c) c = cu;
        }
        if (c > c0) {
            atomicMax(&color[w], c);
            *changed = 1;
        }
    }
}

// roots of the colour classes; in-class reach-to-root marking
__global__ void k_color_roots(int32_t n, const int32_t* __restrict__ color, int32_t* comp_next) {
    GSTRIDE_LOOP(v, n) {
        if (color[v] == (int32_t)v) comp_next[v] = (int32_t)v;
    }
}

__global__ void k_color_back(int32_t n, const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                             const int32_t* __restrict__ comp, const int32_t* __restrict__ color,
                             int32_t* comp_next, int32_t* changed) {
    GSTRIDE_LOOP(v, n) {
        if (comp[v] >= 0 || ld_rel(&comp_next[v]) >= 0) continue;
        int32_t c = color[v];
        for (int32_t e = rp[v]; e < rp[v + 1]; ++e) {
            int32_t w = col[e];
            if (comp[w] >= 0 || color[w] != c) continue;
            if (ld_rel(&comp_next[w]) == c) {
                __hip_atomic_store(&comp_next[v], c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                *changed = 1;
                break;
            }
        }
    }
}

__global__ void k_color_commit(int32_t n, int32_t* comp, const int32_t* __restrict__ comp_next, int32_t* left) {
    GSTRIDE_LOOP(v, n) {
        if (comp[v] >= 0) continue;
        if (comp_next[v] >= 0) comp[v] = comp_next[v];
        else atomicAdd(left, 1);
    }
}

// dense component ids: is_root scan
__global__ void k_is_root(int32_t n, const int32_t* __restrict__ comp, int32_t* __restrict__ flag) {
    GSTRIDE_LOOP(v, n) flag[v] = comp[v] == (int32_t)v ? 1 : 0;
}

// The component of `common` (the pivot's, mostly the giant one; -1: none) is
// counted per workgroup, the others per wave.
__global__ __launch_bounds__(kBlk) void k_cid(int32_t n, const int32_t* __restrict__ comp,
                                              const int32_t* __restrict__ rootpos, int32_t common,
                                              int32_t* __restrict__ cid, uint32_t* __restrict__ wsize) {
    __shared__ uint32_t s_common;
    if (threadIdx.x == 0) s_common = 0;
    __syncthreads();
    const int32_t cc = common >= 0 ? rootpos[common] : -1;
    uint32_t mine = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < n; base += stride) {
        const int64_t v = base + threadIdx.x;
        const bool on = v < n;
        int32_t c = 0;
        if (on) {
            c = rootpos[comp[v]];
            cid[v] = c;
            mine += c == cc;
        }
        wave_count_key(on && c != cc, c, wsize);
    }
    if (mine) atomicAdd(&s_common, mine);
    __syncthreads();
    if (threadIdx.x == 0 && s_common) atomicAdd(&wsize[cc], s_common);
}

// Arcs between components, one arc per thread, one append per tile (positions
// within it are claimed per wave in LDS).
__global__ __launch_bounds__(kArcBlk) void k_dag_arcs(int32_t n, int64_t m, const int32_t* __restrict__ rp,
                                                      const int32_t* __restrict__ col, const int32_t* __restrict__ cid,
                                                      uint64_t* __restrict__ keys, int32_t* cnt) {
    __shared__ ArcRowLds L;
    __shared__ uint32_t s_n, s_base;
    const int32_t e0 = tile_first(blockIdx.x), len = tile_arcs(e0, m);
    block_arc_rows(rp, n, e0, len, L);
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    constexpr int kPer = kArcTile / kArcBlk;
    uint64_t key[kPer];
    uint32_t pos[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const int32_t i = j * kArcBlk + (int32_t)threadIdx.x;
        bool on = false;
        key[j] = 0;
        if (i < len) {
            const int32_t cu = cid[L.row[i]], cw = cid[col[e0 + i]];
            on = cu != cw;
            key[j] = ((uint64_t)(uint32_t)cu << 32) | (uint32_t)cw;
        }
        pos[j] = wave_claim(on, &s_n);
        if (!on) pos[j] = 0xFFFFFFFFu;
    }
    __syncthreads();
    if (threadIdx.x == 0) s_base = s_n ? (uint32_t)atomicAdd(cnt, (int32_t)s_n) : 0u;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        if (pos[j] != 0xFFFFFFFFu) keys[s_base + pos[j]] = key[j];
}

// sorted keys -> per-component distinct successor lists (CSR by source); the
// arcs of a component are consecutive, so a wave takes one atomic per
// component it holds
__global__ void k_dag_count(int32_t na, const uint64_t* __restrict__ keys, uint32_t* __restrict__ dcnt) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < na; base += stride) {
        const int64_t i = base + threadIdx.x;
        const bool on = i < na && (i == 0 || keys[i] != keys[i - 1]);
        wave_count_key(on, on ? (int32_t)(keys[i] >> 32) : 0, dcnt);
    }
}

__global__ void k_dag_fill(int32_t na, const uint64_t* __restrict__ keys, const int32_t* __restrict__ drp,
                           uint32_t* __restrict__ dfill, int32_t* __restrict__ dcol) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < na; base += stride) {
        const int64_t i = base + threadIdx.x;
        const bool on = i < na && (i == 0 || keys[i] != keys[i - 1]);
        const int32_t c = on ? (int32_t)(keys[i] >> 32) : 0;
        const uint32_t p = wave_claim_key(on, c, dfill);
        if (on) dcol[drp[c] + (int32_t)p] = (int32_t)(keys[i] & 0xFFFFFFFFu);
    }
}

// The refinement's inputs (BigScc::c < 0: plain recurrence only).
struct BigScc {
    int32_t c;            // component T
    uint64_t rT;          // |R(T)|
    const int32_t* inRT;  // per component: 1 if reachable from T (T included)
    uint64_t* omega2;     // per component outside R(T): omega' (recurrence outside R(T))
    int32_t* toT;         // per component: 1 if it reaches T (T itself: 0)
};

// Successor values of a component, gathered over some of its arcs.  The sums
// need no cap on the way (nc successors of at most n each stay below 2^62);
// capping the total at n gives the same value as capping every partial sum.
struct DagSum {
    uint64_t amax, osum, osum2;
    uint32_t reaches;
};

__device__ inline bool dag_done(const int32_t* done, int32_t d) {
    return __hip_atomic_load(&done[d], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) != 0;
}

__device__ inline void dag_take(int32_t d, const uint64_t* alpha, const uint64_t* omega, const BigScc& B, DagSum& A) {
    const uint64_t a = __hip_atomic_load(&alpha[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (a > A.amax) A.amax = a;
    A.osum += __hip_atomic_load(&omega[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (B.c >= 0) {
        if (d == B.c || __hip_atomic_load(&B.toT[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) A.reaches = 1;
        if (!B.inRT[d]) A.osum2 += __hip_atomic_load(&B.omega2[d], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// alpha(c), omega(c) from its successors' sums; c becomes final.
__device__ inline void dag_close(int32_t c, const DagSum& A, const uint32_t* wsize, uint64_t* alpha, uint64_t* omega,
                                 int32_t* done, uint64_t ncap, const BigScc& B) {
    const uint64_t w = wsize[c];
    uint64_t a = w + A.amax;
    uint64_t o = min(w + A.osum, ncap);
    if (B.c >= 0) {
        uint64_t o2 = min(w + A.osum2, ncap);
        if (c == B.c) {
            a = o = B.rT;  // exact, from the breadth-first search
            o2 = 0;
        } else if (A.reaches) {
            o = min(o, min(B.rT + o2, ncap));
        }
        __hip_atomic_store(&B.omega2[c], o2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&B.toT[c], A.reaches ? 1 : 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __hip_atomic_store(&alpha[c], a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&omega[c], o, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&done[c], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// One round of the alpha/omega recurrence: every component whose successors
// are all final becomes final.  Three kernels share a round by the length of
// the successor list: one thread (up to kDagLight), one wave (up to
// kDagHeavy), many workgroups (the giant component, whose list alone held
// one thread for the whole round: R-MAT scale 18, 4382 -> 40 us a round).
constexpr int32_t kDagLight = 16;
constexpr int32_t kDagHeavy = 8192;

__global__ void k_dag_classes(int32_t nc, const int32_t* __restrict__ drp, int32_t* mid, int32_t* heavy,
                              uint32_t* cnt) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < nc; base += stride) {
        const int64_t c = base + threadIdx.x;
        const int32_t len = c < nc ? drp[c + 1] - drp[c] : 0;
        const bool hv = len > kDagHeavy, md = len > kDagLight && !hv;
        const uint32_t pm = wave_claim(md, &cnt[0]), ph = wave_claim(hv, &cnt[1]);
        if (md) mid[pm] = (int32_t)c;
        if (hv) heavy[ph] = (int32_t)c;
    }
}

__global__ void k_dag_round(int32_t nc, const int32_t* __restrict__ drp, const int32_t* __restrict__ dcol,
                            const uint32_t* __restrict__ wsize, uint64_t* alpha, uint64_t* omega,
                            int32_t* done, uint64_t ncap, int32_t* left, BigScc B) {
    GSTRIDE_LOOP(c, nc) {
        const int32_t b = drp[c], end = drp[c + 1];
        if (end - b > kDagLight || done[c]) continue;
        DagSum A{0, 0, 0, 0};
        bool ready = true;
        for (int32_t e = b; e < end && ready; ++e) {
            const int32_t d = dcol[e];
            ready = dag_done(done, d);
            if (ready) dag_take(d, alpha, omega, B, A);
        }
        if (!ready) { atomicAdd(left, 1); continue; }
        dag_close((int32_t)c, A, wsize, alpha, omega, done, ncap, B);
    }
}

__device__ inline uint64_t wave_add64(uint64_t x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
    return x;
}

__global__ __launch_bounds__(kBlk) void k_dag_mid(const int32_t* __restrict__ mid, const uint32_t* __restrict__ cnt,
                                                  const int32_t* __restrict__ drp, const int32_t* __restrict__ dcol,
                                                  const uint32_t* __restrict__ wsize, uint64_t* alpha, uint64_t* omega,
                                                  int32_t* done, uint64_t ncap, int32_t* left, BigScc B) {
    const int lane = threadIdx.x & 63;
    const uint32_t waves = gridDim.x * (kBlk / 64), nm = cnt[0];
    for (uint32_t q = blockIdx.x * (kBlk / 64) + (threadIdx.x >> 6); q < nm; q += waves) {
        const int32_t c = mid[q];
        if (done[c]) continue;
        const int32_t end = drp[c + 1];
        DagSum A{0, 0, 0, 0};
        bool ready = true;
        for (int64_t e0 = drp[c]; e0 < end && ready; e0 += 64) {
            const int64_t e = e0 + lane;
            bool ok = true;
            if (e < end) {
                const int32_t d = dcol[e];
                ok = dag_done(done, d);
                if (ok) dag_take(d, alpha, omega, B, A);
            }
            ready = __ballot(!ok) == 0ull;
        }
        if (ready) {
            A.amax = wave_max64(A.amax);
            A.osum = wave_add64(A.osum);
            A.osum2 = wave_add64(A.osum2);
            A.reaches = __ballot(A.reaches != 0) != 0ull;
        }
        if (lane == 0) {
            if (ready) dag_close(c, A, wsize, alpha, omega, done, ncap, B);
            else atomicAdd(left, 1);
        }
    }
}

// heavy components: sums over the grid into acc (4 words each: amax, osum,
// osum2, reaches | not-ready << 32), closed by k_dag_heavy_close, which also
// clears acc for the next round
__global__ __launch_bounds__(kBlk) void k_dag_heavy(const int32_t* __restrict__ heavy,
                                                    const uint32_t* __restrict__ cnt, const int32_t* __restrict__ drp,
                                                    const int32_t* __restrict__ dcol, const uint64_t* alpha,
                                                    const uint64_t* omega, const int32_t* done,
                                                    unsigned long long* acc, BigScc B) {
    const uint32_t nh = cnt[1];
    for (uint32_t q = blockIdx.y; q < nh; q += gridDim.y) {
        const int32_t c = heavy[q];
        if (done[c]) continue;
        const int32_t end = drp[c + 1];
        DagSum A{0, 0, 0, 0};
        bool ready = true;
        for (int64_t e = (int64_t)drp[c] + blockIdx.x * kBlk + threadIdx.x; e < end && ready;
             e += (int64_t)gridDim.x * kBlk) {
            const int32_t d = dcol[e];
            ready = dag_done(done, d);
            if (ready) dag_take(d, alpha, omega, B, A);
        }
        const unsigned long long a = wave_max64(A.amax), o = wave_add64(A.osum), o2 = wave_add64(A.osum2);
        const bool rc = __ballot(A.reaches != 0) != 0ull, nr = __ballot(!ready) != 0ull;
        if ((threadIdx.x & 63) == 0) {
            if (a) atomicMax(&acc[4 * q], a);
            if (o) atomicAdd(&acc[4 * q + 1], o);
            if (o2) atomicAdd(&acc[4 * q + 2], o2);
            if (rc || nr) atomicOr(&acc[4 * q + 3], (rc ? 1ull : 0ull) | (nr ? 1ull << 32 : 0ull));
        }
    }
}

__global__ void k_dag_heavy_close(const int32_t* __restrict__ heavy, const uint32_t* __restrict__ cnt,
                                  const uint32_t* __restrict__ wsize, uint64_t* alpha, uint64_t* omega, int32_t* done,
                                  uint64_t ncap, int32_t* left, unsigned long long* acc, BigScc B) {
    const uint32_t nh = cnt[1];
    for (uint32_t q = blockIdx.x * blockDim.x + threadIdx.x; q < nh; q += gridDim.x * blockDim.x) {
        const int32_t c = heavy[q];
        if (done[c]) continue;
        const DagSum A{acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], (uint32_t)(acc[4 * q + 3] & 1ull)};
        const bool ready = (acc[4 * q + 3] >> 32) == 0;
        acc[4 * q] = acc[4 * q + 1] = acc[4 * q + 2] = acc[4 * q + 3] = 0;
        if (ready) dag_close(c, A, wsize, alpha, omega, done, ncap, B);
        else atomicAdd(left, 1);
    }
}

// The largest component: max over nodes of (w(cid[v]) << 32 | (2^31 - 1 - v)),
// i.e. the largest size, then the smallest node id.
__global__ void k_big_pick(int32_t n, const int32_t* __restrict__ cid, const uint32_t* __restrict__ wsize,
                           unsigned long long* best) {
    unsigned long long mx = 0;
    GSTRIDE_LOOP(v, n) {
        unsigned long long key = ((unsigned long long)wsize[cid[v]] << 32) | (uint32_t)(0x7FFFFFFF - (int32_t)v);
        if (key > mx) mx = key;
    }
    block_extreme64(mx, best);
}

// a level of an unrestricted breadth-first search; mark[] = 1 once reached
struct BfsOp {
    uint32_t* mark;
    __device__ bool operator()(int32_t w, uint32_t) const { return !mark[w] && !atomicOr(&mark[w], 1u); }
};

// inRT[c] = 1 for every component holding a node the search reached
__global__ void k_mark_comps(int32_t n, const uint32_t* __restrict__ mark, const int32_t* __restrict__ cid,
                             int32_t* inRT) {
    GSTRIDE_LOOP(v, n) {
        if (mark[v]) inRT[cid[v]] = 1;
    }
}

__global__ void k_reach_out(int32_t n, const int32_t* __restrict__ cid, const uint64_t* __restrict__ alpha,
                            const uint64_t* __restrict__ omega, uint32_t* __restrict__ x0, uint32_t* __restrict__ x1) {
    GSTRIDE_LOOP(v, n) {
        x0[v] = (uint32_t)alpha[cid[v]];
        x1[v] = (uint32_t)omega[cid[v]];
    }
}

template <class F>
bc_status cub_call(F&& f, DevBuf& tmp, hipStream_t s) {
    size_t bytes = 0;
    BC_HIP(f((void*)nullptr, bytes));
    if (tmp.bytes < bytes) BC_TRY(tmp.alloc_on(bytes, s));
    BC_HIP(f(tmp.p, bytes));
    return BC_OK;
}

bc_status read_i32(const int32_t* d, int32_t* h, hipStream_t s) {
    BC_HIP(hipMemcpyAsync(h, d, sizeof(int32_t), hipMemcpyDeviceToHost, s));
    BC_HIP(hipStreamSynchronize(s));
    return BC_OK;
}

}  // namespace

bc_status directed_reach(bc_graph* g) {
    const int32_t n = g->dg.n;
    const int64_t m = g->dg.m;
    hipStream_t s = g->stream;
    const size_t N = (size_t)(n > 0 ? n : 1);
    DevBuf tmp, icnt, fill, flag;
    // in-CSR
    BC_TRY(galloc(g, g->irp, sizeof(int32_t) * (N + 1), s));
    BC_TRY(galloc(g, g->icol, sizeof(int32_t) * (size_t)(m > 0 ? m : 1), s));
    BC_TRY(icnt.alloc_on(sizeof(int32_t) * N, s));
    BC_TRY(fill.alloc_on(sizeof(int32_t) * N, s));
    BC_TRY(flag.alloc_on(sizeof(int32_t) * 8, s));
    int32_t* fl = flag.as<int32_t>();
    BC_HIP(hipMemsetAsync(icnt.p, 0, sizeof(int32_t) * N, s));
    BC_HIP(hipMemsetAsync(fill.p, 0, sizeof(int32_t) * N, s));
    if (n == 0) {
        BC_HIP(hipMemsetAsync(g->irp.p, 0, sizeof(int32_t), s));
        g->dg.irp = g->irp.as<int32_t>();
        g->dg.icol = g->icol.as<int32_t>();
        BC_HIP(hipStreamSynchronize(s));
        return BC_OK;
    }
    if (m > 0) k_indeg<<<grid_for(m), kArcBlk, 0, s>>>(m, g->dg.col, icnt.as<int32_t>());
    BC_TRY(cub_call([&](void* t, size_t& b) {
        return hipcub::DeviceScan::ExclusiveSum(t, b, icnt.as<int32_t>(), g->irp.as<int32_t>(), n, s);
    }, tmp, s));
    k_close<<<1, 1, 0, s>>>(g->irp.as<int32_t>(), n, icnt.as<int32_t>());
    if (m > 0)
        k_fill_in<<<arc_tiles(m), kArcBlk, 0, s>>>(n, m, g->dg.rp, g->dg.col, g->irp.as<int32_t>(), fill.as<int32_t>(),
                                                   g->icol.as<int32_t>());
    g->dg.irp = g->irp.as<int32_t>();
    g->dg.icol = g->icol.as<int32_t>();
    const int32_t *rp = g->dg.rp, *col = g->dg.col, *irp = g->dg.irp, *icol = g->dg.icol;

    // ---- SCCs
    DevBuf comp, comp_next, color, mark, q0, q1, best, hv, lctr;
    BC_TRY(hv.alloc_on(sizeof(uint32_t) * heavy_words(m), s));
    BC_TRY(lctr.alloc_on(sizeof(uint32_t) * kListCtrWords, s));
    BC_TRY(comp.alloc_on(sizeof(int32_t) * N, s));
    BC_TRY(comp_next.alloc_on(sizeof(int32_t) * N, s));
    BC_TRY(color.alloc_on(sizeof(int32_t) * N, s));
    BC_TRY(mark.alloc_on(sizeof(uint32_t) * N, s));
    BC_TRY(q0.alloc_on(sizeof(int32_t) * N, s));
    BC_TRY(q1.alloc_on(sizeof(int32_t) * N, s));
    BC_TRY(best.alloc_on(sizeof(unsigned long long), s));
    int32_t* cp = comp.as<int32_t>();
    k_fill_i32<<<grid_for(n), kBlk, 0, s>>>(n, cp, -1);
    auto trim = [&](int passes) -> bc_status {
        for (int it = 0; it < passes; ++it) {
            BC_HIP(hipMemsetAsync(fl, 0, sizeof(int32_t), s));
            k_trim<<<grid_for(n), kBlk, 0, s>>>(n, rp, col, irp, icol, cp, fl);
            int32_t ch = 0;
            BC_TRY(read_i32(fl, &ch, s));
            if (!ch) break;
        }
        return BC_OK;
    };
    BC_TRY(trim(4));
    // forward-backward from the pivot of largest in-degree x out-degree
    int32_t common = -1;  // the pivot, which is its component's root
    {
        BC_HIP(hipMemsetAsync(best.p, 0, sizeof(unsigned long long), s));
        k_pivot<<<grid_for(n, kReduceGrid), kBlk, 0, s>>>(n, rp, irp, cp, best.as<unsigned long long>());
        unsigned long long bk = 0;
        BC_HIP(hipMemcpyAsync(&bk, best.p, sizeof(bk), hipMemcpyDeviceToHost, s));
        BC_HIP(hipStreamSynchronize(s));
        if ((bk >> 32) > 0) {
            int32_t pivot = (int32_t)(bk & 0xFFFFFFFFu);
            common = pivot;
            BC_HIP(hipMemsetAsync(mark.p, 0, sizeof(uint32_t) * N, s));
            for (int dir = 0; dir < 2; ++dir) {
                const int32_t* R = dir == 0 ? rp : irp;
                const int32_t* C = dir == 0 ? col : icol;
                uint32_t bit = 1u << dir;
                // seed: the pivot itself
                uint32_t pbits = 0;
                BC_HIP(hipMemcpyAsync(&pbits, mark.as<uint32_t>() + pivot, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
                BC_HIP(hipStreamSynchronize(s));
                pbits |= bit;
                BC_HIP(hipMemcpyAsync(mark.as<uint32_t>() + pivot, &pbits, sizeof(uint32_t), hipMemcpyHostToDevice, s));
                BC_HIP(hipMemcpyAsync(q0.p, &pivot, sizeof(int32_t), hipMemcpyHostToDevice, s));
                uint64_t reached = 0;
                BC_TRY(list_bfs(R, C, q0.as<int32_t>(), q1.as<int32_t>(),
                                [&](int32_t) { return ReachOp{cp, mark.as<uint32_t>(), bit}; }, lctr.as<uint32_t>(),
                                hv.as<uint32_t>(), &reached, s));
            }
            k_fwbw_assign<<<grid_for(n), kBlk, 0, s>>>(n, mark.as<uint32_t>(), cp, pivot);
        }
    }
    BC_TRY(trim(4));
    // colouring rounds; every round assigns at least one node
    int32_t prev_left = n + 1;
    for (int round = 0;; ++round) {
        k_color_init<<<grid_for(n), kBlk, 0, s>>>(n, cp, color.as<int32_t>());
        for (;;) {
            BC_HIP(hipMemsetAsync(fl, 0, sizeof(int32_t), s));
            k_color_prop<<<grid_for(n), kBlk, 0, s>>>(n, irp, icol, cp, color.as<int32_t>(), fl);
            int32_t ch = 0;
            BC_TRY(read_i32(fl, &ch, s));
            if (!ch) break;
        }
        k_fill_i32<<<grid_for(n), kBlk, 0, s>>>(n, comp_next.as<int32_t>(), -1);
        k_color_roots<<<grid_for(n), kBlk, 0, s>>>(n, color.as<int32_t>(), comp_next.as<int32_t>());
        for (;;) {
            BC_HIP(hipMemsetAsync(fl, 0, sizeof(int32_t), s));
            k_color_back<<<grid_for(n), kBlk, 0, s>>>(n, rp, col, cp, color.as<int32_t>(), comp_next.as<int32_t>(), fl);
            int32_t ch = 0;
            BC_TRY(read_i32(fl, &ch, s));
            if (!ch) break;
        }
        BC_HIP(hipMemsetAsync(fl + 2, 0, sizeof(int32_t), s));
        k_color_commit<<<grid_for(n), kBlk, 0, s>>>(n, cp, comp_next.as<int32_t>(), fl + 2);
        int32_t left = 0;
        BC_TRY(read_i32(fl + 2, &left, s));
        if (left == 0) break;
        if (left >= prev_left) {
            set_error("SCC colouring made no progress (%d nodes left)", left);
            return BC_EDEVICE;
        }
        prev_left = left;
        BC_TRY(trim(2));
    }

    // ---- condensation DAG and the alpha/omega recurrence
    DevBuf rootpos, cid, wsize, keys, keys2, dcnt, drp, dfill, dcol, alpha, omega, done;
    BC_TRY(rootpos.alloc_on(sizeof(int32_t) * (N + 1), s));
    BC_TRY(cid.alloc_on(sizeof(int32_t) * N, s));
    k_is_root<<<grid_for(n), kBlk, 0, s>>>(n, cp, color.as<int32_t>());
    BC_TRY(cub_call([&](void* t, size_t& b) {
        return hipcub::DeviceScan::ExclusiveSum(t, b, color.as<int32_t>(), rootpos.as<int32_t>(), n, s);
    }, tmp, s));
    k_close<<<1, 1, 0, s>>>(rootpos.as<int32_t>(), n, color.as<int32_t>());
    int32_t nc = 0;
    BC_TRY(read_i32(rootpos.as<int32_t>() + n, &nc, s));
    const size_t NC = (size_t)(nc > 0 ? nc : 1);
    BC_TRY(wsize.alloc_on(sizeof(uint32_t) * NC, s));
    BC_HIP(hipMemsetAsync(wsize.p, 0, sizeof(uint32_t) * NC, s));
    k_cid<<<grid_for(n, 4 * kReduceGrid), kBlk, 0, s>>>(n, cp, rootpos.as<int32_t>(), common, cid.as<int32_t>(), wsize.as<uint32_t>());
    BC_TRY(keys.alloc_on(sizeof(uint64_t) * (size_t)(m > 0 ? m : 1), s));
    BC_TRY(keys2.alloc_on(sizeof(uint64_t) * (size_t)(m > 0 ? m : 1), s));
    BC_HIP(hipMemsetAsync(fl + 3, 0, sizeof(int32_t), s));
    if (m > 0)
        k_dag_arcs<<<arc_tiles(m), kArcBlk, 0, s>>>(n, m, rp, col, cid.as<int32_t>(), keys.as<uint64_t>(), fl + 3);
    int32_t na = 0;
    BC_TRY(read_i32(fl + 3, &na, s));
    if (na > 0) {
        BC_TRY(cub_call([&](void* t, size_t& b) {
            return hipcub::DeviceRadixSort::SortKeys(t, b, keys.as<uint64_t>(), keys2.as<uint64_t>(), na, 0, 64, s);
        }, tmp, s));
    }
    BC_TRY(dcnt.alloc_on(sizeof(int32_t) * NC, s));
    BC_TRY(drp.alloc_on(sizeof(int32_t) * (NC + 1), s));
    BC_TRY(dfill.alloc_on(sizeof(int32_t) * NC, s));
    BC_TRY(dcol.alloc_on(sizeof(int32_t) * (size_t)(na > 0 ? na : 1), s));
    BC_HIP(hipMemsetAsync(dcnt.p, 0, sizeof(int32_t) * NC, s));
    BC_HIP(hipMemsetAsync(dfill.p, 0, sizeof(int32_t) * NC, s));
    if (na > 0) k_dag_count<<<grid_for(na), kBlk, 0, s>>>(na, keys2.as<uint64_t>(), dcnt.as<uint32_t>());
    BC_TRY(cub_call([&](void* t, size_t& b) {
        return hipcub::DeviceScan::ExclusiveSum(t, b, dcnt.as<int32_t>(), drp.as<int32_t>(), nc, s);
    }, tmp, s));
    k_close<<<1, 1, 0, s>>>(drp.as<int32_t>(), nc, dcnt.as<int32_t>());
    if (na > 0)
        k_dag_fill<<<grid_for(na), kBlk, 0, s>>>(na, keys2.as<uint64_t>(), drp.as<int32_t>(), dfill.as<uint32_t>(),
                                                 dcol.as<int32_t>());
    BC_TRY(alpha.alloc_on(sizeof(uint64_t) * NC, s));
    BC_TRY(omega.alloc_on(sizeof(uint64_t) * NC, s));
    BC_TRY(done.alloc_on(sizeof(int32_t) * NC, s));
    BC_HIP(hipMemsetAsync(done.p, 0, sizeof(int32_t) * NC, s));
    // largest-SCC refinement: T, its exact reach, the components in R(T)
    BigScc big{-1, 0, nullptr, nullptr, nullptr};
    DevBuf inRT, omega2, toT;
    if (g->big_scc && nc > 0) {
        BC_HIP(hipMemsetAsync(best.p, 0, sizeof(unsigned long long), s));
        k_big_pick<<<grid_for(n, kReduceGrid), kBlk, 0, s>>>(n, cid.as<int32_t>(), wsize.as<uint32_t>(),
                                                best.as<unsigned long long>());
        unsigned long long bk = 0;
        BC_HIP(hipMemcpyAsync(&bk, best.p, sizeof(bk), hipMemcpyDeviceToHost, s));
        BC_HIP(hipStreamSynchronize(s));
        const int32_t root = 0x7FFFFFFF - (int32_t)(uint32_t)(bk & 0xFFFFFFFFu);
        if (root < 0 || root >= n) {
            set_error("internal: largest SCC root %d out of range", root);
            return BC_EDEVICE;
        }
        uint32_t* mk = mark.as<uint32_t>();
        BC_HIP(hipMemsetAsync(mk, 0, sizeof(uint32_t) * N, s));
        const uint32_t one = 1;
        BC_HIP(hipMemcpyAsync(mk + root, &one, sizeof(uint32_t), hipMemcpyHostToDevice, s));
        BC_HIP(hipMemcpyAsync(q0.p, &root, sizeof(int32_t), hipMemcpyHostToDevice, s));
        uint64_t reached = 0;
        BC_TRY(list_bfs(rp, col, q0.as<int32_t>(), q1.as<int32_t>(), [&](int32_t) { return BfsOp{mk}; },
                        lctr.as<uint32_t>(), hv.as<uint32_t>(), &reached, s));
        int32_t c_big = 0;
        BC_TRY(read_i32(cid.as<int32_t>() + root, &c_big, s));
        BC_TRY(inRT.alloc_on(sizeof(int32_t) * NC, s));
        BC_TRY(omega2.alloc_on(sizeof(uint64_t) * NC, s));
        BC_TRY(toT.alloc_on(sizeof(int32_t) * NC, s));
        BC_HIP(hipMemsetAsync(inRT.p, 0, sizeof(int32_t) * NC, s));
        BC_HIP(hipMemsetAsync(toT.p, 0, sizeof(int32_t) * NC, s));
        k_mark_comps<<<grid_for(n), kBlk, 0, s>>>(n, mk, cid.as<int32_t>(), inRT.as<int32_t>());
        big = BigScc{c_big, reached, inRT.as<int32_t>(), omega2.as<uint64_t>(), toT.as<int32_t>()};
    }
    DevBuf mid, heavy, acc;
    const size_t nh_max = heavy_words(na);  // the same bound: a heavy list is longer than kDagHeavy
    static_assert(kDagHeavy >= (int32_t)kListHeavy, "heavy_words bounds the heavy components");
    BC_TRY(mid.alloc_on(sizeof(int32_t) * ((size_t)na / kDagLight + 1), s));
    BC_TRY(heavy.alloc_on(sizeof(int32_t) * nh_max, s));
    BC_TRY(acc.alloc_on(4 * sizeof(uint64_t) * nh_max, s));
    uint32_t* cls = reinterpret_cast<uint32_t*>(fl + 6);  // mid components, heavy components
    BC_HIP(hipMemsetAsync(cls, 0, 2 * sizeof(uint32_t), s));
    BC_HIP(hipMemsetAsync(acc.p, 0, 4 * sizeof(uint64_t) * nh_max, s));
    k_dag_classes<<<grid_for(nc), kBlk, 0, s>>>(nc, drp.as<int32_t>(), mid.as<int32_t>(), heavy.as<int32_t>(), cls);
    for (int32_t prev = nc + 1;;) {
        BC_HIP(hipMemsetAsync(fl, 0, sizeof(int32_t), s));
        k_dag_round<<<grid_for(nc), kBlk, 0, s>>>(nc, drp.as<int32_t>(), dcol.as<int32_t>(), wsize.as<uint32_t>(),
                                                  alpha.as<uint64_t>(), omega.as<uint64_t>(), done.as<int32_t>(),
                                                  (uint64_t)n, fl, big);
        k_dag_mid<<<1024, kBlk, 0, s>>>(mid.as<int32_t>(), cls, drp.as<int32_t>(), dcol.as<int32_t>(),
                                        wsize.as<uint32_t>(), alpha.as<uint64_t>(), omega.as<uint64_t>(),
                                        done.as<int32_t>(), (uint64_t)n, fl, big);
        k_dag_heavy<<<dim3(64, 4), kBlk, 0, s>>>(heavy.as<int32_t>(), cls, drp.as<int32_t>(), dcol.as<int32_t>(),
                                                 alpha.as<uint64_t>(), omega.as<uint64_t>(), done.as<int32_t>(),
                                                 acc.as<unsigned long long>(), big);
        k_dag_heavy_close<<<1, kBlk, 0, s>>>(heavy.as<int32_t>(), cls, wsize.as<uint32_t>(), alpha.as<uint64_t>(),
                                             omega.as<uint64_t>(), done.as<int32_t>(), (uint64_t)n, fl,
                                             acc.as<unsigned long long>(), big);
        int32_t left = 0;
        BC_TRY(read_i32(fl, &left, s));
        if (left == 0) break;
        if (left >= prev) {
            set_error("condensation DAG has a cycle (%d components unresolved)", left);
            return BC_EDEVICE;
        }
        prev = left;
    }
    k_reach_out<<<grid_for(n), kBlk, 0, s>>>(n, cid.as<int32_t>(), alpha.as<uint64_t>(), omega.as<uint64_t>(),
                                             g->x0.as<uint32_t>(), g->x1.as<uint32_t>());
    BC_HIP(hipStreamSynchronize(s));
    return BC_OK;
}

}  // namespace bc
