// Arc-parallel building blocks of the pre-processing kernels.
//
// Degrees are skewed (an R-MAT scale 18 row holds up to ~10^4 arcs, the
// median row a handful), so a kernel that gives each row to one thread lasts
// as long as its longest row.  Here the arcs are dealt out instead:
//   block_arc_rows   a workgroup takes kArcTile consecutive arcs of a CSR and
//                    recovers the row of each in LDS
//   list_arcs        a workgroup takes a run of frontier entries and walks
//                    their arcs in one flat, coalesced sequence
// and counters or lists that every thread would hit are aggregated per wave or
// per workgroup before the global atomic.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <utility>

#include "bc_internal.h"

namespace bc {

constexpr int kArcBlk = 256;       // threads per workgroup of the arc kernels

// The row of arc e: the last r in [0, n) with rp[r] <= e, which is not empty
// (0 <= e < rp[n]).  One wave, 64 probes a step: four steps for 10^6 rows in
// place of the twenty dependent loads of a binary search.
__device__ inline int32_t wave_row_of(const int32_t* __restrict__ rp, int32_t n, int32_t e) {
    const int32_t lane = (int32_t)__lane_id();
    int32_t lo = 0, hi = n;  // rp[lo] <= e, the answer lies in [lo, hi)
    while (hi - lo > 1) {
        const int32_t step = probe_step(lo, hi);
        const int64_t p = (int64_t)lo + (int64_t)(lane + 1) * step;
        const bool le = p < hi && rp[p] <= e;
        const int32_t c = __popcll(__ballot(le));  // rp is non-decreasing: a prefix of the lanes
        lo += c * step;
        hi = (int32_t)min((int64_t)hi, (int64_t)lo + step);
    }
    return lo;
}

struct ArcRowLds {
    int32_t row[kArcTile];
    int32_t wmax[kArcBlk / 64];
    int32_t r0, r1;
};

// row[i] = row of arc e0 + i, i < len (at most kArcTile arcs, at least one).
// Every non-empty row that starts in the tile marks its first
// arc; a running maximum spreads the marks.  Whole workgroup of kArcBlk.
__device__ inline void block_arc_rows(const int32_t* __restrict__ rp, int32_t n, int32_t e0, int32_t len,
                                      ArcRowLds& L) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int kPer = kArcTile / kArcBlk;
    if (wave == 0) {
        const int32_t r = wave_row_of(rp, n, e0);
        if (lane == 0) L.r0 = r;
    } else if (wave == 1) {
        const int32_t r = wave_row_of(rp, n, e0 + (len - 1));
        if (lane == 0) L.r1 = r;
    }
    for (int i = tid; i < kArcTile; i += kArcBlk) L.row[i] = -1;
    __syncthreads();
    const int64_t r1 = L.r1;
    for (int64_t r = (int64_t)L.r0 + tid; r <= r1; r += kArcBlk) {
        const int32_t b = rp[r];
        if (b < rp[r + 1]) L.row[max(b, e0) - e0] = (int32_t)r;
    }
    __syncthreads();
    int32_t v[kPer], mx = -1;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        mx = max(mx, L.row[tid * kPer + j]);
        v[j] = mx;
    }
    int32_t x = mx;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(x, o);
        if (lane >= o) x = max(x, y);
    }
    if (lane == 63) L.wmax[wave] = x;
    int32_t before = __shfl_up(x, 1);
    if (lane == 0) before = -1;
    __syncthreads();
    for (int k = 0; k < wave; ++k) before = max(before, L.wmax[k]);
#pragma unroll
    for (int j = 0; j < kPer; ++j) L.row[tid * kPer + j] = max(before, v[j]);
    __syncthreads();
}

inline unsigned arc_tiles(int64_t m) { return (unsigned)tile_count(m); }

// ctr[key] += 1 for every lane with `on`, one atomic per distinct key of the
// wave (nodes of one component come in long runs).  Converged wave.
__device__ inline void wave_count_key(bool on, int32_t key, uint32_t* ctr) {
    unsigned long long left = __ballot(on);
    while (left) {
        const int lead = __ffsll((long long)left) - 1;
        const int32_t k = __shfl(key, lead);
        const unsigned long long same = __ballot(on && key == k) & left;
        if ((int)__lane_id() == lead) atomicAdd(&ctr[k], (uint32_t)__popcll(same));
        left &= ~same;
    }
}

// The same counters taken as list lengths: each lane with `on` gets its
// position in the list of its key.
__device__ inline uint32_t wave_claim_key(bool on, int32_t key, uint32_t* ctr) {
    const int lane = (int)__lane_id();
    unsigned long long left = __ballot(on);
    uint32_t pos = 0;
    while (left) {
        const int lead = __ffsll((long long)left) - 1;
        const int32_t k = __shfl(key, lead);
        const unsigned long long same = __ballot(on && key == k) & left;
        uint32_t base = 0;
        if (lane == lead) base = atomicAdd(&ctr[k], (uint32_t)__popcll(same));
        base = __shfl(base, lead);
        if ((same >> lane) & 1ull) pos = base + (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
        left &= ~same;
    }
    return pos;
}

// Position of each lane with `on` in a global list whose length is *ctr: one
// atomic per wave.  Converged wave; lanes without `on` get no position.
__device__ inline uint32_t wave_claim(bool on, uint32_t* ctr) {
    const unsigned long long bal = __ballot(on);
    if (bal == 0) return 0;
    const int lane = (int)__lane_id(), lead = __ffsll((long long)bal) - 1;
    uint32_t base = 0;
    if (lane == lead) base = atomicAdd(ctr, (uint32_t)__popcll(bal));
    return __shfl(base, lead) + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
}

// Maximum (minimum) of a 64-bit value over the wave, in every lane.
__device__ inline unsigned long long wave_max64(unsigned long long x) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const unsigned long long y = __shfl_xor(x, o);
        if (y > x) x = y;
    }
    return x;
}
__device__ inline unsigned long long wave_min64(unsigned long long x) { return ~wave_max64(~x); }

// *out = max(*out, x over the workgroup): one atomic per workgroup.  Atomics
// on one address take about 12 ns each here, so the kernels that end in one
// also keep to kReduceGrid workgroups (k_loc_far over 300,000 nodes: 57 us
// with one atomic per wave of a full grid, 6 us).
constexpr int64_t kReduceGrid = 256;
template <bool kMin = false>
__device__ inline void block_extreme64(unsigned long long x, unsigned long long* out) {
    __shared__ unsigned long long part[kArcBlk / 64];
    x = kMin ? wave_min64(x) : wave_max64(x);
    __syncthreads();  // part may still be read by an earlier call
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 1; k < kArcBlk / 64; ++k) x = kMin ? min(x, part[k]) : max(x, part[k]);
    if (kMin) {
        if (x != ~0ull) atomicMin(out, x);
    } else if (x) {
        atomicMax(out, x);
    }
}

// ---- breadth-first level over a frontier list

constexpr int kListBuf = 1024;      // reached nodes staged in LDS before one global append
constexpr uint32_t kListHeavy = 8192;  // entries with more arcs are spread over many workgroups
constexpr uint32_t kListGrid = 1024;   // workgroups a list is spread over
constexpr int kListAhead = 8;          // levels launched before the host looks at their lengths
constexpr size_t kListCtrWords = 2 * (kListAhead + 1);

struct ListLds {
    int32_t beg[kArcBlk];
    uint32_t off[kArcBlk];
    uint32_t scan[kArcBlk / 64 + 1];
    int32_t buf[kListBuf];
    uint32_t fill, base;
};

// Append w (lanes with `on`) to the LDS stage; the caller keeps room.
__device__ inline void stage_node(bool on, int32_t w, ListLds& L) {
    const uint32_t p = wave_claim(on, &L.fill);
    if (on) L.buf[p] = w;
}
// Write the stage out behind one global atomic.  Whole workgroup, after a
// barrier that follows the last stage_node.
__device__ inline void stage_flush(ListLds& L, int32_t* N, uint32_t* ncount) {
    const uint32_t f = L.fill;
    if (f == 0) return;  // the same in every thread
    if (threadIdx.x == 0) L.base = atomicAdd(ncount, f);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < f; i += kArcBlk) N[L.base + i] = L.buf[i];
    __syncthreads();
    if (threadIdx.x == 0) L.fill = 0;
    __syncthreads();
}

// Every out-arc of the frontier entries F[0, *flen_p): op(target, entry index)
// says whether the target joins the list N.  A workgroup takes `per` (at most
// kArcBlk) entries at a time, so that a short list of long rows fills the chip
// too.  Entries above kListHeavy arcs go to the heavy list instead.
template <class Op>
__global__ __launch_bounds__(kArcBlk) void k_list_arcs(const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                       const int32_t* F, const uint32_t* flen_p, Op op, int32_t* N,
                                                       uint32_t* ncount, uint32_t* heavy, uint32_t* hcount) {
    const uint32_t flen = *flen_p;
    if (flen == 0) return;
    const uint32_t per = min((flen + gridDim.x - 1) / gridDim.x, (uint32_t)kArcBlk);
    __shared__ ListLds L;
    const uint32_t tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    if (tid == 0) L.fill = 0;
    for (uint64_t e0 = (uint64_t)blockIdx.x * per; e0 < flen; e0 += (uint64_t)gridDim.x * per) {
        const uint64_t e = e0 + tid;
        uint32_t deg = 0;
        int32_t beg = 0;
        if (tid < per && e < flen) {
            const int32_t u = F[e];
            beg = rp[u];
            deg = (uint32_t)(rp[u + 1] - beg);
            if (deg > kListHeavy) {
                heavy[atomicAdd(hcount, 1u)] = (uint32_t)e;
                deg = 0;
            }
        }
        uint32_t x = deg;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(x, o);
            if (lane >= o) x += y;
        }
        if (lane == 63) L.scan[wave] = x;
        __syncthreads();
        uint32_t before = 0, total = 0;
#pragma unroll
        for (int k = 0; k < kArcBlk / 64; ++k) {
            if (k < wave) before += L.scan[k];
            total += L.scan[k];
        }
        L.beg[tid] = beg;
        L.off[tid] = before + x - deg;
        __syncthreads();
        for (uint32_t a0 = 0; a0 < total; a0 += kArcBlk) {
            const uint32_t a = a0 + tid;
            bool on = false;
            int32_t w = 0;
            if (a < total) {
                uint32_t lo = 0, hi = kArcBlk;  // owner: the last i with off[i] <= a
                while (lo < hi) {
                    const uint32_t mid = (lo + hi) >> 1;
                    if (L.off[mid] <= a) lo = mid + 1; else hi = mid;
                }
                w = col[L.beg[lo - 1] + (int32_t)(a - L.off[lo - 1])];
                on = op(w, (uint32_t)(e0 + lo - 1));
            }
            stage_node(on, w, L);
            __syncthreads();
            if (L.fill + kArcBlk > kListBuf) stage_flush(L, N, ncount);
            else __syncthreads();  // every thread has read fill before it grows again
        }
    }
    __syncthreads();
    stage_flush(L, N, ncount);
}

// The heavy entries: grid.y of them at a time, each walked by grid.x workgroups.
template <class Op>
__global__ __launch_bounds__(kArcBlk) void k_list_heavy(const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                        const int32_t* F, Op op, int32_t* N, uint32_t* ncount,
                                                        const uint32_t* heavy, const uint32_t* hcount) {
    __shared__ ListLds L;
    const uint32_t nh = *hcount;
    if (nh == 0) return;
    if (threadIdx.x == 0) L.fill = 0;
    __syncthreads();
    for (uint32_t h = blockIdx.y; h < nh; h += gridDim.y) {
        const uint32_t i = heavy[h];
        const int32_t u = F[i], b = rp[u], end = rp[u + 1];
        for (int64_t e0 = (int64_t)b + (int64_t)blockIdx.x * kArcBlk; e0 < end; e0 += (int64_t)gridDim.x * kArcBlk) {
            const int64_t e = e0 + threadIdx.x;
            bool on = false;
            int32_t w = 0;
            if (e < end) {
                w = col[e];
                on = op(w, i);
            }
            stage_node(on, w, L);
            __syncthreads();
            if (L.fill + kArcBlk > kListBuf) stage_flush(L, N, ncount);
            else __syncthreads();
        }
    }
    __syncthreads();
    stage_flush(L, N, ncount);
}

// Entries of one list with more than kListHeavy arcs (rows are distinct).
inline size_t heavy_words(int64_t m) { return (size_t)(m / kListHeavy) + 1; }

// One breadth-first level over F[0, *flen): the reached nodes go to N, their
// count to ctr[0] (ctr[0] and ctr[1] are zero on entry; heavy holds
// heavy_words(m) words).
template <class Op>
inline void list_arcs(const int32_t* rp, const int32_t* col, const int32_t* F, const uint32_t* flen, Op op, int32_t* N,
                      uint32_t* ctr, uint32_t* heavy, hipStream_t s) {
    k_list_arcs<Op><<<kListGrid, kArcBlk, 0, s>>>(rp, col, F, flen, op, N, ctr, heavy, ctr + 1);
    k_list_heavy<Op><<<dim3(64, 16), kArcBlk, 0, s>>>(rp, col, F, op, N, ctr, heavy, ctr + 1);
}

// Breadth-first search from q0[0], all levels: make_op(d) visits the arcs out
// of level d.  kListAhead levels are launched at a time, each reading its
// length on the device; a level past the end costs two empty launches, a
// round trip to the host per level cost more than most levels.  ctr holds
// kListCtrWords words; *reached counts the nodes, the source among them.
template <class MakeOp>
inline bc_status list_bfs(const int32_t* rp, const int32_t* col, int32_t* q0, int32_t* q1, MakeOp make_op,
                          uint32_t* ctr, uint32_t* heavy, uint64_t* reached, hipStream_t s) {
    uint32_t len[kListCtrWords] = {1};
    BC_HIP(hipMemcpyAsync(ctr, len, sizeof(uint32_t), hipMemcpyHostToDevice, s));
    *reached = 1;
    for (int32_t d = 0;;) {
        BC_HIP(hipMemsetAsync(ctr + 2, 0, sizeof(uint32_t) * (kListCtrWords - 2), s));
        for (int l = 0; l < kListAhead; ++l, ++d) {
            list_arcs(rp, col, q0, ctr + 2 * l, make_op(d), q1, ctr + 2 * (l + 1), heavy, s);
            std::swap(q0, q1);
        }
        BC_HIP(hipMemcpyAsync(len, ctr, sizeof(len), hipMemcpyDeviceToHost, s));
        BC_HIP(hipStreamSynchronize(s));
        for (int l = 1; l <= kListAhead; ++l) *reached += len[2 * l];
        if (len[2 * kListAhead] == 0) return BC_OK;
        BC_HIP(hipMemcpyAsync(ctr, ctr + 2 * kListAhead, sizeof(uint32_t), hipMemcpyDeviceToDevice, s));
    }
}

}  // namespace bc
