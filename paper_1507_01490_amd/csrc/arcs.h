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

namespace bc {

constexpr int kArcBlk = 256;       // threads per workgroup of the arc kernels
constexpr int kArcTile = 2048;     // consecutive arcs per workgroup: 8 per thread

// The row of arc e: the last r in [0, n) with rp[r] <= e, which is not empty
// (0 <= e < rp[n]).  One wave, 64 probes a step: four steps for 10^6 rows in
// place of the twenty dependent loads of a binary search.
__device__ inline int32_t wave_row_of(const int32_t* __restrict__ rp, int32_t n, int32_t e) {
    const int32_t lane = (int32_t)__lane_id();
    int32_t lo = 0, hi = n;  // rp[lo] <= e, the answer lies in [lo, hi)
    while (hi - lo > 1) {
        const int32_t step = (hi - lo + 63) / 64;
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

// row[i] = row of arc e0 + i, e0 <= e0 + i < e1 (at most kArcTile arcs, at
// least one).  Every non-empty row that starts in the tile marks its first
// arc; a running maximum spreads the marks.  Whole workgroup of kArcBlk.
__device__ inline void block_arc_rows(const int32_t* __restrict__ rp, int32_t n, int32_t e0, int32_t e1,
                                      ArcRowLds& L) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int kPer = kArcTile / kArcBlk;
    if (wave == 0) {
        const int32_t r = wave_row_of(rp, n, e0);
        if (lane == 0) L.r0 = r;
    } else if (wave == 1) {
        const int32_t r = wave_row_of(rp, n, e1 - 1);
        if (lane == 0) L.r1 = r;
    }
    for (int i = tid; i < kArcTile; i += kArcBlk) L.row[i] = -1;
    __syncthreads();
    const int32_t r1 = L.r1;
    for (int32_t r = L.r0 + tid; r <= r1; r += kArcBlk) {
        const int32_t b = rp[r];
        if (b < rp[r + 1]) L.row[max(b, e0) - e0] = r;
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

inline unsigned arc_tiles(int64_t m) { return (unsigned)((m + kArcTile - 1) / kArcTile); }

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

// ---- breadth-first level over a frontier list

constexpr int kListBuf = 1024;      // reached nodes staged in LDS before one global append
constexpr uint32_t kListHeavy = 8192;  // entries with more arcs are spread over many workgroups
constexpr uint32_t kListGrid = 1024;   // workgroups a long list is spread over

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

// Every out-arc of the frontier entries F[0, flen), `per` (at most kArcBlk)
// entries a workgroup: op(target, entry index) says whether the target joins
// the list N.  Entries above kListHeavy arcs go to the heavy list instead.
template <class Op>
__global__ __launch_bounds__(kArcBlk) void k_list_arcs(const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                                                       const int32_t* F, uint32_t flen, uint32_t per, Op op,
                                                       int32_t* N, uint32_t* ncount, uint32_t* heavy, uint32_t* hcount) {
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

// One breadth-first level: ctr[0] (list length) and ctr[1] (heavy entries)
// are zero on entry; heavy holds heavy_words(m) words.  `per` spreads the list over
// kListGrid workgroups, so that a short list of long rows fills the chip too.
template <class Op>
inline void list_arcs(const int32_t* rp, const int32_t* col, const int32_t* F, uint32_t flen, Op op, int32_t* N,
                      uint32_t* ctr, uint32_t* heavy, hipStream_t s) {
    uint32_t per = (flen + kListGrid - 1) / kListGrid;
    if (per > (uint32_t)kArcBlk) per = kArcBlk;
    if (per < 1) per = 1;
    uint32_t blocks = (flen + per - 1) / per;
    if (blocks > 8192) blocks = 8192;
    if (blocks < 1) blocks = 1;
    k_list_arcs<Op><<<blocks, kArcBlk, 0, s>>>(rp, col, F, flen, per, op, N, ctr, heavy, ctr + 1);
    k_list_heavy<Op><<<dim3(64, 16), kArcBlk, 0, s>>>(rp, col, F, op, N, ctr, heavy, ctr + 1);
}

}  // namespace bc
