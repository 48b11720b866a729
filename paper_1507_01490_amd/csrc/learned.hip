// Learned source order.  Algorithm 1 returns the same top-k for every
// processing order; the order only decides how soon the k-th best value is
// known (Section 2.1).  The paper uses decreasing degree.  Here a small
// perceptron scores every node from three features and the sources are
// processed by decreasing score (ties by decreasing degree, then id):
//
//   x0 = log(1 + outdeg(v))
//   x1 = log(1 + sum of outdeg(u) over the out-arcs v -> u)
//   x2 = log(1 + core(v))   core(v): largest c such that v lies in a subgraph
//                           where every node keeps >= c out-neighbours
//
// each column standardised over the nodes ((x - mean) / population std; a
// column whose integers are all equal is 0).  core(v) is the fixed point of
// the in-place h-index iteration h(v) <- max{c : at least c out-neighbours u
// have h(u) >= c}, started from the out-degree: every estimate stays >= the
// core number, and a sweep that changes nothing leaves a fixed point, which
// is <= the core number.
//
// Perceptron 3 -> 64 -> 64 -> 1 with ReLU, fp32, parameters in one vector
//   W1[64][3] @0, b1 @192, W2[64][64] @256, b2 @4352, w3 @4416, b3 @4480.
// The trainer uses the loss sum w (y - t)^2 / sum w, its gradient and Adam.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>

#include "arcs.h"
#include "bc_internal.h"

namespace bc {

namespace {

constexpr int kBlk = 256;
constexpr int kH = 64;
constexpr int kOffW1 = 0, kOffB1 = 192, kOffW2 = 256, kOffB2 = 4352, kOffW3 = 4416, kOffB3 = 4480;
constexpr int kNP = BC_MLP_PARAMS;
static_assert(kOffB3 + 1 == kNP, "parameter layout");
constexpr int kTile = 128;        // samples per workgroup in the gradient kernel
constexpr int kRedBlocks = 512;   // partial sums of the feature statistics

inline unsigned grid_for(int64_t work, int64_t cap = 8192) {
    int64_t b = (work + kBlk - 1) / kBlk;
    if (b < 1) b = 1;
    if (b > cap) b = cap;
    return (unsigned)b;
}

__device__ inline uint32_t ld_relaxed(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// --------------------------------------------------------------- features

// Nodes of degree >= kHeavy take one wave each in the kernels below, the
// others one thread: a thread alone with a row of 255 arcs set the time of a
// sweep (collaboration graph of 300,000 actors: 92 us a sweep at 64 against
// 182 at 256, 288 -> 46 us for the neighbour sums).
constexpr uint32_t kHeavy = 64;

// s2[v] = sum of deg(u) over the out-arcs of v (light nodes); h[v] = deg(v)
// (core start).
__global__ void k_feat_init(int32_t n, const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                            const uint32_t* __restrict__ deg, uint64_t* __restrict__ s2, uint32_t* __restrict__ h) {
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        h[v] = deg[v];
        if (deg[v] >= kHeavy) continue;
        uint64_t s = 0;
        for (int32_t e = rp[v]; e < rp[v + 1]; ++e) s += deg[col[e]];
        s2[v] = s;
    }
}

__global__ void k_feat_heavy(const int32_t* __restrict__ list, const uint32_t* __restrict__ len,
                             const int32_t* __restrict__ rp, const int32_t* __restrict__ col,
                             const uint32_t* __restrict__ deg, uint64_t* __restrict__ s2) {
    const int lane = threadIdx.x & 63;
    const uint32_t nh = *len, waves = gridDim.x * (blockDim.x / 64);
    for (uint32_t q = blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64; q < nh; q += waves) {
        const int32_t v = list[q];
        uint64_t s = 0;
        const int64_t end = rp[v + 1];
        for (int64_t e = (int64_t)rp[v] + lane; e < end; e += 64) s += deg[col[e]];
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
        if (lane == 0) s2[v] = s;
    }
}

__device__ inline uint32_t count_at_least(const int32_t* __restrict__ col, int32_t b, int32_t e, const uint32_t* h,
                                          uint32_t c) {
    uint32_t cnt = 0;
    for (int32_t i = b; i < e; ++i) cnt += ld_relaxed(&h[col[i]]) >= c;
    return cnt;
}

// One in-place sweep of the h-index iteration over the nodes of degree <
// kHeavy (one thread each).  Estimates only decrease and other threads may
// lower them meanwhile; any value read is >= the core number, which keeps
// every update >= the core number.
__global__ void k_hindex(int32_t n, const int32_t* __restrict__ rp, const int32_t* __restrict__ col, uint32_t* h,
                         uint32_t* changed) {
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        uint32_t hv = ld_relaxed(&h[v]);
        if (hv == 0 || (uint32_t)(rp[v + 1] - rp[v]) >= kHeavy) continue;
        int32_t b = rp[v], e = rp[v + 1];
        if (count_at_least(col, b, e, h, hv) >= hv) continue;
        // largest c in [0, hv - 1] with count(c) >= c (c = 0 always holds)
        uint32_t lo = 0, hi = hv - 1;
        while (lo < hi) {
            uint32_t mid = lo + (hi - lo + 1) / 2;
            if (count_at_least(col, b, e, h, mid) >= mid) lo = mid;
            else hi = mid - 1;
        }
        __hip_atomic_store(&h[v], lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *changed = 1u;
    }
}

// Nodes of degree >= kHeavy, one wave each (the lanes split the adjacency).
__global__ void k_heavy_list(int32_t n, const uint32_t* __restrict__ deg, int32_t* __restrict__ list,
                             uint32_t* __restrict__ len) {
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < n; base += stride) {
        const int64_t v = base + threadIdx.x;
        const bool on = v < n && deg[v] >= kHeavy;
        const uint32_t p = wave_claim(on, len);
        if (on) list[p] = (int32_t)v;
    }
}

__device__ inline uint32_t wave_count_at_least(const int32_t* __restrict__ col, int32_t b, int32_t e,
                                               const uint32_t* h, uint32_t c, int lane) {
    uint32_t cnt = 0;
    for (int64_t i = (int64_t)b + lane; i < e; i += 64) cnt += ld_relaxed(&h[col[i]]) >= c;
    for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off, 64);
    return cnt;  // every lane holds the total
}

__global__ void k_hindex_heavy(const int32_t* __restrict__ list, const uint32_t* __restrict__ len,
                               const int32_t* __restrict__ rp, const int32_t* __restrict__ col, uint32_t* h,
                               uint32_t* changed) {
    const int lane = threadIdx.x & 63;
    const uint32_t nh = *len;
    const uint32_t waves = gridDim.x * (blockDim.x / 64);
    for (uint32_t q = blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64; q < nh; q += waves) {
        const int32_t v = list[q];
        const uint32_t hv = ld_relaxed(&h[v]);
        if (hv == 0) continue;
        const int32_t b = rp[v], e = rp[v + 1];
        if (wave_count_at_least(col, b, e, h, hv, lane) >= hv) continue;
        uint32_t lo = 0, hi = hv - 1;
        while (lo < hi) {
            uint32_t mid = lo + (hi - lo + 1) / 2;
            if (wave_count_at_least(col, b, e, h, mid, lane) >= mid) lo = mid;
            else hi = mid - 1;
        }
        if (lane == 0) {
            __hip_atomic_store(&h[v], lo, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *changed = 1u;
        }
    }
}

__device__ inline void raw3(int64_t v, const uint32_t* deg, const uint64_t* s2, const uint32_t* core, double r[3]) {
    r[0] = log1p((double)deg[v]);
    r[1] = log1p((double)s2[v]);
    r[2] = log1p((double)core[v]);
}

// Block sums of the raw features (pass 0) or of their squared deviations
// from the mean (pass 1), one row of 3 doubles per workgroup.
__global__ __launch_bounds__(kBlk) void k_feat_sums(int32_t n, const uint32_t* __restrict__ deg,
                                                    const uint64_t* __restrict__ s2,
                                                    const uint32_t* __restrict__ core, const double* __restrict__ mean,
                                                    double* __restrict__ part) {
    __shared__ double red[3][kBlk];
    double a[3] = {0.0, 0.0, 0.0};
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        double r[3];
        raw3(v, deg, s2, core, r);
        for (int j = 0; j < 3; ++j) {
            double d = mean ? r[j] - mean[j] : r[j];
            a[j] += mean ? d * d : d;
        }
    }
    for (int j = 0; j < 3; ++j) red[j][threadIdx.x] = a[j];
    __syncthreads();
    for (int s = kBlk / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int j = 0; j < 3; ++j) red[j][threadIdx.x] += red[j][threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x < 3) part[blockIdx.x * 3 + threadIdx.x] = red[threadIdx.x][0];
}

// Sum the block rows in a fixed order; out[j] = total / n (mean or variance).
// The rows come through LDS: three threads on dependent global loads took 51 us.
__global__ __launch_bounds__(kBlk) void k_feat_finish(int32_t n, int nparts, const double* __restrict__ part,
                                                      double* __restrict__ out) {
    __shared__ double row[kRedBlocks * 3];
    for (int i = threadIdx.x; i < nparts * 3; i += kBlk) row[i] = part[i];
    __syncthreads();
    const int j = threadIdx.x;
    if (j >= 3) return;
    double s = 0.0;
    for (int b = 0; b < nparts; ++b) s += row[b * 3 + j];
    out[j] = s / (double)n;
}

__global__ void k_feat_write(int32_t n, const uint32_t* __restrict__ deg, const uint64_t* __restrict__ s2,
                             const uint32_t* __restrict__ core, const double* __restrict__ mean,
                             const double* __restrict__ var, const unsigned long long* __restrict__ mm,
                             float* __restrict__ x) {
    bool cst[3] = {mm[0] == mm[1], mm[2] == mm[3], mm[4] == mm[5]};
    double sd[3];
    for (int j = 0; j < 3; ++j) sd[j] = sqrt(var[j]);
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        double r[3];
        raw3(v, deg, s2, core, r);
        for (int j = 0; j < 3; ++j) x[v * 3 + j] = cst[j] ? 0.f : (float)((r[j] - mean[j]) / sd[j]);
    }
}

// integer min and max of the three integer columns (for the constant test)
__global__ void k_feat_minmax(int32_t n, const uint32_t* __restrict__ deg, const uint64_t* __restrict__ s2,
                              const uint32_t* __restrict__ core, unsigned long long* mm) {
    unsigned long long lo[3] = {~0ull, ~0ull, ~0ull}, hi[3] = {0, 0, 0};
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        const unsigned long long x[3] = {deg[v], s2[v], core[v]};
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            lo[j] = min(lo[j], x[j]);
            hi[j] = max(hi[j], x[j]);
        }
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) {
        block_extreme64<true>(lo[j], &mm[2 * j]);
        block_extreme64(hi[j], &mm[2 * j + 1]);
    }
}

__global__ void k_minmax_init(unsigned long long* mm) {
    if (threadIdx.x < 6) mm[threadIdx.x] = (threadIdx.x & 1) ? 0ull : ~0ull;
}

// ------------------------------------------------------------ perceptron

// h1 = relu(W1 x + b1) for one sample
__device__ inline void layer1(const float* P, float x0, float x1, float x2, float h1[kH]) {
#pragma unroll
    for (int i = 0; i < kH; ++i) {
        float a = P[kOffB1 + i];
        a = fmaf(P[kOffW1 + i * 3 + 0], x0, a);
        a = fmaf(P[kOffW1 + i * 3 + 1], x1, a);
        a = fmaf(P[kOffW1 + i * 3 + 2], x2, a);
        h1[i] = fmaxf(a, 0.f);
    }
}

// h2_j = relu(W2[j] . h1 + b2_j)
__device__ inline float unit2(const float* P, const float h1[kH], int j) {
    float a = P[kOffB2 + j];
#pragma unroll
    for (int i = 0; i < kH; ++i) a = fmaf(P[kOffW2 + j * kH + i], h1[i], a);
    return fmaxf(a, 0.f);
}

// Weights are read at wave-uniform addresses straight from the parameter
// vector (scalar loads, no LDS staging); one sample per thread.
__global__ __launch_bounds__(kBlk) void k_mlp_forward(const float* __restrict__ P, const float* __restrict__ x,
                                                      int64_t count, float* __restrict__ y) {
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < count; s += stride) {
        float h1[kH];
        layer1(P, x[s * 3], x[s * 3 + 1], x[s * 3 + 2], h1);
        float out = P[kOffB3];
#pragma unroll 1
        for (int j = 0; j < kH; ++j) out = fmaf(P[kOffW3 + j], unit2(P, h1, j), out);
        y[s] = out;
    }
}

// Loss gradient over one tile of kTile samples per workgroup (four waves of 32
// samples), with the unnormalised output gradient dy = 2 w (y - t); the
// reduction kernel sums the tiles in a fixed order and divides by sum w.
// Partial row per tile: the kNP gradient entries, then sum w r^2 and sum w.
//
// The three 64-wide products (layer 2 forward, its input gradient G1 = G2 W2,
// its weight gradient G2' H1) run on the matrix cores in fp32, 32x32x2 tiles:
// lane l holds A[l % 32][l / 32] and B[l / 32][l % 32], and register r of the
// result is row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.  Layer 1 is
// computed straight in the A layout; only H1 and G2 pass through LDS (rows of
// kH + 2 words: the 64 lanes of an A read then fall on 64 banks).  32,768
// samples are 256 tiles, one per compute unit: bound by the products, 192
// matrix instructions a wave (5 us).  Measured 22 us; one thread per sample
// with the activations in rows of 64 words (all lanes on one bank) took 91.
using v16f = __attribute__((ext_vector_type(16))) float;
constexpr int kRow = kH + 2;

struct GradLds {
    float W2[kH * kRow];
    float W1[3 * kH], B1[kH], B2[kH], W3[kH];
    float X[kTile][3];
    float T[kTile], WS[kTile], DY[kTile], WR2[kTile];
    float H1[kTile * kRow], G2[kTile * kRow];
    float red[kBlk / 64][6][kH];  // per wave: db1, dW1 (3), db2, dw3
};

__device__ inline v16f mfma32(float a, float b, v16f c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

__global__ __launch_bounds__(kBlk) void k_mlp_grad(const float* __restrict__ params, const float* __restrict__ x,
                                                   const float* __restrict__ t, const float* __restrict__ w,
                                                   int64_t rows, const int32_t* __restrict__ idx, int64_t count,
                                                   float* __restrict__ part, uint32_t* __restrict__ bad) {
    __shared__ GradLds L;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sl = lane & 31, h = lane >> 5;
    const int s0 = wave * 32;  // this wave's samples
    const int64_t base = (int64_t)blockIdx.x * kTile;
    for (int i = tid; i < kH * kH; i += kBlk) L.W2[(i / kH) * kRow + i % kH] = params[kOffW2 + i];
    if (tid < 3 * kH) L.W1[tid] = params[kOffW1 + tid];
    if (tid < kH) {
        L.B1[tid] = params[kOffB1 + tid];
        L.B2[tid] = params[kOffB2 + tid];
        L.W3[tid] = params[kOffW3 + tid];
    }
    const float b3 = params[kOffB3];
    if (tid < kTile) {
        const int64_t s = base + tid;
        float x0 = 0.f, x1 = 0.f, x2 = 0.f, ws = 0.f, tv = 0.f;
        int64_t v = s < count ? (idx ? (int64_t)idx[s] : s) : -1;
        if (s < count && (v < 0 || v >= rows)) {
            *bad = 1u;  // the sample is left out (weight 0); the call fails
            v = -1;
        }
        if (v >= 0) {
            x0 = x[v * 3];
            x1 = x[v * 3 + 1];
            x2 = x[v * 3 + 2];
            ws = w ? w[v] : 1.f;
            tv = t[v];
        }
        L.X[tid][0] = x0;
        L.X[tid][1] = x1;
        L.X[tid][2] = x2;
        L.T[tid] = tv;
        L.WS[tid] = ws;  // 0 outside the sample range
    }
    __syncthreads();
    // layer 1: lane (sl, h) takes the units of parity h of its sample
    float h1[kH / 2];
    {
        const float x0 = L.X[s0 + sl][0], x1 = L.X[s0 + sl][1], x2 = L.X[s0 + sl][2];
#pragma unroll
        for (int k = 0; k < kH / 2; ++k) {
            const int i = 2 * k + h;
            float a = L.B1[i];
            a = fmaf(L.W1[i * 3 + 0], x0, a);
            a = fmaf(L.W1[i * 3 + 1], x1, a);
            a = fmaf(L.W1[i * 3 + 2], x2, a);
            h1[k] = fmaxf(a, 0.f);
            L.H1[(s0 + sl) * kRow + i] = h1[k];
        }
    }
    // layer 2 pre-activations Z[s][j], j = sl and sl + 32
    v16f z0, z1;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        z0[r] = L.B2[sl];
        z1[r] = L.B2[32 + sl];
    }
#pragma unroll
    for (int k = 0; k < kH / 2; ++k) {
        z0 = mfma32(h1[k], L.W2[sl * kRow + 2 * k + h], z0);
        z1 = mfma32(h1[k], L.W2[(32 + sl) * kRow + 2 * k + h], z1);
    }
    // output, residual and G2 = dL/dZ; this lane's column sums of G2 and dy H2
    const float w30 = L.W3[sl], w31 = L.W3[32 + sl];
    float b20 = 0.f, b21 = 0.f, g30 = 0.f, g31 = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int s = s0 + 8 * (r >> 2) + 4 * h + (r & 3);
        const float a0 = fmaxf(z0[r], 0.f), a1 = fmaxf(z1[r], 0.f);
        float out = fmaf(a1, w31, a0 * w30);
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) out += __shfl_xor(out, o);
        const float res = out + b3 - L.T[s];
        const float dy = 2.f * L.WS[s] * res;
        if (sl == 0) {
            L.DY[s] = dy;
            L.WR2[s] = L.WS[s] * res * res;
        }
        const float g0 = a0 > 0.f ? dy * w30 : 0.f, g1 = a1 > 0.f ? dy * w31 : 0.f;
        L.G2[s * kRow + sl] = g0;
        L.G2[s * kRow + 32 + sl] = g1;
        b20 += g0;
        b21 += g1;
        g30 = fmaf(dy, a0, g30);
        g31 = fmaf(dy, a1, g31);
    }
    __syncthreads();
    // G1 = (G2 W2) where layer 1 was active; column sums of G1 and G1 x
    v16f y0 = {}, y1 = {};
#pragma unroll
    for (int k = 0; k < kH / 2; ++k) {
        const float a = L.G2[(s0 + sl) * kRow + 2 * k + h];
        y0 = mfma32(a, L.W2[(2 * k + h) * kRow + sl], y0);
        y1 = mfma32(a, L.W2[(2 * k + h) * kRow + 32 + sl], y1);
    }
    float c0[4] = {0.f, 0.f, 0.f, 0.f}, c1[4] = {0.f, 0.f, 0.f, 0.f};  // db1, dW1 of units sl and sl + 32
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int s = s0 + 8 * (r >> 2) + 4 * h + (r & 3);
        const float g0 = L.H1[s * kRow + sl] > 0.f ? y0[r] : 0.f;
        const float g1 = L.H1[s * kRow + 32 + sl] > 0.f ? y1[r] : 0.f;
        c0[0] += g0;
        c1[0] += g1;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            c0[1 + c] = fmaf(g0, L.X[s][c], c0[1 + c]);
            c1[1 + c] = fmaf(g1, L.X[s][c], c1[1 + c]);
        }
    }
    const float col0[6] = {c0[0], c0[1], c0[2], c0[3], b20, g30};
    const float col1[6] = {c1[0], c1[1], c1[2], c1[3], b21, g31};
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const float u = col0[q] + __shfl_xor(col0[q], 32), v = col1[q] + __shfl_xor(col1[q], 32);
        L.red[wave][q][lane] = h ? v : u;  // lanes 0..31: units 0..31, lanes 32..63: units 32..63
    }
    // dW2[j][i] = sum over the tile of G2[s][j] H1[s][i], one quadrant per wave
    const int j0 = 32 * (wave >> 1), i0 = 32 * (wave & 1);
    v16f d = {};
#pragma unroll 16
    for (int k = 0; k < kTile / 2; ++k)
        d = mfma32(L.G2[(2 * k + h) * kRow + j0 + sl], L.H1[(2 * k + h) * kRow + i0 + sl], d);
    float* out = part + (size_t)blockIdx.x * (kNP + 2);
#pragma unroll
    for (int r = 0; r < 16; ++r)
        out[kOffW2 + (j0 + 8 * (r >> 2) + 4 * h + (r & 3)) * kH + i0 + sl] = d[r];
    __syncthreads();
    // the small entries: waves in order
    for (int e = tid; e < 6 * kH; e += kBlk) {
        const int q = e / kH, i = e % kH;
        float a = 0.f;
        for (int k = 0; k < kBlk / 64; ++k) a += L.red[k][q][i];
        const int dst = q == 0 ? kOffB1 + i : (q < 4 ? kOffW1 + 3 * i + q - 1 : (q == 4 ? kOffB2 + i : kOffW3 + i));
        out[dst] = a;
    }
    if (wave < 3) {
        const float* v = wave == 0 ? L.DY : (wave == 1 ? L.WR2 : L.WS);
        float a = v[lane] + v[lane + 64];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o);
        if (lane == 0) out[wave == 0 ? kOffB3 : kNP + wave - 1] = a;
    }
}
static_assert(kTile == 128 && kBlk == 256, "four waves of 32 samples, two sums of 64");

// grad[p] = (sum over tiles, in double, in an order set by ntiles alone) / sum
// w; loss likewise.  64 entries per workgroup, the tiles dealt over its 16
// waves: one thread per entry and a serial sum of w took 117 us on 256 tiles,
// this 8 us.
constexpr int kRedBlk = 1024;
__global__ __launch_bounds__(kRedBlk) void k_mlp_grad_reduce(int ntiles, const float* __restrict__ part,
                                                             float* __restrict__ grad, double* __restrict__ loss) {
    __shared__ double s_w[kRedBlk / 64];
    __shared__ double s_p[kRedBlk / 64][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    constexpr int kG = kRedBlk / 64;
    double sw = 0.0;
    for (int b = threadIdx.x; b < ntiles; b += kRedBlk) sw += part[(size_t)b * (kNP + 2) + kNP + 1];
    for (int o = 32; o > 0; o >>= 1) sw += __shfl_xor(sw, o);
    if (lane == 0) s_w[g] = sw;
    const int p = blockIdx.x * 64 + lane;
    double a = 0.0;
    if (p < kNP + 1)
        for (int b = g; b < ntiles; b += kG) a += part[(size_t)b * (kNP + 2) + p];
    s_p[g][lane] = a;
    __syncthreads();
    if (g != 0 || p >= kNP + 1) return;
    sw = 0.0;
    a = 0.0;
    for (int k = 0; k < kG; ++k) {
        sw += s_w[k];
        a += s_p[k][lane];
    }
    const double v = sw > 0.0 ? a / sw : 0.0;
    if (p < kNP) grad[p] = (float)v;
    else *loss = v;
}

__global__ void k_adam(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, int count, float lr, float b1, float b2, float eps, float c1, float c2) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    float gi = g[i];
    float mi = b1 * m[i] + (1.f - b1) * gi;
    float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

}  // namespace

// Features of the graph into g->feat (n x 3 float) and g->core (u32), built
// once per graph.
bc_status graph_features(bc_graph* g, hipStream_t s) {
    std::lock_guard<std::mutex> lk(g->cache_mu);
    if (g->have_feat) return BC_OK;
    const int32_t n = g->dg.n;
    Carve out;
    out.add(g->feat, sizeof(float) * 3 * (size_t)std::max(n, 1));
    out.add(g->core, sizeof(uint32_t) * (size_t)std::max(n, 1));
    BC_TRY(gplace(g, out, g->fbase, s));
    if (n == 0) {
        g->have_feat = true;
        return BC_OK;
    }
    DevBuf all, s2, mm, flag, part, stat, heavy, nheavy;
    Carve c;
    c.add(s2, sizeof(uint64_t) * (size_t)n);
    c.add(heavy, sizeof(int32_t) * (size_t)n);
    c.add(nheavy, sizeof(uint32_t));
    c.add(mm, sizeof(unsigned long long) * 6);
    c.add(flag, sizeof(uint32_t));
    c.add(part, sizeof(double) * 3 * kRedBlocks);
    c.add(stat, sizeof(double) * 6);
    BC_TRY(c.place_on(all, s));
    uint32_t* h = g->core.as<uint32_t>();
    k_minmax_init<<<1, 64, 0, s>>>(mm.as<unsigned long long>());
    BC_HIP(hipMemsetAsync(nheavy.p, 0, sizeof(uint32_t), s));
    k_heavy_list<<<grid_for(n), kBlk, 0, s>>>(n, g->dg.deg, heavy.as<int32_t>(), nheavy.as<uint32_t>());
    k_feat_init<<<grid_for(n), kBlk, 0, s>>>(n, g->dg.rp, g->dg.col, g->dg.deg, s2.as<uint64_t>(), h);
    k_feat_heavy<<<1024, kBlk, 0, s>>>(heavy.as<int32_t>(), nheavy.as<uint32_t>(), g->dg.rp, g->dg.col, g->dg.deg,
                                       s2.as<uint64_t>());
    // h-index sweeps until one changes nothing; every sweep that changes
    // something lowers the sum of the estimates, so this ends
    for (;;) {
        BC_HIP(hipMemsetAsync(flag.p, 0, sizeof(uint32_t), s));
        k_hindex<<<grid_for(n), kBlk, 0, s>>>(n, g->dg.rp, g->dg.col, h, flag.as<uint32_t>());
        k_hindex_heavy<<<1024, kBlk, 0, s>>>(heavy.as<int32_t>(), nheavy.as<uint32_t>(), g->dg.rp, g->dg.col, h,
                                             flag.as<uint32_t>());
        uint32_t changed = 0;
        BC_HIP(hipMemcpyAsync(&changed, flag.p, sizeof(changed), hipMemcpyDeviceToHost, s));
        BC_HIP(hipStreamSynchronize(s));
        ++g->core_sweeps;
        if (!changed) break;
    }
    k_feat_minmax<<<grid_for(n, kReduceGrid), kBlk, 0, s>>>(n, g->dg.deg, s2.as<uint64_t>(), h, mm.as<unsigned long long>());
    const unsigned nb = grid_for(n, kRedBlocks);
    double* mean = stat.as<double>();
    double* var = mean + 3;
    k_feat_sums<<<nb, kBlk, 0, s>>>(n, g->dg.deg, s2.as<uint64_t>(), h, nullptr, part.as<double>());
    k_feat_finish<<<1, kBlk, 0, s>>>(n, (int)nb, part.as<double>(), mean);
    k_feat_sums<<<nb, kBlk, 0, s>>>(n, g->dg.deg, s2.as<uint64_t>(), h, mean, part.as<double>());
    k_feat_finish<<<1, kBlk, 0, s>>>(n, (int)nb, part.as<double>(), var);
    k_feat_write<<<grid_for(n), kBlk, 0, s>>>(n, g->dg.deg, s2.as<uint64_t>(), h, mean, var,
                                              mm.as<unsigned long long>(), g->feat.as<float>());
    BC_HIP(hipGetLastError());
    BC_HIP(hipStreamSynchronize(s));
    g->have_feat = true;
    return BC_OK;
}

bc_status mlp_forward(const float* params, const float* x, int64_t count, float* y, hipStream_t s) {
    if (count == 0) return BC_OK;
    k_mlp_forward<<<grid_for(count, 16384), kBlk, 0, s>>>(params, x, count, y);
    BC_HIP(hipGetLastError());
    return BC_OK;
}

bc_status mlp_loss_grad(const float* params, const float* x, const float* t, const float* w, int64_t rows,
                        const int32_t* idx, int64_t count, float* grad, double* loss, hipStream_t s) {
    if (!idx && count > rows) {
        set_error("count %lld exceeds rows %lld", (long long)count, (long long)rows);
        return BC_EINVAL;
    }
    const int64_t ntiles = std::max<int64_t>(1, (count + kTile - 1) / kTile);
    if (ntiles > (int64_t)1 << 24) {
        set_error("too many samples in one gradient call (%lld)", (long long)count);
        return BC_EINVAL;
    }
    DevBuf all, part, dres;
    Carve c;
    c.add(part, sizeof(float) * (kNP + 2) * (size_t)ntiles);
    c.add(dres, sizeof(double) * 2);
    BC_TRY(c.place_on(all, s));
    BC_HIP(hipMemsetAsync(dres.p, 0, sizeof(double) * 2, s));
    uint32_t* d_bad = reinterpret_cast<uint32_t*>(dres.as<double>() + 1);
    k_mlp_grad<<<(unsigned)ntiles, kBlk, 0, s>>>(params, x, t, w, rows, idx, count, part.as<float>(), d_bad);
    k_mlp_grad_reduce<<<(kNP + 1 + 63) / 64, kRedBlk, 0, s>>>((int)ntiles, part.as<float>(), grad, dres.as<double>());
    BC_HIP(hipGetLastError());
    double res[2] = {0.0, 0.0};
    BC_HIP(hipMemcpyAsync(res, dres.p, sizeof(res), hipMemcpyDeviceToHost, s));
    BC_HIP(hipStreamSynchronize(s));  // `part` is released on return
    uint32_t bad = 0;
    std::memcpy(&bad, &res[1], sizeof(bad));
    if (bad) {
        set_error("idx holds an entry outside [0, rows)");
        return BC_EINVAL;
    }
    if (loss) *loss = res[0];
    return BC_OK;
}

bc_status mlp_adam(float* params, const float* grad, float* m, float* v, int32_t step, float lr, float beta1,
                   float beta2, float eps, hipStream_t s) {
    const double c1 = 1.0 / (1.0 - std::pow((double)beta1, (double)step));
    const double c2 = 1.0 / (1.0 - std::pow((double)beta2, (double)step));
    k_adam<<<(kNP + kBlk - 1) / kBlk, kBlk, 0, s>>>(params, grad, m, v, kNP, lr, beta1, beta2, eps, (float)c1,
                                                    (float)c2);
    BC_HIP(hipGetLastError());
    return BC_OK;
}

}  // namespace bc
