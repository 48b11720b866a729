// Index arithmetic and rules of the kernels and their launches that need no
// device builtin: plain C++, so that the tests run the same code on the CPU
// (under the undefined-behaviour sanitizer) at sizes no test graph reaches.
#pragma once

#include <stddef.h>
#include <stdint.h>

#if defined(__HIPCC__)
#define BC_HD __host__ __device__ __forceinline__
#else
#define BC_HD inline
#endif

namespace bc {

// ---- arcs dealt out in tiles
//
// Offsets and ids are int32 and go up to 2^31 - 2, so an index that steps by
// more than one passes 2^31 - 1 behind the last arc of the largest graphs.
// Loops over a tile therefore run over the arcs' positions in the tile, and
// loops over a whole list in 64 bits.

constexpr int kArcTile = 2048;  // consecutive arcs per workgroup of the arc kernels: 8 per thread

BC_HD int64_t tile_count(int64_t m) { return (m + kArcTile - 1) / kArcTile; }
BC_HD int32_t tile_first(int64_t tile) { return (int32_t)(tile * kArcTile); }
// arcs in the tile whose first arc is e0 < m
BC_HD int32_t tile_arcs(int32_t e0, int64_t m) { return (int32_t)(m - e0 < kArcTile ? m - e0 : kArcTile); }

// The positions of a tile of `len` arcs that thread tid of kBlk takes.
template <int kBlk, class F>
BC_HD void tile_each(int32_t tid, int32_t len, F f) {
    for (int32_t i = tid; i < len; i += kBlk) f(i);
}

// Distance of the 64 probes of a search over [lo, hi), lo < hi.
BC_HD int32_t probe_step(int32_t lo, int32_t hi) { return (hi - lo - 1) / 64 + 1; }

// The end of the first `most` arcs of the row [b, e).
BC_HD int32_t first_arcs(int32_t b, int32_t e, int32_t most) { return e - b > most ? b + most : e; }


// ---- direction of the levels

// Whether the next level runs bottom up: from m / alpha frontier arcs on (alpha
// = 0: never), and until the frontier holds less than n / beta nodes.  Written
// as products: two quotients cost 0.3 us a level in the persistent kernels.
BC_HD uint32_t next_direction(uint32_t pull, uint64_t arcs, uint32_t nodes, int64_t n, int64_t m, float alpha,
                              float beta) {
    if (!pull && alpha > 0.f && (double)arcs * alpha > (double)m) return 1;
    if (pull && (double)nodes * beta < (double)n) return 0;
    return pull;
}

// The arcs that count as all of them for a level of one workgroup: its
// bottom-up step passes over every node, whose cost a graph of few arcs per
// node does not earn back (2 * 10^6 nodes, 1,500 of them with arcs: 7.5 ms a
// step, against 1 us for the frontier of a batch top down).  A connected
// undirected graph has 2 n - 2 arcs or more.
BC_HD int64_t block_pull_arcs(int64_t n, int64_t m) { return m > 2 * n ? m : 2 * n; }

// The factor of pull_alpha for levels of one workgroup at W = 256, where a
// bottom-up step reads four words of every node that is not complete.  (Job
// launches of one query, k = 10; ms at factor 1 and at the one taken, and top
// down only before there was a bottom-up step.)
//   directed: a node that no source reaches is scanned in full, level after
//     level (R-MAT scale 17, batched query: 6.4 -> 3.5, before 6.1)
//   most arcs at a few nodes of many: these take a wave each and are walked one
//     after the other (collaboration graph of 20,000 nodes 7.2 -> 6.1, before
//     7.1; 60,000 29.4 -> 25.3, before 25.4; 200,000 71 -> 64; 500,000 269 ->
//     241).  Where fewer of the arcs are theirs (Barabasi-Albert graph, 60 arcs
//     a node) it would lose, 21.4 -> 23.8, or where most nodes are such (a
//     random graph of 120 arcs a node), 31 -> 41.
BC_HD float block_alpha(bool directed, int64_t n, int64_t m, int64_t heavy, int64_t heavy_arcs) {
    if (directed) return 2.f / 3.f;
    return 2 * heavy_arcs > m && 2 * heavy < n ? 0.4f : 1.f;
}

// ---- bottom-up step
//
// WW lanes share a node, lane j on word j, and a wave takes 64 nodes in WW
// rounds; a node of more than kPullWave in-arcs takes the whole wave.

constexpr int32_t kPullWave = 64;

// Node of a lane in round r of the 64 nodes from `base` on, and the word of a
// wave's buffer for what it found: node i of the 64 has words i WW .. i WW + WW - 1.
template <int WW>
BC_HD int64_t pull_node(int64_t base, int r, int lane) {
    return base + r * (64 / WW) + lane / WW;
}
BC_HD int pull_word(int r, int lane) { return r * 64 + lane; }

// The arcs e0, e0 + step, ... below e1 of a lane's part of a list: the bits of
// `unv` found among the neighbours' words cur_j.  kAhead arcs at a time, their
// targets and then their words all in flight together, until every bit is
// found.  Returns the arcs read.
template <int WW, int kAhead, class Col, class Cur>
BC_HD uint32_t pull_walk(const Col& icol, const Cur& cur_j, int64_t e0, int32_t e1, int32_t step, uint64_t unv,
                         uint64_t& acc) {
    uint32_t read = 0;
    int64_t e = e0;
    while (e < e1 && acc != unv) {
        int32_t u[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const int64_t x = e + (int64_t)q * step;
            u[q] = icol[x < e1 ? x : e];  // past the end: the first arc again
        }
        uint64_t c = 0;
#pragma unroll
        for (int q = 0; q < kAhead; ++q) c |= cur_j[(size_t)u[q] * WW];
        acc |= c & unv;
        read += kAhead;
        e += (int64_t)kAhead * step;
    }
    return read;
}

// A short list [e0, e1), walked by the lane of each word; the arcs read.
template <int WW, int kAhead, class Col, class Cur>
BC_HD uint32_t pull_short(const Col& icol, const Cur& cur_j, int32_t e0, int32_t e1, uint64_t unv, uint64_t& acc) {
    const uint32_t read = pull_walk<WW, kAhead>(icol, cur_j, e0, e1, 1, unv, acc), len = (uint32_t)(e1 - e0);
    return read < len ? read : len;
}

// A lane's arcs among the next (64 / WW) kAhead of a long list from eb on; the
// end of those.
template <int WW, int kAhead, class Col, class Cur>
BC_HD int32_t pull_long(const Col& icol, const Cur& cur_j, int64_t eb, int32_t h1, int lane, uint64_t unv,
                        uint64_t& acc) {
    constexpr int kGroups = 64 / WW;
    const int64_t to = eb + kGroups * kAhead;
    const int32_t end = (int32_t)(to < h1 ? to : h1);
    (void)pull_walk<WW, kAhead>(icol, cur_j, eb + lane / WW, end, kGroups, unv, acc);
    return end;
}

// Threads a bottom-up step has work for: one per node, and a wave for each of
// the `heavy` nodes of many in-arcs, which outnumber the others' waves on a
// dense graph (3,000 nodes of 600 arcs: 3 workgroups by the nodes alone, the
// seed batch of a query 0.34 ms; 188 by the heavy ones, 0.14 ms).
BC_HD int64_t pull_threads(int64_t n, int64_t heavy) { return heavy * 64 > n ? heavy * 64 : n; }

// ---- uploads

// Whether the first build of a renumbered graph (n nodes, at most m arcs),
// which ends with the upload, comes from the stream-ordered pool.  The pool
// never gives memory back, and later calls size their slots by what is free,
// so only up to 1 GiB of it does: there new memory (0.1 ms a MB) and the free
// of a plain allocation (250 us) would take longer than the build's kernels.
BC_HD bool pooled_first_build(int64_t n, int64_t m) { return 12 * m + 16 * n <= (int64_t)1 << 30; }

// ---- level-synchronous slots

// Bytes per node of a slot of W = 64 WW sources: seen and nxt, cur, stamp (WW >
// 1), three lists.
constexpr uint64_t slot_node_bytes(int W) { return 24 * (uint64_t)(W / 64) + (W > 64 ? 4 : 0) + 12; }

constexpr uint64_t kLvBytes = (uint64_t)1 << 30;  // of their slots, unless one alone needs more
constexpr int kMaxSlots = 32;                     // batches the level-synchronous kernels run side by side
constexpr uint64_t kLvCtlBytes = 18 << 10;        // of a slot's control block and sources

// Slots for `batches` batches within `room` bytes: a power of two (so that
// graphs of a size ask the pool for the same bytes), at most kLvBytes: eight
// batches fill the GPU on a graph whose slot takes 100 MB, and new memory
// costs 0.1 ms a MB.
inline int lv_slots(uint64_t batches, uint64_t slot_bytes, uint64_t room) {
    if (room > kLvBytes) room = kLvBytes;
    int lv = 1;
    while (lv < kMaxSlots && (uint64_t)lv < batches && 2 * (uint64_t)lv * slot_bytes <= room) lv *= 2;
    return lv;
}

// Width and number of the seed batches of a query (k results, n nodes, W
// sources per batch) for the options seed_width (0: automatic) and
// seed_batches (negative: enough for k sources).
struct SeedPlan {
    int sw;
    uint32_t batches;  // of width sw
};
inline SeedPlan seed_plan(int32_t seed_width, int32_t seed_batches, int32_t k, int32_t n, int W) {
    int sw = seed_width > 0 ? seed_width : (k > W ? 256 : W);
    if (sw < W || sw % W != 0) sw = W;
    const int64_t nb = ((int64_t)n + sw - 1) / sw;
    const int64_t sb = seed_batches >= 0 ? seed_batches : ((int64_t)k + sw - 1) / sw;
    return SeedPlan{sw, (uint32_t)(sb < nb ? sb : nb)};
}

// The first of want, want / 2, ... 1 that `fits` takes, or 0 if it takes none.
template <class Fits>
inline int halve_until(int want, Fits fits) {
    for (int k = want; k > 0; k /= 2)
        if (fits(k)) return k;
    return 0;
}

}  // namespace bc
