"""The bottom-up step's index arithmetic on the CPU: the walks are the
kernels' own (rules.h), over checked arrays, lane by lane as a wave runs them.
Every index of the row pointers, arcs, cur words and buffers stays in bounds,
and the bits found are the OR over all in-neighbours u of cur[u] & unseen."""

import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1507_01490_amd", "csrc")

PROGRAM = r"""
#include "rules.h"
#include <cassert>
#include <cstdio>
#include <initializer_list>
#include <random>
#include <vector>
using namespace bc;

template <class T>
struct Checked {  // an array whose reads are checked, from an offset on
    const std::vector<T>* v;
    size_t off = 0;
    T operator[](size_t i) const {
        assert(off + i < v->size());
        return (*v)[off + i];
    }
};

struct Graph {
    int32_t n;
    std::vector<int32_t> irp, icol;
};

// in-lists of the given lengths, then random ones
static Graph lists(int32_t n, const std::vector<int>& len, std::mt19937_64& rng) {
    Graph g{n, {0}, {}};
    for (int32_t v = 0; v < n; ++v) {
        const int d = v < (int)len.size() ? len[(size_t)v] : (int)(rng() % 12);
        for (int i = 0; i < d; ++i) g.icol.push_back((int32_t)(rng() % (uint64_t)n));
        g.irp.push_back((int32_t)g.icol.size());
    }
    return g;
}

template <int WW, int kAhead>
static void step(const Graph& g, double density, std::mt19937_64& rng) {
    const int32_t n = g.n;
    std::vector<uint64_t> seen((size_t)n * WW), cur((size_t)n * WW), got((size_t)n * WW, 0), act(WW);
    auto word = [&](double p) {
        uint64_t x = 0;
        for (int b = 0; b < 64; ++b) x |= (uint64_t)(rng() % 1000 < (uint64_t)(1000 * p)) << b;
        return x;
    };
    for (auto& x : seen) x = word(0.5);
    for (auto& x : cur) x = word(density);
    for (auto& x : act) x = rng() % 4 ? ~0ull : word(0.5);
    const Checked<int32_t> irp{&g.irp}, icol{&g.icol};
    const Checked<uint64_t> sn{&seen};
    uint64_t read = 0;
    // pull_nodes: 64 nodes of a wave in WW rounds, then node i reads its words back
    for (int64_t base = 0; base < n; base += 64) {
        std::vector<uint64_t> buf(64 * WW, 0);
        for (int r = 0; r < WW; ++r)
            for (int lane = 0; lane < 64; ++lane) {
                const int64_t w = pull_node<WW>(base, r, lane);
                const int j = lane % WW;
                uint64_t acc = 0;
                assert(w >= base && w < base + 64);
                if (w < n) {
                    const uint64_t unv = act[(size_t)j] & ~sn[(size_t)w * WW + j];
                    const int32_t e0 = irp[(size_t)w], e1 = irp[(size_t)w + 1];
                    if (unv && e1 - e0 <= kPullWave) {
                        const uint32_t k = pull_short<WW, kAhead>(icol, Checked<uint64_t>{&cur, (size_t)j}, e0, e1, unv, acc);
                        assert(k <= (uint32_t)(e1 - e0));
                        read += k;
                    }
                }
                const int at = pull_word(r, lane);
                assert(at >= 0 && at < 64 * WW);
                buf[(size_t)at] = acc;
            }
        for (int lane = 0; lane < 64; ++lane)
            for (int q = 0; q < WW; ++q)
                if (base + lane < n) got[(size_t)(base + lane) * WW + q] = buf[(size_t)(lane * WW + q)];
                else assert(buf[(size_t)(lane * WW + q)] == 0);
    }
    // pull_heavy: all 64 lanes on one list, joined per word after every part
    for (int32_t w = 0; w < n; ++w) {
        const int32_t h0 = irp[(size_t)w], h1 = irp[(size_t)w + 1];
        if (h1 - h0 <= kPullWave) continue;
        std::vector<uint64_t> acc(WW, 0), unv(WW);
        for (int j = 0; j < WW; ++j) unv[(size_t)j] = act[(size_t)j] & ~sn[(size_t)w * WW + j];
        for (int64_t eb = h0; eb < h1; eb += (64 / WW) * kAhead) {
            if (acc == unv) break;
            std::vector<uint64_t> joined(acc);
            for (int lane = 0; lane < 64; ++lane) {
                const int j = lane % WW;
                uint64_t part = acc[(size_t)j];
                const int32_t end = pull_long<WW, kAhead>(icol, Checked<uint64_t>{&cur, (size_t)j}, eb, h1, lane,
                                                          unv[(size_t)j], part);
                assert(end > eb && end <= h1 && end <= eb + (64 / WW) * kAhead);
                joined[(size_t)j] |= part;
            }
            acc = joined;
        }
        for (int j = 0; j < WW; ++j) got[(size_t)w * WW + j] = acc[(size_t)j];
    }
    for (int32_t w = 0; w < n; ++w)
        for (int j = 0; j < WW; ++j) {
            uint64_t want = 0;
            for (int32_t e = g.irp[(size_t)w]; e < g.irp[(size_t)w + 1]; ++e)
                want |= cur[(size_t)g.icol[(size_t)e] * WW + j];
            assert(got[(size_t)w * WW + j] == (want & act[(size_t)j] & ~seen[(size_t)w * WW + j]));
        }
    assert(read <= (uint64_t)g.icol.size() * WW);
}

int main() {
    std::mt19937_64 rng(7);
    const std::vector<int> edge = {0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 66, 96, 127, 128, 129,
                                   255, 256, 257, 511, 512, 513, 1025, 0};
    for (int32_t n : {1, 31, 63, 64, 65, 200, 1100})
        for (double density : {0.0, 0.002, 0.05, 0.9}) {
            Graph g = lists(n, edge, rng);
            step<1, 8>(g, density, rng); step<1, 4>(g, density, rng);
            step<2, 8>(g, density, rng); step<2, 4>(g, density, rng);
            step<4, 8>(g, density, rng); step<4, 4>(g, density, rng);
        }
    // lists that end at the largest arc count: positions only, the arrays are virtual
    struct AnyArc { int32_t operator[](int64_t e) const { assert(e >= 2147483000 && e < 2147483646); return 0; } };
    struct NoBits { uint64_t operator[](size_t) const { return 0; } };
    uint64_t acc = 0;
    const uint32_t k = pull_short<1, 8>(AnyArc{}, NoBits{}, 2147483601, 2147483646, ~0ull, acc);
    assert(k == 45 && acc == 0);
    for (int lane = 0; lane < 64; ++lane)
        for (int64_t eb : {2147483000LL, 2147483300LL, 2147483640LL})
            assert((pull_long<1, 8>(AnyArc{}, NoBits{}, eb, 2147483646, lane, ~0ull, acc) <= 2147483646));
    std::puts("ok");
}
"""


def test_walks_stay_in_bounds_and_find_every_bit(tmp_path):
    src = tmp_path / "pull.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "pull"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unknown-pragmas", "-Werror", "-fsanitize=undefined,address",
                    "-fno-sanitize-recover=all", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout == "ok\n"


def test_kernels_run_these_walks():
    text = open(os.path.join(CSRC, "topk.hip")).read()
    for name in ("pull_node<WW>(", "pull_word(", "pull_short<WW, kAhead>(", "pull_long<WW, kAhead>("):
        assert text.count(name) == 1, name
    assert "icol[" not in text
