"""Index arithmetic of the arc kernels at the largest arc and node counts the
library accepts (2^31 - 2), where a 32-bit index that steps by more than one
wraps.  The kernels' own helpers run on the CPU under the undefined-behaviour
sanitizer; the sources hold no other loop of that kind."""

import glob
import os
import re
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1507_01490_amd", "csrc")

PROGRAM = r"""
#include "rules.h"
#include <cassert>
#include <cstdio>
#include <initializer_list>
#include <vector>
using namespace bc;

// every arc of the tile that starts at e0 is taken once, by one thread
static void tile(int64_t m, int32_t e0) {
    const int32_t len = tile_arcs(e0, m);
    assert(len >= 1 && len <= kArcTile && (int64_t)e0 + len <= m);
    std::vector<int> seen((size_t)len, 0);
    for (int32_t tid = 0; tid < 256; ++tid)
        tile_each<256>(tid, len, [&](int32_t i) {
            const int32_t e = e0 + i;
            assert(e >= e0 && e < m);
            ++seen[(size_t)i];
        });
    for (int x : seen) assert(x == 1);
}

// the 64-probe search with the row starts rp(r) = r * step_ (r <= n)
static int32_t row_of(int32_t n, int64_t per, int64_t e) {
    int32_t lo = 0, hi = n;
    for (int rounds = 0; hi - lo > 1; ++rounds) {
        assert(rounds < 8);
        const int32_t step = probe_step(lo, hi);
        assert(step >= 1);
        int32_t c = 0;
        for (int lane = 0; lane < 64; ++lane) {
            const int64_t p = (int64_t)lo + (int64_t)(lane + 1) * step;
            c += p < hi && p * per <= e;
        }
        lo += c * step;
        const int64_t next = (int64_t)lo + step;
        if (next < hi) hi = (int32_t)next;
    }
    return lo;
}

int main() {
    const int64_t top = 2147483646;  // the largest count accepted
    const int64_t ms[] = {1, 255, 256, 257, 2047, 2048, 2049, 5000, top, top - 1, top - 254, top - 255, top - 256,
                          top - 2046, top - 2047, top - 2048};
    for (int64_t m : ms) {
        assert(tile_count(m) * kArcTile >= m && (tile_count(m) - 1) * kArcTile < m);
        tile(m, tile_first(0));
        tile(m, tile_first(tile_count(m) - 1));
    }
    const int32_t ns[] = {1, 2, 63, 64, 65, 1000, 4097, (int32_t)top, (int32_t)top - 62, (int32_t)top - 63};
    for (int32_t n : ns)
        for (int64_t r : {(int64_t)0, (int64_t)n / 3, (int64_t)n - 2, (int64_t)n - 1})
            if (r >= 0) assert(row_of(n, 1, r) == r);
    for (int32_t b : {0, 5, (int32_t)top - 5, (int32_t)top - 2, (int32_t)top})
        for (int64_t d : {0, 1, 3, 4, 5, 9}) {
            const int64_t e = b + d > top ? top : b + d;
            const int32_t x = first_arcs(b, (int32_t)e, 4);
            assert(x >= b && x <= e && x - b == (e - b > 4 ? 4 : e - b));
        }
    std::puts("ok");
}
"""


def test_tiles_and_searches_at_the_limit(tmp_path):
    src = tmp_path / "limits.cpp"
    src.write_text(PROGRAM)
    exe = tmp_path / "limits"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unknown-pragmas", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I", CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout == "ok\n"


def strided_int_loops(text):
    """Loops over a signed 32-bit index that a stride of more than one carries past its bound."""
    out = []
    for var, bound, step in re.findall(r"for \(int32_t (\w+) = [^;]+; ([^;]+); ([^{;]+?)\)", text):
        m = re.search(rf"\b{var} \+= (.+)$", step.strip())
        if m and m.group(1).strip() != "1":
            out.append((var, bound, m.group(1)))
    return out


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(CSRC, "*.h")) + glob.glob(os.path.join(CSRC, "*.hip"))),
                         ids=os.path.basename)
def test_no_strided_32_bit_index(path):
    # bounds that are small by construction: positions in a tile (len), results copied in chunks (cnt <= k)
    loops = [x for x in strided_int_loops(open(path).read()) if x[1] not in ("i < len", "i0 < cnt")]
    assert not loops, loops
