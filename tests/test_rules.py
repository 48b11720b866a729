"""Rules of the launches (rules.h), run on the CPU."""

import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1507_01490_amd", "csrc")


def run(tmp_path, body):
    src = tmp_path / "rules.cpp"
    src.write_text('#include "rules.h"\n#include <cassert>\n#include <cstdio>\n#include <initializer_list>\nusing namespace bc;\nint main() {\n'
                   + body + '\nstd::puts("ok");\n}\n')
    exe = tmp_path / "rules"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unknown-pragmas", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-I", CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout == "ok\n"


def test_slots_shrink_to_what_fits(tmp_path):
    """An allocation that fails is tried with half the slots, down to one."""
    run(tmp_path, r"""
    for (int want : {1, 2, 3, 7, 8, 32})
        for (int room = 0; room <= 33; ++room) {
            int tries = 0;
            const int got = halve_until(want, [&](int k) { ++tries; return k <= room; });
            assert(got <= room && got <= want && tries <= 6);
            assert(room == 0 ? got == 0 : got >= 1);
            assert(room < want || (got == want && tries == 1));
            assert(got == 0 || got == want || 2 * got + 1 >= room);
        }
    """)


def test_only_small_first_builds_stay_in_the_pool(tmp_path):
    """12 bytes an arc and 16 a node of the first build: the pool keeps at most 1 GiB of them."""
    run(tmp_path, r"""
    const int64_t gib = (int64_t)1 << 30;
    assert(pooled_first_build(100000, 0) && pooled_first_build(300000, 5700000));
    for (int64_t n : {(int64_t)100000, (int64_t)4000000, (int64_t)2147483646})
        for (int64_t m : {(int64_t)0, (int64_t)89000000, (int64_t)90000000, (int64_t)2147483646})
            assert(pooled_first_build(n, m) == (12 * m + 16 * n <= gib));
    assert(!pooled_first_build(2147483646, 2147483646) && !pooled_first_build(500000, 180000000));
    """)


def test_direction_of_the_levels(tmp_path):
    """Bottom up from m / alpha frontier arcs on, top down below n / beta nodes."""
    run(tmp_path, r"""
    const int64_t n = 1000, m = 6000;
    for (uint64_t arcs = 0; arcs <= 6000; arcs += 1) {
        assert(next_direction(0, arcs, 10, n, m, 3.f, 24.f) == (arcs > 2000));
        assert(next_direction(0, arcs, 10, n, m, 2.f, 24.f) == (arcs > 3000));
        assert(next_direction(0, arcs, 10, n, m, 0.f, 24.f) == 0);
        assert(next_direction(0, arcs, 10, n, m, -1.f, 24.f) == 0);
        assert(next_direction(0, arcs, 10, n, m, 1e9f, 1e9f) == (arcs > 0));
    }
    for (uint32_t nodes = 0; nodes <= 1000; ++nodes) {
        assert(next_direction(1, 0, nodes, n, m, 3.f, 20.f) == (nodes >= 50));
        assert(next_direction(1, 0, nodes, n, m, 3.f, 1e-9f) == 0);
        assert(next_direction(1, 0, nodes, n, m, 3.f, 1e9f) == (nodes > 0));
    }
    const int64_t top = 2147483646;
    assert(next_direction(0, (uint64_t)top, 1, top, top, 1.5f, 24.f) == 1);
    assert(next_direction(0, (uint64_t)top, 1, top, top, 1.f, 24.f) == 0);
    """)


def test_a_bottom_up_step_has_a_wave_per_heavy_node(tmp_path):
    run(tmp_path, r"""
    assert(pull_threads(3000, 0) == 3000 && pull_threads(3000, 3000) == 192000);
    assert(pull_threads(6400, 100) == 6400 && pull_threads(6400, 101) == 6464);
    assert(pull_threads(2147483646, 33038209) == 2147483646 && pull_threads(40000000, 33038209) == 2114445376);
    """)


def test_one_workgroup_goes_bottom_up_on_graphs_with_arcs_only(tmp_path):
    run(tmp_path, r"""
    // connected graphs (m >= 2 n - 2): the rule on the arcs alone
    assert(block_pull_arcs(1000, 6000) == 6000 && block_pull_arcs(1000, 2000) == 2000);
    // few arcs per node: never, at the default
    const int64_t n = 2000000, m = 9000;
    assert(next_direction(0, m, 1500, n, block_pull_arcs(n, m), 3.f, 24.f) == 0);
    assert(next_direction(0, m, 1500, n, m, 3.f, 24.f) == 1);
    assert(next_direction(0, 1, 1, n, block_pull_arcs(n, m), 1e9f, 24.f) == 1);
    assert(block_pull_arcs(2147483646, 5) == 4294967292);
    """)


def test_factor_of_the_wide_batches_in_one_workgroup(tmp_path):
    run(tmp_path, r"""
    assert(block_alpha(true, 1000, 9000, 900, 9000) == 2.f / 3.f && block_alpha(true, 1000, 0, 0, 0) == 2.f / 3.f);
    assert(block_alpha(false, 60000, 1105268, 6300, 784000) == 0.4f);   // most arcs at a tenth of the nodes
    assert(block_alpha(false, 50000, 2999070, 10950, 1412000) == 1.f);  // less than half of the arcs
    assert(block_alpha(false, 30000, 3600000, 29990, 3599000) == 1.f);  // nearly all nodes
    assert(block_alpha(false, 1000, 6000, 0, 0) == 1.f && block_alpha(false, 5, 0, 0, 0) == 1.f);
    """)
