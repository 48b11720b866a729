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
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-fsanitize=undefined", "-fno-sanitize-recover=all",
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
