"""Every kernel that indexes a level's lists by their lengths checks these
against n first, and the host stops at what they report."""

import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1507_01490_amd", "csrc")
TEXT = open(os.path.join(CSRC, "topk.hip")).read()


def body(head):
    at = TEXT.index(head)
    i = TEXT.index("{", at)
    depth, j = 0, i
    while True:
        depth += {"{": 1, "}": -1}.get(TEXT[j], 0)
        j += 1
        if depth == 0:
            return TEXT[i:j]


def test_wide_kernels_check_the_reached_list():
    for kernel, inner in (("void k_plain_count(", "plain_count_body"), ("void k_plain_build(", "plain_build_body")):
        b = body(kernel)
        assert 0 < b.index("list_outgrown(G, C)") < b.index(inner)
    assert "C->nlen <= (uint32_t)G.n" in body("bool list_outgrown(")


def test_narrow_kernel_checks_all_three_lists():
    b = body("void k_plain_run(")
    assert re.search(r"if \(bad \|\| flen > n \|\| clen > n\) \{\s*state = LV_BAD;\s*break;", b)
    assert b.index("bad = nlen > n;") < b.index("build_level<WW>(")
    assert "bool bad = C->err != 0;" in b


def test_host_stops_at_a_bad_list():
    b = body("bc_status lv_host_loop(")
    assert "r.state == LV_BAD ||" in b and b.index("LV_BAD") < b.index("k_plain_expand<WW>")
