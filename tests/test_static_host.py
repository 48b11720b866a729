"""bc_topk_static allocates nothing on the host either: neither it nor the
level loop it runs holds a container or an allocation."""

import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1507_01490_amd", "csrc")


def body(text, head):
    """The text of the function whose definition starts with `head`, braces matched."""
    at = text.index(head)
    i = text.index("{", text.index(")", at))
    depth, j = 0, i
    while True:
        depth += {"{": 1, "}": -1}.get(text[j], 0)
        j += 1
        if depth == 0:
            return re.sub(r"//[^\n]*", "", text[i:j])


@pytest.mark.parametrize("head", ["bc_status lv_host_loop(", "bc_status run_topk_static("])
def test_no_host_allocation(head):
    code = body(open(os.path.join(CSRC, "topk.hip")).read(), head)
    assert len(code) > 1000
    found = re.findall(r"std::vector|std::string|std::deque|\bnew\b|\bmalloc\b|_ptr<|push_back|DevBuf|hipMalloc|"
                       r"hipHostMalloc", code)
    assert not found, found
