"""The index rules of csrc/bounds.h at the ends of their ranges (CPU: compiled
as constant expressions, so that a wrong value is a compile error)."""
import os
import subprocess

import pytest

from paper_2110_02848_amd import build

CASES = {
    # a heavy list whose refused entries would lie past its end
    "list_entries": """
        static_assert(list_entries(0, 0, 0) == 0);
        static_assert(list_entries(0, 256, 4096) == 256);
        static_assert(list_entries(4090, 6, 4096) == 6);
        static_assert(list_entries(4090, 7, 4096) == 6);
        static_assert(list_entries(4096, 1, 4096) == 0);
        static_assert(list_entries(4097, 5, 4096) == 0);
        static_assert(list_entries(1, 0xffffffffu, 4096) == 4095);
        static_assert(list_entries(0xfffffff0u, 256, 0xffffffffu) == 15);
    """,
    # 64 states at a time up to the largest graph
    "lane_state": """
        static_assert(lane_state(0, 0, 0) == 0);
        static_assert(lane_state(0, 5, 5) == 5);
        static_assert(lane_state(0, 4, 5) == 4);
        static_assert(lane_state(1, 0, 64) == 64);
        static_assert(lane_state(0x1ffffff, 62, 0x7fffffff) == 0x7ffffffe);
        static_assert(lane_state(0x1ffffff, 63, 0x7fffffff) == 0x7fffffff);
        static_assert(lane_state(0x1ffffff, 63, 0x7fffffc1) == 0x7fffffc1);
        static_assert(lane_state(0x2000000, 0, 0x7fffffff) == 0x7fffffff);
    """,
}


@pytest.mark.parametrize("rule", sorted(CASES))
def test_rule(rule, tmp_path):
    src = tmp_path / "rule.cpp"
    src.write_text('#include "bounds.h"\nusing namespace fstc;\n' + CASES[rule])
    p = subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-Wall", "-Werror", "-I",
                        os.path.abspath(build.CSRC), str(src)], capture_output=True, text=True)
    assert p.returncode == 0, p.stderr
