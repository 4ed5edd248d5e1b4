"""Every kernel the planner launches for a transform has its algorithmic bytes in
bench.py, under the name it is launched with."""
import os
import re

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def launch_names():
    with open(os.path.join(ROOT, "paper_2608_24738_amd", "csrc", "edt_host.hip"), encoding="utf-8") as f:
        text = re.sub(r"//[^\n]*|#include[^\n]*", " ", f.read())
    names = set(re.findall(r'"([a-z][a-z0-9]*_[a-z0-9_]*(?:\.[a-z0-9]+)*)"', text))
    return names - {"dt_bf", "mask_nonzero"}            # no roofline: neither is a separable pass


def test_every_launch_has_its_bytes():
    names = launch_names()
    assert {"scan_word.o16", "line_bracket_final.i16", "cdt_bracket_final", "line_bracket_idx_final",
            "line_pair_rag_final", "line_search_final", "plane_final.i8"} <= names
    for name in sorted(names):
        assert bench.algorithmic_bytes(name, 1000, 2, True) > 0, name
