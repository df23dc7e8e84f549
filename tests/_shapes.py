"""The dispatch rules of csrc/shapes.h, asked through a small host program (no HIP), and the cases
that the GPU tests take from them: each names the form that it has to reach, which
test_shapes.py checks at 256 CUs (the MI355X's number)."""
from __future__ import annotations

import functools
import os
import subprocess
import tempfile

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CUS = 256

_MAIN = r"""
#include "paper_2503_08467_amd/csrc/shapes.h"
#include <iostream>
#include <string>
using namespace moe;
int main() {
    std::string what;
    while (std::cin >> what) {
        if (what == "route") {  // bf16 T h E k grouping-wanted cus
            int bf16, h, E, k, want, cus; int64_t T;
            std::cin >> bf16 >> T >> h >> E >> k >> want >> cus;
            const bool group = want && route_groups(bf16, T, h, E, k);
            if (route_in_lds(bf16, h, E)) { std::cout << "lds" << (group ? " grouped" : "") << "\n"; continue; }
            const int b = route_blocks(T, E, group, cus);
            std::cout << b << " x " << route_stage(E, b, route_run(bf16, h, E)) << (group ? " grouped" : "") << "\n";
        }
    }
}
"""


@functools.lru_cache(None)
def _program():
    d = tempfile.TemporaryDirectory()
    src, exe = os.path.join(d.name, "main.cpp"), os.path.join(d.name, "main")
    with open(src, "w", encoding="utf-8") as fh:
        fh.write(_MAIN)
    subprocess.run(["g++", "-std=c++17", "-I", ROOT, "-o", exe, src], check=True)
    return d, exe


def ask(lines):
    """Answers of the rules to query lines, one each."""
    out = subprocess.run([_program()[1]], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True).stdout
    got = out.splitlines()
    assert len(got) == len(lines), (len(got), len(lines))
    return got


# (dtype, T, h, E, k) -> form of the routing launch of moe_route_dispatch: blocks of 16 tokens per
# workgroup x K steps per stage
ROUTE_FORMS = [
    ("bf16", 64, 4096, 8, 2, "1 x 4"),              # rows too long for one workgroup's 64 tokens
    ("f32", 64, 264, 32, 2, "1 x 2"),
    ("bf16", 100, 1280, 20, 2, "1 x 5"),              # one stage holds a wave's run
    ("f32", 80, 776, 8, 2, "1 x 4"),
    ("bf16", 100, 1536, 16, 2, "1 x 6"),
    ("bf16", 64, 1000, 60, 2, "2 x 1"),
    ("bf16", 40, 512, 24, 2, "4 x 1 grouped"),
    ("f32", 33, 256, 16, 8, "4 x 2 grouped"),
    ("bf16", 32, 1000, 60, 2, "2 x 1 grouped"),
    ("bf16", 32, 1536, 8, 2, "2 x 2 grouped"),
    ("bf16", 17, 768, 8, 2, "2 x 3 grouped"),
    ("f32", 32, 1024, 16, 2, "1 x 4"),
    ("f32", 20, 2048, 32, 2, "2 x 1 grouped"),
    ("bf16", 4097, 1024, 16, 2, "2 x 2"),           # an even number of steps in a wave's run
    ("bf16", 4097, 776, 3, 2, "2 x 2"),
    ("bf16", 4100, 768, 8, 1, "2 x 3"),             # a run of three steps
    ("f32", 5000, 328, 12, 3, "2 x 3"),
    ("bf16", 16384, 264, 24, 2, "4 x 1"),
    ("f32", 16399, 72, 32, 2, "4 x 1"),
    ("bf16", 4099, 264, 200, 2, "2 x 1"),           # E > 128: two blocks past one round of the CUs
    ("f32", 4097, 72, 256, 3, "2 x 1"),
    ("bf16", 4096, 264, 200, 2, "1 x 1"),
]
