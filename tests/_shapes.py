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
static const char* name(GemmShape s) {
    switch (s) {
        case kTurns256x256: return "turns";
        case kPairs128x256: return "pairs";
        case kTile64x128: return "64x128";
        case kTile64x256: return "64x256";
        case kTile128x128: return "128x128";
        case kTile128x256: return "128x256";
        case kTile128x384: return "128x384";
    }
    return "?";
}
static std::string streamed(int64_t A, int E, int64_t N, bool swiglu, bool bf16, int cus) {
    const int nc = stream_width(A, E, N, swiglu, cus);
    const int blocks = nc == 64 ? stream_launch_blocks(A, E, tiles_of(N, swiglu ? 32 : 64), bf16, cus) : 1;
    return std::to_string(nc) + "x" + std::to_string(blocks);
}
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
        } else if (what == "ffn") {  // bf16 A E h f swiglu cus: up / down
            int bf16, E, h, swiglu, cus; int64_t A, f;
            std::cin >> bf16 >> A >> E >> h >> f >> swiglu >> cus;
            const int64_t fp = (f + 127) / 128 * 128;
            if (stream_rows(A, E, h, fp, swiglu, bf16, cus))
                std::cout << "stream " << streamed(A, E, fp, swiglu, bf16, cus) << " / " << streamed(A, E, h, false, bf16, cus);
            else if (!bf16) std::cout << "fp32";
            else std::cout << name(up_shape(A, E, h, static_cast<int>(fp), swiglu, cus)) << " / "
                           << name(down_shape(A, E, static_cast<int>(fp), h, cus));
            std::cout << (hands_over_sums(A, fp, bf16) ? " sums " + std::to_string(down_parts(A, fp, bf16,
                          stream_rows(A, E, h, fp, swiglu, bf16, cus))) : "") << "\n";
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

# (rows per expert, h, f, act) -> tiles of the bf16 expert step, up / down
TILE_FORMS = [
    ([37] * 14 + [40, 64, 0], 96, 200, "gelu", "64x128 / 128x128"),      # thin experts, few columns
    ([20] * 127 + [64], 384, 384, "gelu", "64x256 / 64x256"),            # ... many
    ([20] * 127 + [64], 384, 200, "swiglu", "64x256 / 64x256"),
    ([47] * 100 + [65, 1], 192, 384, "gelu", "64x256 / 128x128"),        # 48 rows each, room in the last round
    ([600, 129, 1], 160, 300, "gelu", "64x128 / 128x128"),               # at most a quarter of a tile per CU
    ([600, 129, 1], 160, 300, "swiglu", "64x128 / 128x128"),
    ([900, 900, 127, 700], 544, 1300, "gelu", "128x128 / 128x128"),      # ... 5/8
    ([900, 900, 127, 700], 544, 640, "swiglu", "128x128 / 128x128"),
    ([900, 900, 127, 700], 544, 1300, "swiglu", "128x256 / 128x128"),    # h not a multiple of 64
    ([128] * 119 + [129], 288, 136, "gelu", "128x256 / 128x384"),
    ([3000, 2500, 1, 2499], 768, 640, "gelu", "pairs / 128x384"),
    ([1024] * 7 + [1000, 24], 1024, 256, "gelu", "128x128 / 128x384"),   # short K: wasted columns
    ([128] * 119 + [129], 256, 136, "gelu", "pairs / 128x256"),
    ([128] * 119 + [129], 256, 136, "swiglu", "pairs / 128x256"),
    # h not a multiple of 32: row-major weights
    ([600, 129, 1], 168, 300, "gelu", "64x128 / 128x128"),
    ([600, 129, 1], 168, 300, "swiglu", "64x128 / 128x128"),
    ([20] * 127 + [64], 200, 384, "gelu", "64x256 / 128x128"),
    ([20] * 127 + [64], 200, 200, "swiglu", "64x256 / 128x128"),
    ([900, 900, 127, 700], 520, 1300, "gelu", "128x128 / 128x128"),
    ([900, 900, 127, 700], 520, 640, "swiglu", "128x128 / 128x128"),
    ([128] * 119 + [129], 264, 136, "gelu", "128x256 / 128x384"),
    ([128] * 119 + [129], 264, 136, "swiglu", "128x256 / 128x384"),
]

# 256 x 256 tiles: (rows per expert, h, f, {act: tiles, up / down}, {act: the same beside so many
# empty experts that there are fewer than 192 rows per expert})
WIDE_FORMS = [
    ([33000], 72, 1536,                     # down-projection, N below one tile
     {"gelu": "128x256 / turns", "swiglu": "128x256 / turns"}, {"gelu": "128x256 / 128x256", "swiglu": "128x256 / 128x256"}),
    ([16200, 31, 800, 1], 264, 1600,        # N just over a tile; last row tiles of 72, 31, 32 and 1 rows
     {"gelu": "128x256 / turns", "swiglu": "128x256 / turns"}, {"gelu": "128x256 / 128x384", "swiglu": "128x256 / 128x384"}),
    ([256, 8192], 776, 1700,                # whole row tiles, N = 3 tiles and 8 columns
     {"gelu": "128x256 / turns", "swiglu": "128x256 / turns"}, {"gelu": "128x256 / 128x256", "swiglu": "128x256 / 128x256"}),
    ([1023], 3072, 12200,                   # up-projection (K = 3072: 0.84 rounds of tiles, SwiGLU 1.7)
     {"gelu": "turns / 128x128", "swiglu": "turns / 128x128"}, {"gelu": "pairs / 128x128", "swiglu": "pairs / 128x128"}),
    ([1500, 700], 1536, 16900,              # ... K = 1536, 5 rounds for SwiGLU
     {"gelu": "pairs / 128x128", "swiglu": "turns / 128x128"}, {"gelu": "pairs / 128x128", "swiglu": "pairs / 128x128"}),
]


def empty_beside(A, E):
    """Empty experts that bring A rows of E experts below 192 rows per expert."""
    return A // 192 + 1 - E


# the same for streamed weights: weight rows x blocks of 16 rows of a workgroup; "sums": the second
# product's fp32 sums go to the combine, in so many parts
STREAM_FORMS = [
    ([1], 8, 1, "gelu", "stream 16x1 / 16x1"),                      # one 16-byte chunk of K: most waves have none
    ([16, 0, 17, 1, 15], 200, 129, "gelu", "stream 16x1 / 16x1"),   # row-tile edges; K ends inside a step
    ([5] * 40, 136, 640, "gelu", "stream 64x1 / 32x1 sums 1"),
    ([64, 0], 1544, 300, "gelu", "stream 16x1 / 32x1"),
    ([300, 212], 64, 1000, "gelu", "stream 64x2 / 16x1 sums 1"),    # 512 rows: the most at any number of experts
    ([9] * 72, 32, 96, "gelu", "stream 32x1 / 16x1"),               # 648 rows: streamed for their number of experts
    # 32 rows each on average: three blocks, around their edges (47, 48, 49, more than two tiles)
    ([32, 48, 49, 16, 47, 0, 33, 31, 97, 10, 32, 30, 20, 40, 3, 24], 1104, 1100, "gelu", "stream 64x3 / 64x3 sums 1"),
    ([32, 48, 49, 16, 47, 0, 33, 31, 97, 10, 32, 30, 20, 40, 3, 24], 200, 700, "swiglu", "stream 64x3 / 32x1 sums 1"),
    ([9] * 72, 520, 1024, "gelu", "stream 64x2 / 64x2"),
]

# decode-sized calls on weights too large to stream: (experts, rows, h, f, act)
SUMS_FORMS = [
    (28, 504, 928, 900, "swiglu", "64x256 / 128x128 sums 1"),
]
