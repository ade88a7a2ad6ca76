"""How many workgroups share the keys of a tree-attention call (csrc/attn_plan.h), on the CPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# lines of batch, query heads, kv heads, nodes, head dim, prefix length -> workgroups of a batch of equal units, of a ragged one, units, blocks a unit
DRIVER = r"""
#include <cstdio>
#include "attn_plan.h"
using namespace fspad_detail;
int main() {
  fspad_attn_desc d{};
  int L;
  while (std::scanf("%d %d %d %d %d %d", &d.batch, &d.n_q_heads, &d.n_kv_heads, &d.n_nodes_max, &d.head_dim, &L) == 6) {
    Plan pl{};
    plan_rows(d, pl);
    const int64_t units = (int64_t)d.batch * d.n_kv_heads * pl.GY, blocks = blocks_of(L, d.n_nodes_max);
    std::printf("%d %d %lld %lld\n", plan_wgs(pl, units * blocks, units, true, 0), plan_wgs(pl, units * blocks, units, false, 0), (long long)units, (long long)blocks);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    at = tmp_path_factory.mktemp("plan")
    (at / "plan.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "include"), "-I",
                    os.path.join(ROOT, "paper_2408_15562_amd", "csrc"), "-o", str(at / "plan"), str(at / "plan.cpp")], check=True)

    def run(shapes):
        text = "".join(" ".join(map(str, s)) + "\n" for s in shapes)
        out = subprocess.run([str(at / "plan")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return run


def test_equal_units_fill_the_chip(plan):
    """Two workgroups a compute unit for 16-row tiles that fill them evenly (draft steps of 8 x 16 heads, 10 nodes; 1 x 16 heads, 4 nodes, a long prefix), one
    for the other tilings; as many pieces of every unit as that gives; short units in sufficient number whole."""
    want = {(8, 16, 16, 10, 64, 1050): 512, (8, 16, 16, 10, 64, 1200): 512, (8, 16, 16, 10, 64, 1300): 512, (1, 16, 16, 4, 128, 8300): 512,
            (1, 32, 32, 26, 128, 2048): 256, (1, 32, 8, 60, 128, 4096): 256, (1, 64, 8, 60, 128, 16384): 256, (4, 52, 52, 60, 128, 4096): 208,
            (4, 32, 8, 60, 128, 330): 256, (4, 32, 8, 60, 128, 220): 64, (2, 12, 2, 1, 128, 5030): 80, (1, 40, 8, 64, 128, 6445): 240}
    assert {s: got[0] for s, got in zip(want, plan(want))} == want


def test_workgroups_over_the_range(plan):
    """At most as many workgroups as blocks and as 16-row tiles fill the chip with, or one for each whole unit; an equal batch in two or more pieces a unit has
    two blocks for every key-splitting wavefront of a piece."""
    heads = [(8, 8), (16, 16), (32, 32), (52, 52), (4, 4), (12, 2), (28, 4), (32, 8), (64, 8), (8, 1)]
    shapes = [(B, q, kv, N, D, L) for B in (1, 2, 5, 16, 128) for q, kv in heads for N in (1, 4, 17, 26, 60, 64) for D in (64, 128)
              for L in (0, 1, 31, 97, 330, 1040, 2048, 5000, 16384, 60000)]
    for shape, (equal, ragged, units, blocks) in zip(shapes, plan(shapes)):
        for wgs in (equal, ragged):
            assert 1 <= wgs <= units * blocks and (wgs <= 512 or wgs == units), shape
        if equal > units and equal % units == 0:
            assert blocks * units >= 2 * equal, shape
