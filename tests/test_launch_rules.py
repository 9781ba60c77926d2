"""The rules that choose a launch's form (csrc/launch_rules.h), on the host: where a form was measured to be the slower one, its
rule does not take it, and what it takes is within the bounds that the launch relies on."""
import os
import random
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2304_01089_amd", "csrc")
PROGRAM = r"""
#include <iostream>
#include <string>
#include "launch_rules.h"
int main() {
  std::string what;
  while (std::cin >> what) {
    long long v[6];
    for (auto& x : v) std::cin >> x;
    if (what == "tail") std::cout << rptq::gemm_tail_columns(v[0], v[1], static_cast<int>(v[2] / 32), static_cast<int>(v[3]), v[4] != 0) << "\n";
    else std::cout << rptq::ln_rows_per_workgroup(v[0], static_cast<int>(v[1]), static_cast<int>(v[2]), static_cast<int>(v[3]), static_cast<int>(v[4]), v[5] != 0) << "\n";
  }
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    at = tmp_path_factory.mktemp("rules")
    (at / "rules.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(at / "rules.cpp"), "-o", str(at / "rules")], check=True)

    def ask(what, queries):
        text = "".join("%s %s\n" % (what, " ".join(str(int(v)) for v in (*q, 0)[:6])) for q in queries)
        return [int(v) for v in subprocess.run([str(at / "rules")], input=text, capture_output=True, text=True, check=True).stdout.split()]
    return ask


@pytest.mark.parametrize("M,N", [(2048, 4608), (1024, 9216), (2048, 5120), (2100, 4500), (1600, 5376), (3072, 3072), (8190, 1248)])
def test_second_round_of_products_stays_on_small_tiles(rule, M, N):
    """513 to 704 tiles of 64 x 256 (here with at most 128 beyond 512): 64 x 128 tiles throughout were ahead of large tiles with
    small ones behind (up to 17 % at K = 768, 3 to 10 at 2048), except for 8-bit codes from K = 5120 on."""
    queries = [(M, N, K, bits, cw) for K in (768, 2048, 3008, 5120, 12288) for bits in (3, 4, 8) for cw in (0, 1)]
    for (_, _, K, bits, cw), cols in zip(queries, rule("tail", queries)):
        assert (cols > 0) == (bits == 8 and K >= 5120 and not cw), (K, bits, cw)


def test_last_columns_are_the_few_beyond_a_whole_number(rule):
    """What the launch relies on: some columns of large tiles stay, and the small ones are one per compute unit at most."""
    rng = random.Random(5)
    queries = [(2048, 8704, 5120, 4, 0), (2100, 8000, 768, 3, 1), (2900, 4099, 2048, 8, 0), (4096, 20992, 5120, 4, 0), (2048, 6144, 5120, 4, 0)]
    queries += [(rng.randint(1, 20000), rng.randint(1, 60000), rng.choice([256, 5120]), rng.choice([3, 4, 8]), rng.randint(0, 1)) for _ in range(20000)]
    got = rule("tail", queries)
    assert got[:5] == [2, 1, 1, 2, 0]
    taken = [(-(-M // 64), -(-N // 256), c) for (M, N, _, _, _), c in zip(queries, got) if c]
    assert len(taken) > 1000
    for rows, cols, c in taken:
        over = rows * cols % 256
        assert 0 < over <= c * rows <= 128 and (c - 1) * rows < over and c < cols


def test_rows_of_a_workgroup_where_one_form_was_ahead(rule):
    """Rows, waves of a row and units of a thread on 256 compute units: one row was behind two by 2 to 15 % (the first lines), two
    behind four or one by 2 to 9 % (the next), one ahead by 8 to 27 % (the last)."""
    two = [(1500, 2, 1, 8, 0), (2000, 2, 1, 4, 0), (2500, 2, 1, 8, 0), (1500, 2, 1, 3, 0), (300, 8, 1, 4, 0), (500, 8, 1, 8, 0), (300, 7, 1, 8, 0),
           (512, 6, 1, 3, 0), (400, 7, 1, 3, 0), (300, 8, 1, 3, 0), (2500, 2, 1, 4, 1), (400, 8, 2, 4, 1), (512, 8, 2, 8, 1), (1500, 8, 1, 4, 0)]
    four = [(600, 8, 2, 8, 1), (800, 8, 2, 4, 1), (600, 6, 1, 3, 1), (1000, 6, 1, 3, 1), (800, 7, 1, 3, 1), (700, 8, 1, 3, 1), (600, 5, 1, 3, 1), (1750, 7, 1, 4, 1)]
    one = [(900, 7, 1, 4, 1), (2816, 2, 1, 4, 1), (1000, 2, 1, 8, 1), (1280, 3, 1, 4, 1), (1200, 5, 1, 4, 1), (1000, 2, 1, 4, 0), (700, 8, 2, 4, 0), (600, 7, 1, 3, 0)]
    for rows, points in ((2, two), (4, four), (1, one)):
        queries = [(M, waves, units, 256, bits, ln) for M, waves, units, bits, ln in points]
        assert [(q, r) for q, r in zip(queries, rule("ln", queries)) if r != rows] == []


def test_rows_of_a_workgroup_fit_its_waves(rule):
    queries = [(M, waves, units, cus, bits, ln) for M in (1, 2, 255, 256, 257, 512, 513, 700, 1024, 1025, 3000, 20000, 2 ** 40) for waves in range(1, 16)
               for units in (1, 2) for cus in (32, 256, 304) for bits in (3, 4, 8) for ln in (0, 1)]
    for q, r in zip(queries, rule("ln", queries)):
        assert r in (1, 2, 4) and r <= q[1], q
