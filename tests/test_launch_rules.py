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
    long long v[5];
    for (auto& x : v) std::cin >> x;
    if (what == "tail") std::cout << rptq::gemm_tail_columns(v[0], v[1], static_cast<int>(v[2] / 32), static_cast<int>(v[3]), v[4] != 0) << "\n";
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
        text = "".join("%s %s\n" % (what, " ".join(str(int(v)) for v in q)) for q in queries)
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
