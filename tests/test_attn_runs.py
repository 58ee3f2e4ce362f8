"""The attention planner's run lengths (csrc/attn_runs.hpp), compiled with the host compiler.

Where a forward's pages spread evenly, its workgroups fit one round; where they cannot (one long
request among many short ones, few work items per head), no run is much longer than a wave's even
share of the pages, and never shorter than the caller's base."""
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_31580_amd", "csrc")
MAIN = """
#include <cstdio>
#include <vector>
#include "attn_runs.hpp"
int main() {
  int n, heads, resident, base;
  while (std::scanf("%d %d %d %d", &n, &heads, &resident, &base) == 4) {
    std::vector<laser::RunGroup> g(n);
    for (auto& x : g) std::scanf("%d %d", &x.pages, &x.tiles);
    std::printf("%d\\n", laser::run_pages(g.data(), n, heads, 4, resident, base));
  }
}
"""


@pytest.fixture(scope="module")
def run_pages(tmp_path_factory):
    d = tmp_path_factory.mktemp("runs")
    (d / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-std=c++17", "-Wall", "-Werror", f"-I{CSRC}", "-o", str(d / "runs"), str(d / "main.cpp")], check=True)

    def call(groups, heads, resident=512, base=4):
        line = f"{len(groups)} {heads} {resident} {base} " + " ".join(f"{p} {t}" for p, t in groups)
        return int(subprocess.run([str(d / "runs")], input=line, capture_output=True, text=True, check=True).stdout)

    return call


def _items(groups, b):
    return sum(-(-p // (4 * b)) * t for p, t in groups)


def _share(groups, heads, resident):
    return sum(p * t for p, t in groups) * heads / (4 * resident)


@pytest.mark.parametrize("groups,heads,resident", [
    ([(188, 1)] * 7 + [(875, 1)], 8, 512),
    ([(188 + 98 * i, 1) for i in range(8)], 8, 512),     # batch 8, 3,000 to 14,000 positions
    ([(188 + 98 * i, 1) for i in range(4)], 4, 512),
    ([(126, 1)] * 64, 8, 512),
    ([(188, 1)] * 24, 16, 512),
    ([(566, 5)], 8, 512),                                # a prompt chunk: five pairs of query tiles
    ([(300, 2), (300, 1), (700, 2), (700, 1)], 8, 512),
    ([(188 + 98 * i, 1) for i in range(8)], 8, 768),
])
def test_even_batches_fit_one_round(run_pages, groups, heads, resident):
    b = run_pages(groups, heads, resident)
    assert _items(groups, b) * heads <= resident
    assert b == 4 or _items(groups, b - 1) * heads > resident, "longer than one round needs"
    assert b <= 2 * _share(groups, heads, resident) + 1


@pytest.mark.parametrize("groups,heads", [
    ([(7, 1)] * 63 + [(875, 1)], 8),    # one long request among one-page-per-wave ones that fill the round
    ([(63, 1)] * 63 + [(875, 1)], 8),
    ([(7, 1)] * 15 + [(875, 1)], 32),
    ([(32, 1)] * 31 + [(875, 1)], 32),
    ([(7, 1)] * 3 + [(875, 1)], 32),    # reachable, with 16 items on 8 XCDs
    ([(188 + 98 * i, 1) for i in range(8)], 32),
    ([(1, 1)] * 63 + [(4096, 1)], 32),
])
def test_uneven_batches_keep_short_runs(run_pages, groups, heads):
    b = run_pages(groups, heads)
    assert 4 <= b <= 8 and b <= max(4, _share(groups, heads, 512))


def test_alike_groups_past_one_round(run_pages):
    # more groups than one round holds, all alike: each is one workgroup; not so when they differ
    assert run_pages([(188, 1)] * 24, 32) == 47
    assert run_pages([(126, 1)] * 63 + [(127, 1)], 32) == 32
    assert run_pages([(8 + 6 * i, 1) for i in range(40)], 32) == 8
    assert run_pages([(1100, 1)] * 64, 32) == 8  # runs past the longest


@pytest.mark.parametrize("groups,b", [
    ([(500, 1)] * 16, 125),                              # two items on every XCD, all alike
    ([(188, 1)] * 24, 47),
    ([(875, 1)] * 24, 219),
    ([(500, 1)] * 8, 42),                                # three of each group
    ([(500, 1)] * 5, 8),                                 # 20 items: three on half of the XCDs, two on the others
    ([(500, 1)] * 17, 8),
    ([(7 + 16 * i, 1) for i in range(16)], 8),           # 24 items of several lengths
    ([(63 + 54 * i, 1) for i in range(16)], 8),
    ([(7 + 10 * i, 1) for i in range(24)], 8),
])
def test_few_items_are_one_round_where_the_xcds_are_even(run_pages, groups, b):
    # 32 KV heads, three workgroups per CU: at most 24 items per head are resident
    assert run_pages(groups, 32, 768) == b


def test_base_is_kept_where_it_fits(run_pages):
    for base in (1, 2, 3, 4):
        assert run_pages([(13, 1)], 2, 512, base) == base
        assert run_pages([(100, 1)] * 16, 4, 512, base) >= base
