"""Order and groups of a batch's instances (csrc/mc_plan.h, compiled by g++):
every tile of a group is found in its own instance by the search that the
kernels make, wherever instances with launches of their own lie in size."""

import os
import subprocess

import numpy as np
import pytest

from tests.conftest import ROOT

MAIN = r"""
#include <cstdio>
#include "mc_plan.h"
int main() {
    int n;
    while (scanf("%d", &n) == 1) {
        std::vector<mc::PlanItem> items(n);
        for (auto &t : items) {
            int own;
            long long dim;
            if (scanf("%d %d %lld %d", &t.M, &t.kind, &dim, &own) != 4) return 1;
            t.dim = dim, t.tiles = (dim + 63) / 64, t.own = own != 0;
        }
        std::vector<int32_t> sorted;
        std::vector<int64_t> prefix;
        const auto groups = mc::plan_groups(items, sorted, prefix);
        for (int s : sorted) printf("%d ", s);
        printf("|");
        for (long long p : prefix) printf("%lld ", p);
        printf("|");
        for (const auto &g : groups)
            printf("%d %d %d %d %lld ", g.M, g.kind, g.first, g.count, (long long)g.tiles);
        printf("\n");
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.cpp").write_text(MAIN)
    exe = str(d / "plan")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I",
                           os.path.join(ROOT, "paper_2005_13679_amd", "csrc"),
                           str(d / "plan.cpp"), "-o", exe])
    return exe


def instance_of(item, first, count, prefix):
    j = 0
    while j + 1 < count and prefix[first + j + 1] <= item:
        j += 1
    return j


def check(batch, line):
    parts = [[int(x) for x in p.split()] for p in line.split("|")]
    order, prefix = parts[0], parts[1]
    groups = [parts[2][i:i + 5] for i in range(0, len(parts[2]), 5)]
    assert sorted(order) == list(range(len(batch)))
    assert len({(g[0], g[1]) for g in groups}) == len(groups)
    seen = set()
    for M, kind, first, count, tiles in groups:
        at = 0
        for j in range(count):
            i = order[first + j]
            m, k, dim, own = batch[i]
            assert (m, k, own) == (M, kind, 0) and i not in seen
            seen.add(i)
            last = at + (dim + 63) // 64 - 1
            for item in (at, (at + last) // 2, last):
                assert instance_of(item, first, count, prefix) == j, (batch, item)
            assert prefix[first + j] == at
            at = last + 1
        assert at == tiles
    assert seen == {i for i, t in enumerate(batch) if not t[3]}


def test_groups_are_consecutive(program):
    batches = [[(5, 5, 156340626, 0), (5, 5, 4598126, 1), (5, 5, 82251, 0)],
               [(8, 5, 346104, 0), (8, 5, 154143080, 0), (8, 5, 10295472, 1)], [(3, 4, 45, 0)],
               [(6, 5, 300000, 1)]]
    rng = np.random.default_rng(0)
    for _ in range(400):
        n = int(rng.integers(1, 24))
        batches.append([(int(rng.integers(1, 9)), int(rng.integers(0, 6)),
                         int(2.0 ** rng.uniform(0, 28)), int(rng.random() < 0.4))
                        for _ in range(n)])
    text = "\n".join(f"{len(b)} " + " ".join(f"{m} {k} {d} {o}" for m, k, d, o in b)
                     for b in batches)
    out = subprocess.run([program], input=text, capture_output=True, text=True, check=True)
    lines = out.stdout.strip().split("\n")
    assert len(lines) == len(batches)
    for b, line in zip(batches, lines):
        check(b, line)
