"""Grouping of classes into launches (group_add of csrc/jk_common.h), on the
host: every unit of every class is in exactly one launch, found by the kernels'
search, and no launch exceeds 2^32 - 1 work-items."""
import os
import shutil
import subprocess

import pytest

from paper_2507_09772_amd import build_lib

PROGRAM = r"""
#include "jk_common.h"
#include <cstdio>
#include <vector>
using namespace jk;
struct Part { int cls; int64_t lo, hi; };
// the kernels' search for the class of unit g, and its unit there
static int find(const ClsGroup &grp, int &g) {
    int lo = 0, hi = grp.n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (grp.base[mid] <= g) lo = mid;
        else hi = mid - 1;
    }
    g -= grp.base[lo];
    return grp.desc[lo];
}
static int check(const std::vector<int64_t> &units, int lanes, int per) {
    const int64_t max = launch_units_max(lanes, per);
    std::vector<ClsGroup> launches;
    for (size_t c = 0; c < units.size(); ++c) {
        size_t k = 0;
        for (int64_t from = 0; from < units[c]; ++k) {
            if (k == launches.size()) launches.push_back(ClsGroup{});
            group_add(launches[k], (int)c, units[c], max, &from);
            if (k > units.size() + 1000) return 1;
        }
    }
    std::vector<int64_t> next(units.size(), 0);
    for (const ClsGroup &g : launches) {
        const int64_t n = g.base[g.n];
        if (g.n < 1 || g.n > GROUP_MAX || n < 1 || (n + per - 1) / per * lanes >= (int64_t)1 << 32) return 2;
        // the first and last unit of every part, and the one between parts
        int64_t at = 0;
        for (int k = 0; k < g.n; ++k) {
            const int64_t end = g.base[k + 1];
            int a = (int)at, b = (int)(end - 1);
            if (find(g, a) != g.desc[k] || find(g, b) != g.desc[k]) return 3;
            if (a != next[g.desc[k]] || b - a != end - 1 - at) return 4;
            next[g.desc[k]] = b + 1;
            at = end;
        }
        if (at != n) return 5;
    }
    for (size_t c = 0; c < units.size(); ++c)
        if (next[c] != units[c]) return 6;
    std::printf("%zu classes %zu launches\n", units.size(), launches.size());
    return 0;
}
int main() {
    const int lanes[][2] = {{256, 1}, {64, 1}, {256, 4}, {128, 1}};
    for (auto &l : lanes) {
        const int64_t m = launch_units_max(l[0], l[1]);
        const std::vector<std::vector<int64_t>> cases = {
            {1}, {5, 1, 7}, std::vector<int64_t>(200, 3), {m}, {m, 1}, {m - 1, 1, 1}, {m + 1}, {3 * m + 5, 10},
            {10, m + 1, 20}, {m / 2, m / 2, m / 2, m / 2}, std::vector<int64_t>(40, m / 3 + 1), {INT32_MAX}};
        for (auto &c : cases)
            if (int rc = check(c, l[0], l[1])) { std::printf("lanes %d: %d\n", l[0], rc); return 1; }
    }
    return 0;
}
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="no g++")
def test_launches_hold_every_unit(tmp_path):
    src, exe = tmp_path / "g.cpp", tmp_path / "g"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", build_lib.CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
