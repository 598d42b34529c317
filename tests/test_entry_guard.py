"""No C++ exception leaves the entry points (csrc/jk_guard.h): host memory that
runs out inside one becomes its status."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2507_09772_amd import build_lib

PROGRAM = r"""
#include "jk_guard.h"
#include <new>
#include <vector>
int main() {
    auto oom = [] { return -3; };
    volatile long long n = -1;
    if (guarded([] { return 7; }, oom) != 7) return 1;
    if (guarded([]() -> int { throw std::bad_alloc(); }, oom) != -3) return 2;
    if (guarded([&] { std::vector<double> v; v.resize((size_t)n); return (int)v.size(); }, oom) != -3) return 3;
    return 0;
}
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="no g++")
def test_exceptions_become_a_status(tmp_path):
    src, exe = tmp_path / "g.cpp", tmp_path / "g"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", build_lib.CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0


@pytest.mark.parametrize("name,unit", [("jk_plan_create", "jk_api"), ("jk_execute", "jk_api"), ("jk_plan_profile", "jk_api"),
                                       ("jk_plan_stats", "jk_api"), ("jk_eri_block", "jk_api"),
                                       ("jk_execute_noalloc", "jk_noalloc"), ("jk_batch_create", "jk_batch"),
                                       ("jk_batch_execute", "jk_batch"), ("jk_batch_stats", "jk_batch")])
def test_entry_points_that_allocate_are_guarded(name, unit):
    text = open(os.path.join(build_lib.CSRC, unit + ".hip")).read()
    assert re.search(r'extern "C" int %s\([^{]*\{\s*return entry\(' % name, text)
