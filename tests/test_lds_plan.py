"""Rows the general path stages: static and dynamic LDS together stay within
what a workgroup may hold, on the device's 160 KiB and on the 64 KiB that every
launch may use, and on the former the plan is the tuned one."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
MAX_Q = 14654

PROGRAM = r"""
#include "tga_internal.h"
#include <cstdio>
int main() {
    for (size_t total : {(size_t)163840, (size_t)65536, (size_t)16384})
        for (int halo : {2, 4})
            for (int np1 = 2; np1 <= 14654; ++np1) {
                const int rows = tga::general_rows(np1, halo, total);
                std::printf("%zu %d %d %d %zu\n", total, halo, np1, rows, tga::general_rows_lds(np1, halo, rows));
            }
    std::printf("queues %zu words %zu\n", tga::kGenQueueBytes, tga::kStaticWordsBytes);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           "-I" + os.path.join(ROOT, "paper_2506_17357_amd", "csrc"), str(src), "-o", str(exe)])
    lines = subprocess.check_output([str(exe)], text=True).split("\n")
    words = lines[-2].split()
    rows = [tuple(map(int, x.split())) for x in lines[:-2]]
    return rows, int(words[1]), int(words[3])


def test_rows_fit(plan):
    rows, queues, words = plan
    assert len(rows) == 3 * 2 * (MAX_Q - 1)
    for total, halo, np1, n, lds in rows:
        assert lds == (n + halo) * 2 * ((np1 + 7) // 8 * 8)
        if n:
            assert 1 <= n <= 24 and lds + queues + words <= total, (total, halo, np1, n)
        else:  # not even one row and its halo
            assert (1 + halo) * 2 * ((np1 + 7) // 8 * 8) + queues + words > total, (total, halo, np1)


def test_rows_on_the_device(plan):
    """The whole LDS of a compute unit: 24 rows, fewer where 56 KiB do not hold them, one where that is too much."""
    for total, halo, np1, n, lds in plan[0]:
        if total == 163840 and n:
            assert n == 24 or n == 1 or lds <= 57344
            assert n == 24 or (n + 1 + halo) * 2 * ((np1 + 7) // 8 * 8) > 57344
