"""Which launches store their rows streaming only and which write them through, from the library's own header compiled for the host:
rows of whole cache lines are always written through, others where that was measured to be no slower.  No GPU needed."""
import os
import subprocess

import pytest

from paper_2605_22428_amd import build

PROGRAM = """
#include <cstdio>
#include "mw_internal.h"
int main()
{
    long long stride, rows;
    while (scanf("%lld %lld", &stride, &rows) == 2)
        printf("%d%d%d%d%d%d\\n", (int)mw_rows_part(stride, rows), (int)mw_step_rows_part(stride),
               (int)mw_relay_rows_part(stride, rows, false, false), (int)mw_relay_rows_part(stride, rows, false, true),
               (int)mw_relay_rows_part(stride, rows, true, false), (int)mw_relay_rows_part(stride, rows, true, true));
}
"""
#       bytes from row to row, rows: pack, step, relay, relay beside an index, packets, packets beside an index
CASES = [((14336, 4096), "000000"), ((128, 1), "000000"), ((128, 65536), "000000"),
         ((272, 7000), "100011"), ((272, 8192), "001111"), ((1200, 1700), "110011"), ((1200, 1800), "011111"), ((1200, 15700), "011111"),
         ((1200, 15800), "111111"), ((2544, 4096), "011111"), ((2576, 4096), "111111"), ((7392, 100), "110011"), ((7392, 4096), "111111"),
         ((2112, 100), "110111"), ((2112, 4096), "010111"), ((4032, 4096), "110111"), ((4160, 4096), "110000"), ((14400, 8000), "110000")]


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    at = tmp_path_factory.mktemp("stores")
    (at / "rule.cpp").write_text(PROGRAM)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "c++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", build.CSRC,
                    "-I", os.path.join(build.ROOT, "include"), "-I", "/opt/rocm/include", str(at / "rule.cpp"), "-o", str(at / "rule")],
                   check=True)

    def run(cases):
        return subprocess.run([str(at / "rule")], input="\n".join("%d %d" % c for c in cases), check=True, stdout=subprocess.PIPE, text=True).stdout.split()
    return run


def test_stores_by_size(rule):
    assert rule([c for c, _ in CASES]) == [want for _, want in CASES]


def test_whole_lines_are_written_through(rule):
    assert set(rule([(128 * n, rows) for n in (1, 3, 8, 58, 112, 512) for rows in (1, 64, 4096, 65536)])) == {"000000"}
