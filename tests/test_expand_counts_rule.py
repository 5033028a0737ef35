"""Which batches' (expert, peer) counts the expander adds up by itself, from the library's own header compiled for the host.  No GPU needed."""
import os
import subprocess

import pytest

from paper_2605_22428_amd import build

PROGRAM = """
#include <cstdio>
#include "mw_internal.h"
int main()
{
    long long n, bytes;
    while (scanf("%lld %lld", &n, &bytes) == 2) printf("%d\\n", (int)mw_counts_by_expander(n, bytes));
}
"""
MB = 1 << 20


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    at = tmp_path_factory.mktemp("rule")
    (at / "rule.cpp").write_text(PROGRAM)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "c++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", build.CSRC,
                    "-I", os.path.join(build.ROOT, "include"), "-I", "/opt/rocm/include", str(at / "rule.cpp"), "-o", str(at / "rule")],
                   check=True)

    def run(*args):
        out = subprocess.run([str(at / "rule")], input="%d %d" % args, check=True, stdout=subprocess.PIPE, text=True).stdout
        return bool(int(out))
    return run


def test_a_rank_without_experts_has_no_counts_to_add_up(rule):
    assert not rule(0, 0) and not rule(0, 1000 * MB)


def test_most_counts(rule):
    assert rule(1, MB) and rule(256, MB) and rule(512, MB) and not rule(513, MB) and not rule(1 << 22, 0)
    assert rule(257, 128 * MB) and not rule(257, 128 * MB + 1)
