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
    long long n_local, n_peers, bytes;
    int packets, folded;
    double hits;
    while (scanf("%lld %lld %d %d %lf %lld", &n_local, &n_peers, &packets, &folded, &hits, &bytes) == 6)
        printf("%d\\n", (int)mw_counts_by_expander(n_local, n_peers, packets != 0, folded != 0, hits, bytes));
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
        out = subprocess.run([str(at / "rule")], input="%d %d %d %d %f %d" % args, check=True, stdout=subprocess.PIPE, text=True).stdout
        return bool(int(out))
    return run


def test_a_rank_without_experts_has_no_counts_to_add_up(rule):
    for folded in (0, 1):
        assert not rule(0, 256, 0, folded, 1.0, 0) and not rule(0, 1, 1, folded, 1.0, 1000 * MB)


@pytest.mark.parametrize("packets", [0, 1])
@pytest.mark.parametrize("L,P,folded,hits,most", [(1, 1, 0, 1.0, 720), (1, 256, 0, 1.0, 720), (32, 8, 0, 1.5, 720), (1, 256, 1, 1.0, 288), (4, 64, 1, 1.19, 192),
                                                  (1, 2, 1, 1.0, 161), (16, 16, 1, 1.2, 448), (257, 1, 0, 2.0, 128), (8, 64, 1, 1.0, 128)])
def test_most_bytes(rule, L, P, packets, folded, hits, most):
    """What adding up costs grows with the payload, what it saves with the peers (measured; the figures stand beside the rule)."""
    if packets and folded and hits < 1.2 and L * P <= 256:
        most -= 56
    assert rule(L, P, packets, folded, hits, 0) and rule(L, P, packets, folded, hits, most * MB)
    assert not rule(L, P, packets, folded, hits, most * MB + 1)


def test_most_counts(rule):
    for folded in (0, 1):
        assert rule(2, 256, 0, folded, 1.0, MB) and not rule(513, 1, 0, folded, 1.0, MB) and not rule(1 << 14, 256, 0, folded, 2.0, 0)
