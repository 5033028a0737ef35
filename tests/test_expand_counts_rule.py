"""Which batches' (expert, peer) counts the expander adds up by itself, from the library's own header compiled for the host.  No GPU needed."""
import os
import subprocess

import pytest

import bench
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


def test_the_bench_names_the_kernel_that_is_launched(rule):
    """Row shapes and hits a row as the library derives them, for the configurations of the bench line and around the rule's sides."""
    for L, P, E, K, chunks, folded in ((4, 64, 256, 8, 896, 0), (4, 64, 256, 8, 462, 0), (1, 256, 256, 8, 896, 0), (2, 8, 16, 2, 32, 0), (1, 256, 256, 8, 264, 1),
                                       (16, 16, 256, 8, 264, 1), (6, 64, 384, 8, 462, 0), (8, 128, 1024, 8, 64, 0), (1, 64, 64, 8, 528, 1), (0, 8, 16, 2, 32, 0)):
        share = L / E
        hits = K * share / (1 - (1 - share) ** K) if L else 1.0
        for mib in (1, 127, 129, 191, 193, 287, 289, 447, 449, 719, 721, 4000):
            rows = (mib << 20) // (16 * chunks)
            want = "k_expand_counts" if rule(L, P, 0, folded, hits, rows * 16 * chunks) else "k_expand"
            assert bench.unpack_expander(L, P, E, K, rows, 16 * chunks) == want, (L, P, chunks, mib)
