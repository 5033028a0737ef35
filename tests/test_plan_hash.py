"""The hash by which the plan of 2049 to 8192 tokens finds equal keys, from the library's own header compiled for the host.  A token
whose key shares its bit with another key takes the slow way through a table; keys with the same hash also probe the same slots.
Destination sets are far from random bits -- three to eight ranks of a few dozen -- and must spread nearly like random ones.  (Of two
ranks there are so few that most tokens have their key in common anyway.)  No GPU needed."""
import os
import subprocess

import numpy as np
import pytest

from paper_2605_22428_amd import build

PROGRAM = """
#include <cstdio>
#include "mw_internal.h"
int main()
{
    unsigned long long k;
    while (scanf("%llu", &k) == 1) printf("%u\\n", mw_key_hash((uint32_t)k, (uint32_t)(k >> 32)));
}
"""


@pytest.fixture(scope="module")
def hash_of(tmp_path_factory):
    at = tmp_path_factory.mktemp("hash")
    (at / "hash.cpp").write_text(PROGRAM)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "c++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", build.CSRC,
                    "-I", os.path.join(build.ROOT, "include"), "-I", "/opt/rocm/include", str(at / "hash.cpp"), "-o", str(at / "hash")],
                   check=True)

    def run(keys):
        out = subprocess.run([str(at / "hash")], input="\n".join(map(str, keys)), check=True, stdout=subprocess.PIPE, text=True).stdout
        return np.array(out.split(), dtype=np.int64)
    return run


def _keys(R, n_ranks, n, rng):
    """Distinct keys of `n` tokens that name `n_ranks` of R ranks each: the bitmap, or beyond 64 ranks the ranks highest first, a byte each."""
    ranks = np.sort(np.argsort(rng.random((n, R)), axis=1)[:, :n_ranks], axis=1)[:, ::-1]
    if R <= 64:
        return sorted({sum(1 << int(r) for r in row) for row in ranks})
    keys = set()
    for row in ranks:
        k = 0
        for b in [int(row[0])] + [int(r) + 1 for r in row[1:]] + [0] * (8 - n_ranks):
            k = k << 8 | b
        keys.add(k)
    return sorted(keys)


@pytest.mark.parametrize("R,n_ranks", [(64, 3), (64, 4), (64, 5), (64, 8), (48, 4), (40, 3), (33, 3), (32, 4), (24, 4), (72, 3), (128, 4), (256, 3),
                                       (256, 8)])
def test_few_keys_share_a_bit_or_a_hash(hash_of, R, n_ranks):
    keys = _keys(R, n_ranks, 8192, np.random.default_rng(R + n_ranks))
    h = hash_of(keys)
    bit = (h >> (32 - 13)) * 32 + ((h >> 12) & 31)           # 2^13 slots of 32 bits: n random keys leave n^2 / 2^18 of them sharing
    shared = int((np.bincount(bit, minlength=1 << 18)[bit] > 1).sum())
    assert shared <= max(64, 4 * len(keys) ** 2 >> 18), (shared, len(keys))
    assert np.unique(h, return_counts=True)[1].max() <= 6
