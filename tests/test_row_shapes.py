"""Launch shapes of the row movers, from the library's own header compiled for the host: no chunk of a row is left out or taken
twice, and a row's last few chunks go to its first lanes only at the widths where that was measured to be ahead (a chunk to sixteen
more than four, eight and sixteen waves).  No GPU needed."""
import os
import subprocess

import pytest

from paper_2605_22428_amd import build

PROGRAM = """
#include <cstdio>
#include "mw_internal.h"
int main()
{
    for (int n = 1; n <= 4200; ++n) {
        const mw_row_shape a = mw_row_shape_of(n), b = mw_row_shape_folded(n);
        printf("%d %d %d %d %d %d\\n", n, a.bs, a.nseg, b.bs, b.nseg, (int)mw_is_folded(b, n));
    }
}
"""


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    at = tmp_path_factory.mktemp("shapes")
    (at / "shapes.cpp").write_text(PROGRAM)
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-x", "c++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", build.CSRC,
                    "-I", os.path.join(build.ROOT, "include"), "-I", "/opt/rocm/include", str(at / "shapes.cpp"), "-o", str(at / "shapes")],
                   check=True)
    out = subprocess.run([str(at / "shapes")], check=True, stdout=subprocess.PIPE, text=True).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def test_every_chunk_has_one_lane(shapes):
    for n, bs, nseg, fbs, fnseg, folded in shapes:
        assert bs % 64 == 0 and 64 <= bs <= 1024 and (nseg - 1) * bs < n <= nseg * bs, n
        if folded:                                   # one workgroup, whose first lanes have a second chunk
            assert fnseg == 1 and fbs % 64 == 0 and fbs <= 1024 and fbs < n <= fbs + 16, n
        else:
            assert (fbs, fnseg) == (bs, nseg), n


def test_rows_are_folded_where_it_was_measured(shapes):
    want = {n for waves in (4, 8, 16) for n in range(64 * waves + 1, 64 * waves + 17)}
    want -= {n for n in want if n > 640 and n % 8 == 0}      # (cut into single waves)
    assert {s[0] for s in shapes if s[5]} == want
