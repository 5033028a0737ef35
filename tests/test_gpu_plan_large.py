"""GPU parity of mw_plan where its arrays in the workspace begin to be needed: the last batch without sorted chunks and the
first with them, the last without row-indexed arrays and the first with them, in contexts that are not a token
larger; keys of one word, of bytes, and bitmaps without a key.  Against the oracle, bit-exact."""
import numpy as np
import pytest

from oracle import ref
from paper_2605_22428_amd import binding as B

import gpu_harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [8192, 8193, 24575, 24576])
@pytest.mark.parametrize("R,E,K", [(8, 16, 2), (130, 260, 8), (130, 260, 9)])
def test_plan_at_the_edges_of_its_arrays(R, E, K, T):
    print("plan", R, E, K, T, flush=True)
    rng = np.random.default_rng(T + K)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    ctx = B.Context(R, E, K, 0, 8, B.MW_ROW_BF16, T, 1, e2r, device=H.DEV)
    tk = rng.integers(0, E, size=(T, K)).astype(np.int32)
    tk[rng.random(T) < 0.05] = -1
    buf = B.SendBuffers(ctx, T)
    ctx.mw_plan(H.dev(tk), buf.mask, buf.perm, buf.desc, buf.stats)
    st = ctx.mw_get_send_stats(buf.stats)
    mask, perm, desc, want = ref.plan(tk, e2r, R, 16)
    assert (int(st["n_rows"]), int(st["n_groups"]), int(st["error_flags"])) == (len(perm), len(desc), 0)
    H.assert_same_bytes(st["rows_per_dest"], want["rows_per_dest"], "rows_per_dest")
    H.assert_same_bytes(H.host(buf.mask).view(np.uint64)[:T], mask, "mask")
    H.assert_same_bytes(H.host(buf.perm)[: len(perm)], perm, "perm")
    H.assert_same_bytes(H.host(buf.desc).reshape(-1).view(B.DESC_DTYPE)[: len(desc)].view(np.uint8), desc.view(np.uint8), "desc")
