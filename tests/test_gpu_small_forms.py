"""GPU parity of the small launches (mw_plan_pack, the small stream step and the one-workgroup index) where
their form changes: lanes a token (64 and 128 tokens), rows longer than a workgroup's lanes, the expert
table in LDS (up to 1024 experts, and where the index's LDS has room) and in memory.  Bit-exact."""
import numpy as np
import pytest

from oracle import ref
from paper_2605_22428_amd import workloads as W

import gpu_harness as H
import test_gpu_fused as fused
import test_gpu_small_step as small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("E,R,R2", [(1023, 33, 93), (1024, 64, 128), (1025, 41, 205), (2050, 50, 205)])
@pytest.mark.parametrize("T", [1, 64, 65, 128, 129, 256])
def test_plan_pack_forms(T, E, R, R2):
    hidden = {1: 4096, 64: 4104, 65: 8192}.get(T, 1024)          # 512, 513, 1024, 128 chunks a row
    fused._one(W.DispatchWorkload("f1", 71, R, E, 8, T, hidden, "bf16", "uniform"), T, 7)
    fused._one(W.DispatchWorkload("f3", 72, R2, E, 5, T, 512 * (1 + T % 2), "fp8", "uniform"), T, 92)


# peers, experts, top_k, tokens: table in LDS at its largest; one more; LDS too full for it (64 local
# experts x 15 peers x 5 words, twice); one peer's record in each of the four scanned waves' ends
STEPS = {"e1024": (16, 1024, 8, 60), "e1025": (41, 1025, 8, 33), "full": (15, 960, 8, 160), "p64": (64, 640, 3, 20),
         "p65": (65, 650, 8, 20), "p256": (256, 512, 4, 9)}


@pytest.mark.parametrize("which", sorted(STEPS))
def test_small_step_forms(which, monkeypatch):
    R, E, K, T = STEPS[which]
    w = W.DispatchWorkload(which, 73, R, E, K, T, 256, "bf16", "uniform")
    monkeypatch.setitem(small.SHAPES, which, (w, R - 1, None))
    small.test_small_stream_steps_match_the_oracle(which)


@pytest.mark.parametrize("E,K", [(16, 4), (16, 16), (1040, 12)])
def test_more_rows_than_the_last_batch(E, K):
    """The one-workgroup index keeps as many rows a lane as the last batch had; a batch of up to 2000 rows after
    one of a few: the further ones go through memory, with more than eight hits a row too."""
    R, T, hidden, my_rank = 8, 250, 64, 5
    w = W.DispatchWorkload("more", 74, R, E, K, T, hidden, "bf16", "uniform")
    e2r = W.expert_to_rank(w)
    ctx = H.make_ctx(w, my_rank)
    mine = np.nonzero(e2r == my_rank)[0]
    rng = np.random.default_rng(E + K)
    for n in (3, 60, T, 100):
        toks, recs = [], []
        for p in range(R):
            tk = np.argsort(rng.random((n, E)), axis=1)[:, :K].astype(np.int32)
            tk[np.arange(n), rng.integers(0, K, n)] = rng.choice(mine, n)
            x = rng.integers(0, 1 << 16, size=(n, hidden), dtype=np.uint16)
            toks.append((tk, x, None))
            recs.append(H.shrink(H.GpuSend(ctx, tk, x, None).deliver(my_rank)))
        cap = sum(r["n_rows"] for r in recs) * min(K, len(mine))
        H.check_unpack(H.GpuUnpack(ctx, recs, cap), ref.dispatch_plain(toks, e2r, my_rank, cap), "%d tokens" % n)
