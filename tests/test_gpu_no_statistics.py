"""GPU parity where nobody has said how many rows the peers hold: contexts much larger than their batches whose
statistics are not read before the calls, and a rank that gets all of its peers' tokens where an even share was to be
expected.  Row movers then stride over a grid sized for the expectation.  Against the oracle's plain definition, bit-exact."""
import numpy as np
import pytest

from oracle import ref
from paper_2605_22428_amd import binding as B

import gpu_harness as H

pytestmark = pytest.mark.gpu


def _batch(rng, ctx, R, E, K, my_rank, hidden, counts):
    """Peers' tokens, `counts[p]` of them, all for this rank; their regions and what must come out."""
    e2r = (np.arange(E) * R // E).astype(np.int32)
    mine = np.nonzero(e2r == my_rank)[0]
    toks, recs = [], []
    for n in counts:
        tk = rng.integers(0, E, size=(n, K)).astype(np.int32)
        tk[:, rng.integers(0, K)] = mine[rng.integers(0, len(mine), size=n)]
        x = rng.integers(0, 1 << 16, size=(n, hidden), dtype=np.uint16)
        recs.append(H.shrink(H.GpuSend(ctx, tk, x, None).deliver(my_rank)))
        toks.append((tk, x, None))
    cap = max(1, sum(counts) * min(K, len(mine)))
    return recs, cap, ref.dispatch_plain(toks, e2r, my_rank, cap)


def _received(ctx, buf):
    gu = H.GpuUnpack.__new__(H.GpuUnpack)
    gu.ctx, gu.buf, gu.stats = ctx, buf, ctx.mw_get_recv_stats(buf.stats)
    gu.Q = int(gu.stats["n_out_rows"])
    return gu


@pytest.mark.parametrize("hidden,R,max_tokens,rows", [(2048, 64, 128, 128), (8, 256, 64, 64), (1032, 64, 4000, 100), (7168, 64, 64, 30)])
def test_unpack_and_combine_of_a_favoured_rank(hidden, R, max_tokens, rows):
    print("favoured rank", hidden, R, max_tokens, rows, flush=True)
    rng = np.random.default_rng(hidden)
    E, K, my_rank = R, 1, 5
    e2r = np.arange(R).astype(np.int32)
    ctx = B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, max_tokens, R * max_tokens, e2r, device=H.DEV)
    recs, cap, want = _batch(rng, ctx, R, E, K, my_rank, hidden, [rows] * R)
    buf, table = B.RecvBuffers(ctx, cap), B.peers_table(recs, H.DEV)
    ctx.mw_unpack(table, R, buf.out_rows, None, cap, buf.out_src_peer, buf.out_src_token, buf.expert_offsets, buf.stats)
    ret = buf.out_rows.new_zeros((cap, 2 * hidden))
    ctx.mw_combine_gather(R, buf.out_rows, cap, ret, cap)     # one expert a row: every row comes back as it was
    H.check_unpack(_received(ctx, buf), want)
    back = np.concatenate([H.host(r["rows"])[: r["n_rows"]] for r in recs])
    H.assert_same_bytes(H.host(ret)[: len(back)], back, "returned rows")
