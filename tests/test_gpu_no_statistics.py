"""GPU parity where nobody has said how many rows the peers hold: contexts much larger than their batches whose
statistics are not read before the calls, and a rank that gets all of its peers' tokens where an even share was to be
expected.  Row movers then stride over a grid sized for the expectation, and the index of a small step chooses
its form on the GPU from the peers' counts.  Against the oracle's plain definition, bit-exact."""
import numpy as np
import pytest
import torch

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


# ranks, experts, top_k, max_tokens, rows of each peer: one more and one less than the one-workgroup index takes,
# none, a region that is cut off at its capacity's edge, several rows a lane of one peer, wide bitmaps, many ids
SMALL = {
    "at_the_limit": (8, 32, 4, 256, [128] * 8),
    "past_the_limit": (8, 32, 4, 256, [128] * 7 + [129]),
    "far_past": (8, 32, 4, 2000, [2000, 0, 2000, 1, 7, 0, 64, 1500]),
    "few_of_many": (8, 32, 4, 2000, [3, 0, 0, 1, 0, 0, 0, 2]),
    "none": (8, 32, 4, 2000, [0] * 8),
    "one_peer": (2, 64, 8, 8192, [5000, 8192]),
    "wide": (130, 260, 8, 120, [120] * 130),
    "wide_even": (130, 260, 8, 120, [4] * 130),
    "many_ids": (256, 256, 12, 60, [60] * 256),
    "table_in_memory": (16, 2000, 3, 700, [300] * 16),
}


@pytest.mark.parametrize("which", sorted(SMALL))
def test_small_steps_without_statistics(which):
    R, E, K, max_tokens, counts = SMALL[which]
    my_rank, hidden, P = R // 2, 64, len(counts)
    print("step without statistics", which, flush=True)
    rng = np.random.default_rng(sorted(SMALL).index(which))
    e2r = (np.arange(E) * R // E).astype(np.int32)
    ctxs = [B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, max_tokens, P * max_tokens, e2r, device=H.DEV) for _ in range(2)]
    quiet = [max(1, c // 50) for c in counts]
    batches = [_batch(rng, ctxs[0], R, E, K, my_rank, hidden, c) for c in (quiet, counts, quiet, counts)]
    own = rng.integers(0, E, size=(60, K)).astype(np.int32)
    x = rng.integers(0, 1 << 16, size=(60, hidden), dtype=np.uint16)
    own_d, x_d = H.dev(own), H.dev(x)
    send = [B.SendBuffers(c, 60) for c in ctxs]
    tables = [B.peers_table(b[0], H.DEV) for b in batches]
    bufs = [B.RecvBuffers(ctxs[i % 2], b[1]) for i, b in enumerate(batches)]
    ctxs[0].mw_plan(own_d, send[0].mask, send[0].perm, send[0].desc, send[0].stats)
    ctxs[0].mw_unpack_index(tables[0], P, batches[0][1], bufs[0].expert_offsets, bufs[0].stats)
    for i in range(3):
        cur, nxt, s, n = ctxs[i % 2], ctxs[(i + 1) % 2], send[i % 2], send[(i + 1) % 2]
        b, cap, ncap = bufs[i], batches[i][1], batches[i + 1][1]
        if i == 1:                                   # without a plan: the index alone rides
            cur.mw_unpack_expand_index_next(P, b.out_rows, None, cap, b.out_src_peer, b.out_src_token, nxt, tables[i + 1], P, ncap,
                                            bufs[i + 1].expert_offsets, bufs[i + 1].stats)
            continue
        cur.mw_stream_step(x_d, None, own_d, s.perm, s.stats, s.packed, s.row_src_token, s.row_topk, P, b.out_rows, None, cap,
                           b.out_src_peer, b.out_src_token, nxt, tables[i + 1], P, ncap, bufs[i + 1].expert_offsets,
                           bufs[i + 1].stats, own_d, n.mask, n.perm, n.desc, n.stats)
        if i == 0:                                   # the third step packs by a plan of ctxs[0] again
            ctxs[0].mw_plan(own_d, send[0].mask, send[0].perm, send[0].desc, send[0].stats)
    b = bufs[3]
    ctxs[1].mw_unpack_expand(P, b.out_rows, None, batches[3][1], b.out_src_peer, b.out_src_token)
    for i in range(4):
        H.check_unpack(_received(ctxs[i % 2], bufs[i]), batches[i][2], "batch %d" % i)
    _, perm, _, _ = ref.plan(own, e2r, R, 2 * hidden)
    packed, _, _ = ref.pack(x, None, own, perm)
    H.assert_same_bytes(H.host(send[0].packed)[: len(perm)], packed, "packed")
    H.assert_same_bytes(H.host(send[1].perm)[: len(perm)], perm, "perm")


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


def test_replayed_small_steps_choose_by_the_counts_of_each_replay():
    """One captured launch, replayed with the peers' records rewritten in between: few rows, more than the one-workgroup
    index takes, few again."""
    R, E, K, max_tokens, my_rank, hidden = 8, 32, 4, 2000, 3, 64
    print("captured step without statistics", flush=True)
    rng = np.random.default_rng(77)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    cur, nxt, maker = (B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, max_tokens, R * max_tokens, e2r, device=H.DEV) for _ in range(3))
    batches = [_batch(rng, maker, R, E, K, my_rank, hidden, c) for c in ([5] * R, [1500] * R, [128] * R, [900, 0, 0, 125, 0, 0, 0, 0], [2] * R)]
    tables = [B.peers_table(b[0], H.DEV) for b in batches]
    cap = max(b[1] for b in batches)
    a, b, table = B.RecvBuffers(cur, cap), B.RecvBuffers(nxt, cap), tables[0].clone()
    cur.mw_unpack_index(tables[0], R, cap, a.expert_offsets, a.stats)

    def step():
        cur.mw_unpack_expand_index_next(R, a.out_rows, None, cap, a.out_src_peer, a.out_src_token, nxt, table, R, cap, b.expert_offsets,
                                        b.stats)
        nxt.mw_unpack_expand(R, b.out_rows, None, cap, b.out_src_peer, b.out_src_token)

    step()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        step()
    for i in (0, 1, 2, 3, 1, 4):
        table.copy_(tables[i])
        b.out_rows.zero_()
        g.replay()
        torch.cuda.synchronize()
        stats = np.frombuffer(H.host(b.stats).tobytes(), dtype=B.RECV_STATS_DTYPE)[0]     # (mw_get_recv_stats would be the hint)
        gu = H.GpuUnpack.__new__(H.GpuUnpack)
        gu.ctx, gu.buf, gu.stats, gu.Q = nxt, b, stats, int(stats["n_out_rows"])
        H.check_unpack(gu, batches[i][2], "replay of batch %d" % i)
