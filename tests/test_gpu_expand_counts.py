"""GPU parity of mw_unpack and mw_unpack_packets where the expander makes its places of the index's counts: one count, a wave of them
and one more or less, the most a wave takes and one more, rows of one and of several workgroups, folded rows; more rows than the launch
was made for, the first ones of every workgroup not addressed; fp8 rows and their scales; a rank without experts; statistics that move
a context to the index that finishes its counts and back; and what is left behind for a second expander.  Bit-exact."""
import numpy as np
import pytest

from oracle import ref
from paper_2605_22428_amd import binding as B

import gpu_harness as H

pytestmark = pytest.mark.gpu


def _filled(gu, ctx, n_peers, cap, want, what):
    """The second expander reads the bases that the first left in the workspace."""
    H.check_unpack(gu, want, what)
    again = B.RecvBuffers(ctx, cap)
    ctx.mw_unpack_expand(n_peers, again.out_rows, again.out_scales, cap, again.out_src_peer, again.out_src_token)
    for a, b in ((again.out_rows, want[0]), (again.out_src_peer, want[2]), (again.out_src_token, want[3])):
        H.assert_same_bytes(H.host(a)[: gu.Q], b, what + ", second expander")


#                         local experts, ranks, tokens, chunks
@pytest.mark.parametrize("L,R,T,chunks", [(1, 1, 700, 1), (7, 9, 300, 1), (8, 8, 300, 65), (5, 13, 200, 1), (15, 17, 100, 264),
                                          (1, 256, 40, 1), (4, 64, 40, 648), (32, 8, 300, 3), (257, 1, 700, 1), (6, 43, 50, 1),
                                          (48, 8, 300, 65), (2, 250, 40, 264), (8, 64, 40, 648), (513, 1, 700, 1), (27, 19, 60, 1)])
def test_counts(L, R, T, chunks):
    print("counts", L, R, T, chunks, flush=True)
    rng = np.random.default_rng(L * 1000 + R)
    E, K, me, hidden = L * R, min(4, L * R), R - 1, 8 * chunks
    e2r = (np.arange(E) // L).astype(np.int32)
    most = 6 * T
    ctx = B.Context(R, E, K, me, hidden, B.MW_ROW_BF16, most, R * most, e2r, device=H.DEV)
    # The last rank's bit is the highest: in a whole sender's buffer the rows for it come last.
    for batch, n, whole in ((0, T, False), (1, most if chunks == 1 else T, True)):
        toks, recs, packets = [], [], []
        for p in range(R):
            tk = rng.integers(0, E, size=(n, K)).astype(np.int32)
            tk[rng.random((n, K)) < 0.1] = -1
            x = rng.integers(0, 1 << 16, size=(n, hidden), dtype=np.uint16)
            toks.append((tk, x, None))
            g = H.GpuSend(ctx, tk, x, None)
            recs.append(g.full_record() if whole else H.shrink(g.deliver(me)))
            mask, perm, _, _ = ref.plan(tk, e2r, R, 2 * hidden)
            packets.append(H.dev(ref.deliver_packets(ref.pack_packets(x, None, tk, mask, perm), me)))
        cap = max(1, R * n * min(K, L))
        want = ref.dispatch_plain(toks, e2r, me, cap)
        for r in ("", " again"):
            _filled(H.GpuUnpack(ctx, recs, cap), ctx, R, cap, want, "batch %d%s" % (batch, r))
        buf = B.RecvBuffers(ctx, cap)
        ctx.mw_unpack_packets(B.packets_table(packets, [int(t.shape[0]) for t in packets], H.DEV), R, buf.out_rows, None, cap,
                              buf.out_src_peer, buf.out_src_token, buf.expert_offsets, buf.stats)
        gu = H.GpuUnpack.__new__(H.GpuUnpack)
        gu.ctx, gu.buf, gu.stats = ctx, buf, ctx.mw_get_recv_stats(buf.stats)
        gu.Q = int(gu.stats["n_out_rows"])
        _filled(gu, ctx, R, cap, want, "packets %d" % batch)
    ctx.close()


def _fp8_batch(rng, ctx, R, E, K, n, hidden, e2r, me):
    toks, recs, packets = [], [], []
    for _ in range(R):
        tk = rng.integers(0, E, size=(n, K)).astype(np.int32)
        x, sc = rng.integers(0, 256, size=(n, hidden), dtype=np.uint8), rng.random((n, hidden // 128), dtype=np.float32)
        toks.append((tk, x, sc))
        recs.append(H.shrink(H.GpuSend(ctx, tk, x, sc).deliver(me)))
        mask, perm, _, _ = ref.plan(tk, e2r, R, hidden + hidden // 32)
        packets.append(H.dev(ref.deliver_packets(ref.pack_packets(x, sc, tk, mask, perm), me)))
    return toks, recs, packets


def _same(ctx, buf, want, what):
    gu = H.GpuUnpack.__new__(H.GpuUnpack)
    gu.ctx, gu.buf, gu.stats = ctx, buf, ctx.mw_get_recv_stats(buf.stats)
    gu.Q = int(gu.stats["n_out_rows"])
    H.check_unpack(gu, want, what)
    return gu


#                         local experts, ranks, tokens, hidden: 64 counts, 65 to 256, 257 to 512, 513; rows folded (4096, 8192) and not
@pytest.mark.parametrize("L,R,T,hidden", [(4, 16, 300, 4096), (5, 13, 300, 4096), (8, 12, 300, 7168), (1, 256, 40, 4096), (4, 64, 40, 8192), (4, 64, 40, 512),
                                          (43, 6, 200, 4096), (48, 8, 200, 7168), (64, 8, 150, 8192), (27, 19, 60, 4096)])
def test_fp8_rows_and_their_scales(L, R, T, hidden):
    """Codes and scales of mw_unpack and mw_unpack_packets, of a second expander behind each, and of the two halves by themselves."""
    print("fp8 counts", L, R, T, hidden, flush=True)
    rng = np.random.default_rng(L * 1000 + R + hidden)
    E, K, me = L * R, min(4, L * R), R // 2
    e2r = (np.arange(E) // L).astype(np.int32)
    ctx = B.Context(R, E, K, me, hidden, B.MW_ROW_FP8_E4M3_BLOCK128, T, R * T, e2r, device=H.DEV)
    toks, recs, packets = _fp8_batch(rng, ctx, R, E, K, T, hidden, e2r, me)
    cap = R * T * min(K, L)
    want = ref.dispatch_plain(toks, e2r, me, cap)
    table, ptable = B.peers_table(recs, H.DEV), B.packets_table(packets, [int(t.shape[0]) for t in packets], H.DEV)
    for turn in ("", " again"):
        for call, tab in ((ctx.mw_unpack, table), (ctx.mw_unpack_packets, ptable)):
            buf, second = B.RecvBuffers(ctx, cap), B.RecvBuffers(ctx, cap)
            call(tab, R, buf.out_rows, buf.out_scales, cap, buf.out_src_peer, buf.out_src_token, buf.expert_offsets, buf.stats)
            ctx.mw_unpack_expand(R, second.out_rows, second.out_scales, cap, second.out_src_peer, second.out_src_token)
            second.expert_offsets.copy_(buf.expert_offsets), second.stats.copy_(buf.stats)
            _same(ctx, buf, want, "unpack" + turn)
            _same(ctx, second, want, "second expander" + turn)
    halves = B.RecvBuffers(ctx, cap)
    ctx.mw_unpack_index(table, R, cap, halves.expert_offsets, halves.stats)
    ctx.mw_unpack_expand(R, halves.out_rows, halves.out_scales, cap, halves.out_src_peer, halves.out_src_token)
    _same(ctx, halves, want, "halves")
    ctx.close()


@pytest.mark.parametrize("L,R,T,hidden", [(4, 64, 40, 7168), (1, 256, 40, 4096), (16, 16, 60, 4096), (48, 8, 100, 4096), (48, 8, 100, 7168)])
def test_statistics_take_a_context_across_the_most_bytes(L, R, T, hidden):
    """The choice follows the rows that the last batch's statistics showed: from few to more than the expander adds up for, and back."""
    print("counts across the bound", L, R, T, hidden, flush=True)
    rng = np.random.default_rng(L + R)
    E, K, me = L * R, min(4, L * R), R - 1
    e2r = (np.arange(E) // L).astype(np.int32)
    ctx = B.Context(R, E, K, me, hidden, B.MW_ROW_FP8_E4M3_BLOCK128, T, R * T, e2r, device=H.DEV)
    toks, recs, packets = _fp8_batch(rng, ctx, R, E, K, T, hidden, e2r, me)
    cap = R * T * min(K, L)
    want = ref.dispatch_plain(toks, e2r, me, cap)
    table, ptable = B.peers_table(recs, H.DEV), B.packets_table(packets, [int(t.shape[0]) for t in packets], H.DEV)
    for seen in (600, 16000, 1 << 20, 700, 40000, 900):
        host = np.zeros(1, dtype=B.RECV_STATS_DTYPE)
        host["n_rows_seen"] = seen
        for call, tab in ((ctx.mw_unpack, table), (ctx.mw_unpack_packets, ptable)):
            ctx.mw_get_recv_stats(H.dev(host.view(np.uint8)))            # (a caller's statistics of some batch)
            buf = B.RecvBuffers(ctx, cap)
            call(tab, R, buf.out_rows, buf.out_scales, cap, buf.out_src_peer, buf.out_src_token, buf.expert_offsets, buf.stats)
            _same(ctx, buf, want, "%d rows seen" % seen)
    ctx.close()


@pytest.mark.parametrize("chunks", [3, 264])
def test_a_rank_without_experts(chunks):
    """No counts at all: whole senders' buffers and packets, of which no row is for this rank."""
    print("no experts", chunks, flush=True)
    rng = np.random.default_rng(chunks)
    R, E, T, K, me, hidden = 5, 8, 400, 3, 2, 8 * chunks
    e2r = np.array([0, 0, 1, 1, 3, 3, 4, 4], dtype=np.int32)
    ctx = B.Context(R, E, K, me, hidden, B.MW_ROW_BF16, T, R * T, e2r, device=H.DEV)
    recs, packets = [], []
    for p in range(R):
        tk = rng.integers(0, E, size=(T, K)).astype(np.int32)
        x = rng.integers(0, 1 << 16, size=(T, hidden), dtype=np.uint16)
        recs.append(H.GpuSend(ctx, tk, x, None).full_record())
        mask, perm, _, _ = ref.plan(tk, e2r, R, 2 * hidden)
        packets.append(H.dev(ref.pack_packets(x, None, tk, mask, perm)))
    table = B.packets_table(packets, [int(t.shape[0]) for t in packets], H.DEV)
    for _ in range(2):                               # (the second time the context knows how many rows there are)
        buf = B.RecvBuffers(ctx, 64)
        for call, tab in ((ctx.mw_unpack, B.peers_table(recs, H.DEV)), (ctx.mw_unpack_packets, table)):
            buf.out_rows.fill_(0x5a), buf.expert_offsets.fill_(-1), buf.stats.fill_(0xff)
            call(tab, R, buf.out_rows, None, 64, buf.out_src_peer, buf.out_src_token, buf.expert_offsets, buf.stats)
            st = ctx.mw_get_recv_stats(buf.stats)
            assert (int(st["n_recv_rows"]), int(st["n_out_rows"]), int(st["error_flags"])) == (0, 0, 0)
            assert int(st["n_rows_seen"]) == R * T and buf.expert_offsets.tolist()[:1] == [0]
            assert bool((buf.out_rows == 0x5a).all())
    ctx.close()


def test_counts_capacity_and_flags():
    """Fewer output rows than arrive, and an id outside the range: what is in front is written, the flags say so, once."""
    rng = np.random.default_rng(5)
    L, R, T, K = 4, 16, 200, 4
    e2r = (np.arange(L * R) // L).astype(np.int32)
    ctx = B.Context(R, L * R, K, 3, 64, B.MW_ROW_BF16, T, R * T, e2r, device=H.DEV)
    toks, recs = [], []
    for p in range(R):
        tk = rng.integers(0, L * R, size=(T, K)).astype(np.int32)
        x = rng.integers(0, 1 << 16, size=(T, 64), dtype=np.uint16)
        toks.append((tk, x, None))
        recs.append(H.shrink(H.GpuSend(ctx, tk, x, None).deliver(3)))
    want = ref.dispatch_plain(toks, e2r, 3, R * T * K)
    q = len(want[2])
    gu = H.GpuUnpack(ctx, recs, q - 7)
    assert int(gu.stats["error_flags"]) == B.MW_FLAG_OUT_CAPACITY and gu.Q == q
    H.assert_same_bytes(H.host(gu.buf.out_rows)[: q - 7], want[0][: q - 7], "rows within the capacity")
    row = int((recs[2]["row_topk"][:, 0] // L == 3).nonzero()[0])        # (a row whose first id is local keeps its place)
    spoilt = recs[2]["row_topk"].clone()
    others = [j for j in range(1, K) if int(spoilt[row, j]) // L != 3]
    spoilt[row, others[0]] = L * R + 5
    gu = H.GpuUnpack(ctx, [dict(r, row_topk=spoilt) if i == 2 else r for i, r in enumerate(recs)], q)
    assert int(gu.stats["error_flags"]) == B.MW_FLAG_BAD_EXPERT
    H.check_unpack(H.GpuUnpack(ctx, recs, q), want, "after an error")
    ctx.close()
