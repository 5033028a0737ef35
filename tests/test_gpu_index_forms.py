"""GPU parity of the receive index where its form changes: experts spread over several workgroups a
peer and over several passes of one, id lists that are not whole 16-byte units or do not start on
one, more than eight ids, more than 64 local experts, more experts than the table in LDS holds, the
largest batch; on its own, in front of or (small batches) beside the expander, from packets, and dropping repeated
rows.  (Riding beside long movers: test_gpu_riding_index.py.)
Against the oracle's plain definition, bit-exact."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2605_22428_amd import binding as B

import gpu_harness as H

pytestmark = pytest.mark.gpu

#          ranks, experts, top_k, tokens, my_rank
SHAPES = {
    "four_parts": (8, 256, 8, 1500, 3),            # 32 experts here, more rows of a peer than lanes
    "parts_and_passes": (2, 128, 8, 8192, 1),      # several experts, long bitmaps
    "sixty_four_local": (4, 256, 8, 300, 2),
    "sixty_five_local": (1, 65, 8, 400, 0),        # no 64-bit set of experts
    "nine_ids": (8, 64, 9, 700, 7),
    "six_ids": (8, 64, 6, 700, 0),                 # ids word by word
    "one_id": (16, 64, 1, 333, 5),
    "table_in_memory": (100, 3000, 4, 300, 99),    # more experts than a small workgroup's table of slots
    "many_local": (2, 2000, 4, 500, 1),            # slots do not fit a byte
    "many_local_one_word": (2, 2000, 4, 30, 0),    # an expert's bits walked by a lane: one word, 24 (the most), 25
    "many_local_24_words": (2, 1200, 4, 768, 1),
    "many_local_25_words": (2, 1200, 4, 769, 0),
    "largest": (1, 1, 1, 65536, 0),                # every row to one expert: the count is 2^16
}


def _tokens(rng, R, E, K, T, hidden):
    tk = rng.integers(0, E, size=(T, K)).astype(np.int32)       # ids repeat by themselves
    if T < 65536:
        tk[rng.random((T, K)) < 0.1] = -1
    return tk, rng.integers(0, 1 << 16, size=(T, hidden), dtype=np.uint16)


def _shifted(t):
    """The same values four bytes into a fresh allocation."""
    flat = torch.zeros(t.numel() + 1, dtype=t.dtype, device=t.device)
    flat[1:] = t.reshape(-1)
    return flat[1:].view(t.shape)


@pytest.mark.parametrize("which", sorted(SHAPES))
def test_index_forms(which):
    R, E, K, T, my_rank = SHAPES[which]
    print("index form", which, flush=True)
    rng = np.random.default_rng(sorted(SHAPES).index(which))
    hidden, n_peers = 8, min(R, 8)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    L = int((e2r == my_rank).sum())
    ctx, nxt = (B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, T, n_peers * T, e2r, device=H.DEV) for _ in range(2))
    toks, recs, packets = [], [], []
    for p in range(n_peers):
        tk, x = _tokens(rng, R, E, K, T, hidden)
        toks.append((tk, x, None))
        g = H.GpuSend(ctx, tk, x, None)
        rec = H.shrink(g.deliver(my_rank))
        if p % 2:
            rec["row_topk"] = _shifted(rec["row_topk"])
        recs.append(rec)
        mask, perm, _, _ = ref.plan(tk, e2r, R, 2 * hidden)
        pk = ref.deliver_packets(ref.pack_packets(x, None, tk, mask, perm), my_rank)
        packets.append(H.dev(pk))
    cap = max(1, sum(r["n_rows"] for r in recs) * min(K, L))
    want = ref.dispatch_plain(toks, e2r, my_rank, cap)
    H.check_unpack(H.GpuUnpack(ctx, recs, cap), want, "alone")
    H.check_unpack(H.GpuUnpack(ctx, recs, cap), want, "alone, row count known")

    a, b = B.RecvBuffers(ctx, cap), B.RecvBuffers(nxt, cap)
    table = B.peers_table(recs, H.DEV)
    if 3 * ((T + 31) // 32) + 64 <= 1280:
        ctx.mw_unpack_expand_index_next(n_peers, a.out_rows, None, cap, a.out_src_peer, a.out_src_token, nxt, table, n_peers,
                                        cap, b.expert_offsets, b.stats)
        nxt.mw_unpack_expand(n_peers, b.out_rows, None, cap, b.out_src_peer, b.out_src_token)
        gu = H.GpuUnpack.__new__(H.GpuUnpack)
        gu.ctx, gu.buf, gu.stats = nxt, b, nxt.mw_get_recv_stats(b.stats)
        gu.Q = int(gu.stats["n_out_rows"])
        H.check_unpack(gu, want, "with an expander")

    ptable = B.packets_table(packets, [int(t.shape[0]) for t in packets], H.DEV)
    nxt.mw_unpack_packets(ptable, n_peers, b.out_rows, None, cap, b.out_src_peer, b.out_src_token, b.expert_offsets, b.stats)
    gu = H.GpuUnpack.__new__(H.GpuUnpack)
    gu.ctx, gu.buf, gu.stats = nxt, b, nxt.mw_get_recv_stats(b.stats)
    gu.Q = int(gu.stats["n_out_rows"])
    H.check_unpack(gu, want, "packets")

    # every region twice over, repeats dropped (regions within max_tokens)
    if max(r["n_rows"] for r in recs) * 2 <= T:
        nxt.mw_ctx_set_options(B.MW_OPT_RECV_DEDUP)
        twice = []
        for r in recs:
            n, d = r["n_rows"], H.host(r["desc"]).reshape(-1).view(B.DESC_DTYPE)[: r["n_desc"]]
            again = d.copy()
            again["row_offset"] += n
            twice.append(dict(desc=H.dev(np.concatenate([d, again]).view(np.uint8)), rows=torch.cat([r["rows"][:n]] * 2),
                              row_src_token=torch.cat([r["row_src_token"][:n]] * 2),
                              row_topk=torch.cat([r["row_topk"][:n]] * 2), n_desc=2 * r["n_desc"], n_rows=2 * n))
        gu = H.GpuUnpack(nxt, twice, cap)
        assert int(gu.stats["error_flags"]) == B.MW_FLAG_DUPLICATE_DROPPED
        gu.stats["error_flags"] = 0
        H.check_unpack(gu, want, "repeats dropped")


@pytest.mark.parametrize("hidden,forced", [(8, False), (8, True), (1024, False), (4096, True)])
@pytest.mark.parametrize("R,E,T,K", [(8, 256, 1100, 8), (4, 16, 2600, 8), (130, 260, 300, 8), (8, 256, 1100, 20), (4, 16, 2600, 9),
                                     (130, 260, 300, 16)])
def test_stream_steps_with_riders_and_without(R, E, T, K, hidden, forced):
    """mw_stream_step where index and plan ride and where they get launches of their own (movers too short),
    and with a plan that is made to ride; rows of a peer spread over several workgroups."""
    print("stream step", R, E, T, K, hidden, forced, flush=True)
    my_rank, n_peers = R // 2, min(R, 8)
    rng = np.random.default_rng(R + T + hidden)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    ctxs = [B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, T, n_peers * T, e2r, device=H.DEV) for _ in range(2)]
    if forced:
        for c in ctxs:
            c.mw_ctx_set_ride_wait_limit((1 << 21) - 1)
    batches = []
    for c in ctxs:
        toks = [_tokens(rng, R, E, K, T, hidden) for _ in range(n_peers)]
        recs = [H.shrink(H.GpuSend(c, tk, x, None).deliver(my_rank)) for tk, x in toks]
        cap = sum(r["n_rows"] for r in recs) * min(K, c.n_local) + 1
        tk, x = _tokens(rng, R, E, K, T, hidden)
        batches.append(dict(toks=[(a, b, None) for a, b in toks], recs=recs, cap=cap, table=B.peers_table(recs, H.DEV), tk=tk, x=x,
                            tk_d=H.dev(tk), x_d=H.dev(x), send=B.SendBuffers(c, T), recv=B.RecvBuffers(c, cap)))
    b0 = batches[0]
    ctxs[0].mw_unpack_index(b0["table"], n_peers, b0["cap"], b0["recv"].expert_offsets, b0["recv"].stats)
    ctxs[0].mw_get_recv_stats(b0["recv"].stats)
    s = b0["send"]
    ctxs[0].mw_plan(b0["tk_d"], s.mask, s.perm, s.desc, s.stats)
    for i in range(4):
        cur, nxt, b, n = ctxs[i % 2], ctxs[(i + 1) % 2], batches[i % 2], batches[(i + 1) % 2]
        s, r, ns, nr = b["send"], b["recv"], n["send"], n["recv"]
        if i > 1:
            ns.perm.fill_(-1)
        cur.mw_stream_step(b["x_d"], None, b["tk_d"], s.perm, s.stats, s.packed, s.row_src_token, s.row_topk, n_peers,
                           r.out_rows, None, b["cap"], r.out_src_peer, r.out_src_token, nxt, n["table"], n_peers, n["cap"],
                           nr.expert_offsets, nr.stats, n["tk_d"], ns.mask, ns.perm, ns.desc, ns.stats)
        if i == 0:
            nxt.mw_get_recv_stats(nr.stats)
    for c, b in zip(ctxs, batches):
        gu = H.GpuUnpack.__new__(H.GpuUnpack)
        gu.ctx, gu.buf, gu.stats = c, b["recv"], c.mw_get_recv_stats(b["recv"].stats)
        gu.Q = int(gu.stats["n_out_rows"])
        H.check_unpack(gu, ref.dispatch_plain(b["toks"], e2r, my_rank, b["cap"]), "step")
        mask, perm, desc, want = ref.plan(b["tk"], e2r, R, 2 * hidden)
        st = c.mw_get_send_stats(b["send"].stats)
        assert (int(st["n_rows"]), int(st["n_groups"]), int(st["error_flags"])) == (len(perm), len(desc), 0)
        H.assert_same_bytes(st["rows_per_dest"], want["rows_per_dest"], "rows_per_dest")
        H.assert_same_bytes(H.host(b["send"].perm)[: len(perm)], perm, "perm")
        H.assert_same_bytes(H.host(b["send"].mask).view(np.uint64)[:T], mask, "mask")
        H.assert_same_bytes(H.host(b["send"].desc).reshape(-1).view(B.DESC_DTYPE)[: len(desc)].view(np.uint8), desc.view(np.uint8), "desc")
        packed, src, rtk = ref.pack(b["x"], None, b["tk"], perm)
        H.assert_same_bytes(H.host(b["send"].packed)[: len(perm)], packed, "packed")


@pytest.mark.parametrize("R,L,n_peers", [(73, 7, 73), (128, 4, 128), (171, 3, 171), (256, 2, 256), (256, 2, 255), (256, 3, 170), (40, 13, 40),
                                         (97, 1, 97), (60, 16, 32), (60, 16, 33)])
def test_counts_finished_by_a_wave_or_a_workgroup(R, L, n_peers):
    """Up to 512 (expert, peer) counts are scanned by the wave that reported last, more by its workgroup; peers of no row, of
    one, and of more rows than lanes; a flag raised by one batch is gone in the next."""
    print("counts", R, L, n_peers, flush=True)
    E, K, T, my_rank, hidden = R * L, 4, 500, R - 1, 8
    rng = np.random.default_rng(R * L + n_peers)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    mine = np.nonzero(e2r == my_rank)[0]
    ctx = B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, T, n_peers * T, e2r, device=H.DEV)
    toks, recs = [], []
    for p in range(n_peers):
        n = T if p == n_peers // 2 else p % 4
        tk = np.argsort(rng.random((n, E)), axis=1)[:, :K].astype(np.int32) if n else np.zeros((0, K), np.int32)
        tk[np.arange(n), rng.integers(0, K, n)] = rng.choice(mine, n)
        x = rng.integers(0, 1 << 16, size=(n, hidden), dtype=np.uint16)
        toks.append((tk, x, None))
        recs.append(H.shrink(H.GpuSend(ctx, tk, x, None).deliver(my_rank)))
    cap = sum(r["n_rows"] for r in recs) * min(K, L)
    want = ref.dispatch_plain(toks, e2r, my_rank, cap)
    H.check_unpack(H.GpuUnpack(ctx, recs, cap), want, "first")
    bad = dict(recs[n_peers // 2], row_topk=recs[n_peers // 2]["row_topk"].clone())
    ids = bad["row_topk"][7]
    ids[~torch.isin(ids, H.dev(mine.astype(np.int32)))] = E
    broken = recs[: n_peers // 2] + [bad] + recs[n_peers // 2 + 1:]
    flagged = bool((ids == E).any())
    for _ in range(2):
        assert int(H.GpuUnpack(ctx, broken, cap).stats["error_flags"]) == (B.MW_FLAG_BAD_EXPERT if flagged else 0)
    H.check_unpack(H.GpuUnpack(ctx, recs, cap), want, "after a flagged batch")


@pytest.mark.parametrize("T", [12, 60, 400, 2000, 4000])
def test_rows_of_other_ranks_are_not_looked_at(T):
    """Whole sender buffers as regions: rows whose group does not name this rank carry ids and source tokens outside every range, and
    raise no flag, whichever form the index takes (one launch with the expander, one workgroup, rows a lane keeps in registers and
    rows beyond them, rows spread over riders)."""
    print("other ranks' rows", T, flush=True)
    R, E, K, my_rank, hidden = 8, 32, 4, 5, 8
    rng = np.random.default_rng(T)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    ctx, nxt, far = (B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, mt, R * mt, e2r, device=H.DEV) for mt in (T, T, 65536))
    recs, bufs = [], []
    for _ in range(R):
        tk = rng.integers(0, E, size=(T, K)).astype(np.int32)
        x = rng.integers(0, 1 << 16, size=(T, hidden), dtype=np.uint16)
        _, perm, desc, _ = ref.plan(tk, e2r, R, 2 * hidden)
        packed, src, rtk = ref.pack(x, None, tk, perm)
        src, rtk, other = src.copy(), rtk.copy(), 0
        for d in desc:
            if not (int(d["mask"][0]) >> my_rank) & 1:
                rows = slice(int(d["row_offset"]), int(d["row_offset"]) + int(d["row_count"]))
                rtk[rows], src[rows], other = E + 5, T + 9, other + int(d["row_count"])
        assert other > 0
        bufs.append((desc, packed, src, rtk))
        recs.append(dict(desc=H.dev(desc.view(np.uint8).reshape(len(desc), -1)), rows=H.dev(packed), row_src_token=H.dev(src), row_topk=H.dev(rtk),
                         n_desc=len(desc), n_rows=len(perm)))
    cap = K * R * T
    want = ref.unpack(bufs, K, e2r, my_rank, 2 * hidden, 0, cap)
    for _ in range(2):
        H.check_unpack(H.GpuUnpack(ctx, recs, cap), want, "unpack")
    table = B.peers_table(recs, H.DEV)
    a, b = B.RecvBuffers(far, cap), B.RecvBuffers(nxt, cap)
    far.mw_unpack_index(table, R, cap, a.expert_offsets, a.stats)
    if 3 * ((T + 31) // 32) + 64 <= 1280:
        far.mw_unpack_expand_index_next(R, a.out_rows, None, cap, a.out_src_peer, a.out_src_token, nxt, table, R, cap, b.expert_offsets, b.stats)
    else:
        nxt.mw_unpack_index(table, R, cap, b.expert_offsets, b.stats)
    nxt.mw_unpack_expand(R, b.out_rows, None, cap, b.out_src_peer, b.out_src_token)
    gu = H.GpuUnpack.__new__(H.GpuUnpack)
    gu.ctx, gu.buf, gu.stats = nxt, b, nxt.mw_get_recv_stats(b.stats)
    gu.Q = int(gu.stats["n_out_rows"])
    H.check_unpack(gu, want, "index beside an expander")
