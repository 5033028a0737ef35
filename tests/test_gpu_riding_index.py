"""GPU parity of the receive index where it really rides in the expander's launch: the experts of a peer over several
workgroups, more chunks of experts than workgroups, a peer's rows over two and four workgroups, more than eight ids, repeated
rows dropped, wide bitmaps, with and without a riding plan, in workgroups of two and of eight waves; and of movers whose
rows are folded, packer and expander, beside index and plan.  The context
whose batch is expanded is made for far more rows than it holds, so that movers are expected that hide any index; that
nothing got a launch of its own is read from the events that bracket such launches.  Against the oracle, bit-exact."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2605_22428_amd import binding as B

import gpu_harness as H

pytestmark = pytest.mark.gpu

#         ranks, experts, top_k, max_tokens of the indexed batch, its rows' tokens per peer, my_rank
SHAPES = {
    "two_parts_four_row_parts": (8, 256, 8, 2048, 1400, 3),     # 24 of 32 experts a workgroup
    "passes": (2, 128, 8, 12000, 2500, 1),                      # 22 chunks of three experts, 16 workgroups
    "two_row_parts": (8, 64, 8, 1000, 900, 5),
    "one_part": (16, 64, 8, 300, 300, 2),
    "nine_ids": (8, 64, 9, 1200, 1000, 7),
    "twenty_ids": (8, 256, 20, 1500, 1100, 0),
    "wide": (130, 260, 8, 400, 400, 77),
    "sixty_four_local": (4, 256, 8, 1100, 1100, 1),
}


def _untouched(ctx, kernel):
    """Two recorded events that a launch of `kernel` on `ctx` would record again; returns the check that none did.  (Reading the same
    two events again can give a nanosecond more or less: device ticks are converted anew each time.)"""
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    a.record()
    torch.zeros(1 << 22, device=H.DEV).add_(1)
    b.record()
    torch.cuda.synchronize()
    was = a.elapsed_time(b)
    ctx.mw_ctx_set_timing_events(kernel, a, b)

    def check(what):
        ctx.mw_ctx_set_timing_events(kernel, None, None)
        assert abs(a.elapsed_time(b) - was) < 1e-5, "%s got a launch of its own" % what
    return check


@pytest.mark.parametrize("plan", [False, True])
@pytest.mark.parametrize("fmt,hidden", [(B.MW_ROW_BF16, 7168), (B.MW_ROW_FP8_E4M3_BLOCK128, 7168)])
@pytest.mark.parametrize("which", sorted(SHAPES))
def test_riding_index(which, fmt, hidden, plan):
    R, E, K, max_tokens, T, my_rank = SHAPES[which]
    print("riding index", which, fmt, plan, flush=True)
    rng = np.random.default_rng(sorted(SHAPES).index(which))
    e2r = (np.arange(E) * R // E).astype(np.int32)
    P, L = min(R, 8), int((e2r == my_rank).sum())
    nxt = B.Context(R, E, K, my_rank, hidden, fmt, max_tokens, P * max_tokens, e2r, device=H.DEV)
    cur = B.Context(R, E, K, my_rank, hidden, fmt, 65536, min(200000, R * 65536), e2r, device=H.DEV)
    nxt.mw_ctx_set_ride_wait_limit((1 << 21) - 1)               # plans ride whatever the sizes
    # The index alone is compared, with rows that say who they are in their first bytes: 64 of them, used in turn.
    small = B.Context(R, E, K, my_rank, 64, B.MW_ROW_BF16, max_tokens, 1, e2r, device=H.DEV)
    toks, recs = [], []
    for p in range(P):
        tk = rng.integers(0, E, size=(T, K)).astype(np.int32)
        tk[rng.random((T, K)) < 0.1] = -1
        x = rng.integers(0, 1 << 16, size=(T, 64), dtype=np.uint16)
        rec = H.shrink(H.GpuSend(small, tk, x, None).deliver(my_rank))
        n = rec["n_rows"]
        rows = torch.zeros((max(n, 1), nxt.row_stride), dtype=torch.uint8, device=H.DEV)
        rows[:, :128] = rec["rows"][: max(n, 1)]
        toks.append((tk, x, None))
        recs.append(dict(rec, rows=rows))
    cap = max(1, sum(r["n_rows"] for r in recs) * min(K, L))
    want = ref.dispatch_plain(toks, e2r, my_rank, cap)
    few = [dict(r, n_desc=min(r["n_desc"], 3), n_rows=int(H.host(r["desc"]).reshape(-1).view(B.DESC_DTYPE)["row_count"][: min(r["n_desc"], 3)].sum()))
           for r in recs]
    table, few_table = B.peers_table(recs, H.DEV), B.peers_table(few, H.DEV)
    a, b = B.RecvBuffers(cur, max(1, sum(r["n_rows"] for r in few) * min(K, L))), B.RecvBuffers(nxt, cap)
    cur.mw_unpack_index(few_table, P, a.capacity, a.expert_offsets, a.stats)
    checks = [(_untouched(nxt, B.MW_KERNEL_RECV_INDEX), "the index")]
    tk = rng.integers(0, E, size=(min(700, max_tokens), K)).astype(np.int32)
    if plan:
        s, tk_d = B.SendBuffers(nxt, len(tk)), H.dev(tk)
        checks += [(_untouched(nxt, B.MW_KERNEL_PLAN_RANK), "the plan"), (_untouched(nxt, B.MW_KERNEL_PLAN_GROUPS), "the plan")]
        cur.mw_unpack_expand_index_plan_next(P, a.out_rows, a.out_scales, a.capacity, a.out_src_peer, a.out_src_token, nxt, table, P,
                                             cap, b.expert_offsets, b.stats, tk_d, s.mask, s.perm, s.desc, s.stats)
    else:
        cur.mw_unpack_expand_index_next(P, a.out_rows, a.out_scales, a.capacity, a.out_src_peer, a.out_src_token, nxt, table, P, cap,
                                        b.expert_offsets, b.stats)
    torch.cuda.synchronize()
    for check, what in checks:
        check(what)
    nxt.mw_unpack_expand(P, b.out_rows, b.out_scales, cap, b.out_src_peer, b.out_src_token)
    st = nxt.mw_get_recv_stats(b.stats)
    q = int(st["n_out_rows"])
    assert int(st["error_flags"]) == 0 and q == len(want[2])
    H.assert_same_bytes(H.host(b.expert_offsets), want[4], "expert_offsets")
    H.assert_same_bytes(H.host(b.out_src_peer)[:q], want[2], "out_src_peer")
    H.assert_same_bytes(H.host(b.out_src_token)[:q], want[3], "out_src_token")
    H.assert_same_bytes(H.host(b.out_rows[:q, :128].contiguous()), want[0], "out_rows")
    if plan:
        _, perm, desc, _ = ref.plan(tk, e2r, R, 128)
        ss = nxt.mw_get_send_stats(s.stats)
        assert (int(ss["n_rows"]), int(ss["n_groups"]), int(ss["error_flags"])) == (len(perm), len(desc), 0)
        H.assert_same_bytes(H.host(s.perm)[: len(perm)], perm, "perm")


def test_riding_index_drops_repeats():
    """One workgroup a peer decides which of the repeats is taken, also where it rides."""
    R, E, K, T, my_rank, P, hidden = 8, 64, 8, 600, 4, 8, 1024
    print("riding index, repeats", flush=True)
    rng = np.random.default_rng(5)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    nxt = B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, 2 * T, 2 * P * T, e2r, device=H.DEV)
    cur = B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, 65536, 200000, e2r, device=H.DEV)
    nxt.mw_ctx_set_options(B.MW_OPT_RECV_DEDUP)
    toks, once, twice = [], [], []
    for p in range(P):
        tk = rng.integers(0, E, size=(T, K)).astype(np.int32)
        x = rng.integers(0, 1 << 16, size=(T, hidden), dtype=np.uint16)
        r = H.shrink(H.GpuSend(nxt, tk, x, None).deliver(my_rank))
        n, d = r["n_rows"], H.host(r["desc"]).reshape(-1).view(B.DESC_DTYPE)[: r["n_desc"]]
        again = d.copy()
        again["row_offset"] += n
        toks.append((tk, x, None))
        once.append(r)
        twice.append(dict(desc=H.dev(np.concatenate([d, again]).view(np.uint8)), rows=torch.cat([r["rows"][:n]] * 2),
                          row_src_token=torch.cat([r["row_src_token"][:n]] * 2), row_topk=torch.cat([r["row_topk"][:n]] * 2),
                          n_desc=2 * r["n_desc"], n_rows=2 * n))
    cap = sum(r["n_rows"] for r in once) * K
    a, b = B.RecvBuffers(cur, cap), B.RecvBuffers(nxt, cap)
    cur.mw_unpack_index(B.peers_table(once, H.DEV), P, cap, a.expert_offsets, a.stats)
    table = B.peers_table(twice, H.DEV)
    check = _untouched(nxt, B.MW_KERNEL_RECV_INDEX)
    cur.mw_unpack_expand_index_next(P, a.out_rows, None, cap, a.out_src_peer, a.out_src_token, nxt, table, P, cap, b.expert_offsets, b.stats)
    torch.cuda.synchronize()
    check("the index")
    nxt.mw_unpack_expand(P, b.out_rows, None, cap, b.out_src_peer, b.out_src_token)
    gu = H.GpuUnpack.__new__(H.GpuUnpack)
    gu.ctx, gu.buf, gu.stats = nxt, b, nxt.mw_get_recv_stats(b.stats)
    gu.Q = int(gu.stats["n_out_rows"])
    assert int(gu.stats["error_flags"]) == B.MW_FLAG_DUPLICATE_DROPPED
    gu.stats["error_flags"] = 0
    H.check_unpack(gu, ref.dispatch_plain(toks, e2r, my_rank, cap))


#                       row format, hidden: chunks of a row
FOLDED = {"257": (B.MW_ROW_BF16, 2056), "264_fp8": (B.MW_ROW_FP8_E4M3_BLOCK128, 4096), "528_fp8": (B.MW_ROW_FP8_E4M3_BLOCK128, 8192),
          "1039": (B.MW_ROW_BF16, 8312), "655_not_folded": (B.MW_ROW_BF16, 5240)}


def _batch(rng, ctx, R, E, K, T, P, hidden, fmt, my_rank):
    """P senders' tokens and regions and this rank's own tokens."""
    def tokens(n):
        tk = rng.integers(0, E, size=(n, K)).astype(np.int32)
        tk[rng.random((n, K)) < 0.1] = -1
        if fmt == B.MW_ROW_BF16:
            return tk, rng.integers(0, 1 << 16, size=(n, hidden), dtype=np.uint16), None
        return tk, rng.integers(0, 256, size=(n, hidden), dtype=np.uint8), rng.random((n, hidden // 128), dtype=np.float32)
    toks = [tokens(T) for _ in range(P)]
    recs = [H.shrink(H.GpuSend(ctx, *t).deliver(my_rank)) for t in toks]
    cap = max(1, sum(r["n_rows"] for r in recs) * min(K, ctx.n_local))
    return dict(toks=toks, recs=recs, cap=cap, table=B.peers_table(recs, H.DEV), own=tokens(T))


@pytest.mark.parametrize("call", ["index", "index_plan", "step"])
@pytest.mark.parametrize("R,E,K,which", [r + (w,) for w in sorted(FOLDED) for r in ((8, 64, 8), (8, 64, 9), (130, 260, 8))] +
                         [(100, 5600, 8, "264_fp8"), (100, 5600, 8, "528_fp8"), (200, 10700, 8, "528_fp8")])
def test_folded_rows_beside_riders(R, E, K, which, call):
    """Every byte of rows whose last chunks go to their first lanes, moved by the launch that also makes the next batch's index and
    plan.  Riders narrow the movers only where these are expected to take a good part longer: 200000 rows at several
    kilobytes, hundreds of microseconds, beside an index of 500 rows a peer, some ten.  (5600 and 10700 experts: their table has no room
    in the LDS of a rider of four and of eight waves, and the index has to ride all the same.)"""
    fmt, hidden = FOLDED[which]
    print("folded beside riders", which, R, K, call, flush=True)
    P, T, my_rank = 8, 500, R // 2
    rng = np.random.default_rng(hidden + R + K)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    nxt = B.Context(R, E, K, my_rank, hidden, fmt, T, P * T, e2r, device=H.DEV)
    cur = B.Context(R, E, K, my_rank, hidden, fmt, 65536, min(200000, R * 65536), e2r, device=H.DEV)
    nxt.mw_ctx_set_ride_wait_limit((1 << 21) - 1)               # plans ride whatever the sizes
    now, then = _batch(rng, nxt, R, E, K, 150, P, hidden, fmt, my_rank), _batch(rng, nxt, R, E, K, T, P, hidden, fmt, my_rank)
    a, b = B.RecvBuffers(cur, now["cap"]), B.RecvBuffers(nxt, then["cap"])
    a.out_rows.fill_(0x5a)
    cur.mw_unpack_index(now["table"], P, now["cap"], a.expert_offsets, a.stats)
    tk, x, sc = now["own"]
    tk_d, x_d, sc_d, s = H.dev(tk), H.dev(x), H.dev(sc), B.SendBuffers(cur, len(tk))
    cur.mw_plan(tk_d, s.mask, s.perm, s.desc, s.stats)
    ntk, ns = H.dev(then["own"][0]), B.SendBuffers(nxt, T)
    s.packed.fill_(0x3c)
    checks = [(_untouched(nxt, B.MW_KERNEL_RECV_INDEX), "the index")]
    if call != "index":
        checks += [(_untouched(nxt, k), "the plan") for k in (B.MW_KERNEL_PLAN_RANK, B.MW_KERNEL_PLAN_GROUPS)]
    expander = (P, a.out_rows, a.out_scales, now["cap"], a.out_src_peer, a.out_src_token)
    index = (nxt, then["table"], P, then["cap"], b.expert_offsets, b.stats)
    if call == "index":
        cur.mw_unpack_expand_index_next(*expander, *index)
    elif call == "index_plan":
        cur.mw_unpack_expand_index_plan_next(*expander, *index, ntk, ns.mask, ns.perm, ns.desc, ns.stats)
    else:
        cur.mw_stream_step(x_d, sc_d, tk_d, s.perm, s.stats, s.packed, s.row_src_token, s.row_topk, *expander, *index, ntk, ns.mask,
                           ns.perm, ns.desc, ns.stats)
    torch.cuda.synchronize()
    for check, what in checks:
        check(what)
    nxt.mw_unpack_expand(P, b.out_rows, b.out_scales, then["cap"], b.out_src_peer, b.out_src_token)
    for ctx, buf, batch, what in ((cur, a, now, "this batch"), (nxt, b, then, "the next")):
        gu = H.GpuUnpack.__new__(H.GpuUnpack)
        gu.ctx, gu.buf, gu.stats = ctx, buf, ctx.mw_get_recv_stats(buf.stats)
        gu.Q = int(gu.stats["n_out_rows"])
        H.check_unpack(gu, ref.dispatch_plain(batch["toks"], e2r, my_rank, batch["cap"]), what)
    if call == "step":
        _, perm, _, _ = ref.plan(tk, e2r, R, cur.row_bytes)
        packed, src, rtk = ref.pack(x, sc, tk, perm)
        H.assert_same_bytes(H.host(s.packed)[: len(perm), : cur.row_bytes], packed, "packed rows")
        assert (H.host(s.packed)[len(perm):] == 0x3c).all(), "rows behind the last packed one were written"
        H.assert_same_bytes(H.host(s.row_src_token)[: len(perm)], src, "row_src_token")
        H.assert_same_bytes(H.host(s.row_topk)[: len(perm)], rtk, "row_topk")
    if call != "index":
        _, perm, desc, _ = ref.plan(then["own"][0], e2r, R, nxt.row_bytes)
        st = nxt.mw_get_send_stats(ns.stats)
        assert (int(st["n_rows"]), int(st["n_groups"]), int(st["error_flags"])) == (len(perm), len(desc), 0)
        H.assert_same_bytes(H.host(ns.perm)[: len(perm)], perm, "perm")
