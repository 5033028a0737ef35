"""GPU parity with id lists of every length and alignment.  The plan of a small batch (mw_plan_pack, a small stream step) and the small
launches' index read four ids a request, wherever they start, and what is left word by word; here lists of whole fours, of one to three
ids more, and of fewer, on a 16-byte unit and four bytes behind one, also for rows beyond one a lane.  Plans beyond 8192 tokens and
riding plans read word by word; they get the same lists.  Bit-exact."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2605_22428_amd import binding as B

import gpu_harness as H
import test_gpu_index_forms as forms

pytestmark = pytest.mark.gpu


def _ids(rng, T, E, K):
    tk = np.argsort(rng.random((T, E)), axis=1)[:, :K].astype(np.int32)
    tk[rng.random((T, K)) < 0.1] = -1
    return tk


def _check(ctx, buf, tk, e2r, R, row_bytes, what):
    st = ctx.mw_get_send_stats(buf.stats)
    mask, perm, desc, want = ref.plan(tk, e2r, R, row_bytes)
    assert (int(st["n_rows"]), int(st["n_groups"]), int(st["error_flags"])) == (len(perm), len(desc), 0), what
    H.assert_same_bytes(H.host(buf.mask).view(np.uint64)[: len(tk)], mask, what + " mask")
    H.assert_same_bytes(H.host(buf.perm)[: len(perm)], perm, what + " perm")
    H.assert_same_bytes(H.host(buf.desc).reshape(-1).view(B.DESC_DTYPE)[: len(desc)].view(np.uint8), desc.view(np.uint8), what + " desc")


@pytest.mark.parametrize("K", [1, 3, 4, 5, 6, 7, 8, 9, 11, 12])
@pytest.mark.parametrize("shifted", [False, True])
def test_id_lists(K, shifted):
    print("id lists", K, shifted, flush=True)
    rng = np.random.default_rng(K)
    move = forms._shifted if shifted else (lambda t: t)
    for R, E, T in ((8, 32, 200), (130, 260, 300), (8, 32, 8300)):
        e2r = (np.arange(E) * R // E).astype(np.int32)
        ctx = B.Context(R, E, K, 1, 8, B.MW_ROW_BF16, T, R * T, e2r, device=H.DEV)
        tk = _ids(rng, T, E, K)
        topk, buf = move(H.dev(tk)), B.SendBuffers(ctx, T)
        if T <= 256:
            x = rng.integers(0, 1 << 16, size=(T, 8), dtype=np.uint16)
            ctx.mw_plan_pack(topk, H.dev(x), None, buf.mask, buf.perm, buf.desc, buf.stats, buf.packed, buf.row_src_token, buf.row_topk)
        else:
            ctx.mw_plan(topk, buf.mask, buf.perm, buf.desc, buf.stats)
        _check(ctx, buf, tk, e2r, R, 16, "%d tokens" % T)
        ctx.close()

    # the one-workgroup index, rows in registers and (a batch of more than 512 rows where a few were seen last) through memory: with
    # the expander in one launch, and by itself
    R, E, T, hidden, my_rank = 8, 32, 700, 8, 3
    e2r = (np.arange(E) * R // E).astype(np.int32)
    ctx = B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, T, R * T, e2r, device=H.DEV)
    sizes = []
    for n in (9, T):
        toks, recs = [], []
        for p in range(R):
            tk, x = _ids(rng, n, E, K), rng.integers(0, 1 << 16, size=(n, hidden), dtype=np.uint16)
            toks.append((tk, x, None))
            r = H.shrink(H.GpuSend(ctx, tk, x, None).deliver(my_rank))
            recs.append(dict(r, row_topk=move(r["row_topk"])))
        cap = max(1, sum(r["n_rows"] for r in recs) * min(K, 4))
        sizes.append((recs, cap, ref.dispatch_plain(toks, e2r, my_rank, cap)))
    (few, few_cap, few_want), (many, cap, want) = sizes
    assert sum(r["n_rows"] for r in few) <= 512 < sum(r["n_rows"] for r in many)
    for halves in (False, True):
        for _ in range(2):                                   # (after the large batch the first one is indexed in the general form)
            H.check_unpack(H.GpuUnpack(ctx, few, few_cap), few_want, "a few rows")
        b = B.RecvBuffers(ctx, cap)
        if halves:
            ctx.mw_unpack_index(B.peers_table(many, H.DEV), R, cap, b.expert_offsets, b.stats)
            ctx.mw_unpack_expand(R, b.out_rows, None, cap, b.out_src_peer, b.out_src_token)
        else:
            ctx.mw_unpack(B.peers_table(many, H.DEV), R, b.out_rows, None, cap, b.out_src_peer, b.out_src_token, b.expert_offsets, b.stats)
        gu = H.GpuUnpack.__new__(H.GpuUnpack)
        gu.ctx, gu.buf, gu.stats = ctx, b, ctx.mw_get_recv_stats(b.stats)
        gu.Q = int(gu.stats["n_out_rows"])
        H.check_unpack(gu, want, "more rows than lanes")
    ctx.close()

    # steps whose index and plan ride
    R, E, T, hidden, my_rank = 8, 32, 60, 64, 3
    e2r = (np.arange(E) * R // E).astype(np.int32)
    ctxs = [B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, T, R * T, e2r, device=H.DEV) for _ in range(2)]
    batches = []
    for c in ctxs:
        toks, recs = [], []
        for p in range(R):
            tk, x = _ids(rng, T, E, K), rng.integers(0, 1 << 16, size=(T, hidden), dtype=np.uint16)
            toks.append((tk, x, None))
            r = H.shrink(H.GpuSend(c, tk, x, None).deliver(my_rank))
            recs.append(dict(r, row_topk=move(r["row_topk"])))
        cap = max(1, sum(r["n_rows"] for r in recs) * min(K, 4))
        H.check_unpack(H.GpuUnpack(c, recs, cap), ref.dispatch_plain(toks, e2r, my_rank, cap), "unpack")
        H.check_unpack(H.GpuUnpack(c, recs, cap), ref.dispatch_plain(toks, e2r, my_rank, cap), "unpack again")
        tk, x = _ids(rng, T, E, K), rng.integers(0, 1 << 16, size=(T, hidden), dtype=np.uint16)
        batches.append(dict(toks=toks, recs=recs, cap=cap, table=B.peers_table(recs, H.DEV), tk=tk, topk=move(H.dev(tk)), x=H.dev(x),
                            send=B.SendBuffers(c, T), recv=B.RecvBuffers(c, cap)))
    for forced in (False, True):                             # (a set wait limit: the plan rides)
        if forced:
            for c in ctxs:
                c.mw_ctx_set_ride_wait_limit((1 << 21) - 1)
        b, n = batches
        ctxs[0].mw_unpack_index(b["table"], R, b["cap"], b["recv"].expert_offsets, b["recv"].stats)
        ctxs[0].mw_plan(b["topk"], b["send"].mask, b["send"].perm, b["send"].desc, b["send"].stats)
        s, r, ns, nr = b["send"], b["recv"], n["send"], n["recv"]
        ns.perm.fill_(-1)
        ctxs[0].mw_stream_step(b["x"], None, b["topk"], s.perm, s.stats, s.packed, s.row_src_token, s.row_topk, R, r.out_rows, None,
                               b["cap"], r.out_src_peer, r.out_src_token, ctxs[1], n["table"], R, n["cap"], nr.expert_offsets, nr.stats,
                               n["topk"], ns.mask, ns.perm, ns.desc, ns.stats)
        ctxs[1].mw_unpack_expand(R, nr.out_rows, None, n["cap"], nr.out_src_peer, nr.out_src_token)
        _check(ctxs[1], ns, n["tk"], e2r, R, 2 * hidden, "plan of a step")
        gu = H.GpuUnpack.__new__(H.GpuUnpack)
        gu.ctx, gu.buf, gu.stats = ctxs[1], nr, ctxs[1].mw_get_recv_stats(nr.stats)
        gu.Q = int(gu.stats["n_out_rows"])
        H.check_unpack(gu, ref.dispatch_plain(n["toks"], e2r, my_rank, n["cap"]), "index of a step")


@pytest.mark.parametrize("shifted", [False, True])
@pytest.mark.parametrize("R,E,K", [(8, 64, 8), (130, 260, 12)])
def test_riding_plan(R, E, K, shifted, monkeypatch):
    """A plan that rides beside rows (300 tokens, several workgroups), its ids on a 16-byte unit and four bytes behind one: read word by
    word either way."""
    if shifted:
        monkeypatch.setattr(forms.H, "dev", lambda a, dev=H.dev: forms._shifted(dev(a)) if getattr(a, "dtype", None) == np.int32 and a.ndim == 2
                            and a.shape[1] == K else dev(a))
    forms.test_stream_steps_with_riders_and_without(R, E, 300, K, 1024, True)
