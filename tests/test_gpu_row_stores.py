"""GPU parity of the packers, the relays and the steps on both sides of the sizes that choose the store of their rows: rows and packets of
whole cache lines, of whole 64-byte pieces and of neither, batches of just under and over 2 and 18 MiB.  Bit-exact; what lies behind the
rows stays as it is."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2605_22428_amd import binding as B
from paper_2605_22428_amd import workloads as W

import gpu_harness as H
import test_gpu_packets as packets
import test_gpu_relay as relay

pytestmark = pytest.mark.gpu


def _workload(name, T, hidden, fmt="bf16", ranks=16):
    return W.DispatchWorkload(name, 81, ranks, 2 * ranks, 4, T, hidden, fmt, "uniform")


@pytest.mark.parametrize("T,hidden,fmt", [(1700, 600, "bf16"), (1800, 600, "bf16"), (15800, 600, "bf16"), (3000, 1224, "bf16"), (3000, 1288, "bf16"),
                                          (1000, 2048, "fp8"), (400, 7168, "fp8"), (7000, 136, "bf16"), (8100, 136, "bf16"), (3000, 640, "bf16"),
                                          (300, 5184, "bf16")])
def test_packers(T, hidden, fmt):
    print("row stores, packers", T, hidden, fmt, flush=True)
    w = _workload("stores", T, hidden, fmt)
    ctx = H.make_ctx(w, 0)
    tk = W.topk_ids(w, 5, 0)
    x, sc = W.payload_rows(w, 5, 0)
    H.check_send(w, H.GpuSend(ctx, tk, x, sc, prefill=0x5c), tk, x, sc)
    g = packets.GpuPackets(ctx, tk, x, sc)
    H.assert_same_bytes(H.host(g.packets)[: g.N], H.oracle_packets(w, tk, x, sc), "packets")
    assert not H.host(g.packets)[g.N:].any(), "packets behind the last one were written"
    ctx.close()


RELAYED = [(1700, 600, "bf16"), (1800, 600, "bf16"), (300, 7168, "fp8"), (200, 7168, "fp8"), (1100, 2048, "fp8"), (500, 2912, "bf16"), (1000, 1504, "bf16"),
           (700, 2048, "bf16")]


@pytest.mark.parametrize("T,hidden,fmt", RELAYED)
def test_relays(T, hidden, fmt):
    """A relay by itself, beside the next buffer's index, and two buffers a launch."""
    print("row stores, relays", T, hidden, fmt, flush=True)
    w = _workload("stores", T, hidden, fmt)
    tables = [((np.arange(16) * 5 // 16).astype(np.int32), 5), ((np.arange(16) % 7).astype(np.int32), 7)]
    ctxs = [relay._ctx(w, 0, 8) for _ in range(4)]
    sends, parents = [], []
    for i in range(4):
        tk = W.topk_ids(w, 6 + i, i)
        x, sc = W.payload_rows(w, 6 + i, i)
        sends.append(H.GpuSend(ctxs[0], tk, x, sc))
        parents.append(H.oracle_send(w, tk, x, sc))
    ch, st, _ = relay.gpu_relay(ctxs[0], sends[0].full_record(), *tables[0], T)
    relay.check_children(ch, st, parents[0], *tables[0], w.row_bytes)
    for i, c in enumerate(ctxs):
        c.mw_set_forwarding(*tables[i % 2])
    kids = [B.RelayChildren(c, tables[i % 2][1], T) for i, c in enumerate(ctxs)]
    recs = [B.peers_table([g.full_record()], H.DEV) for g in sends]
    jobs = [B.relay_job(c, recs[i], kids[i].table, T, kids[i].stats) for i, c in enumerate(ctxs)]
    ctxs[0].mw_relay_index(recs[0], kids[0].table, T, kids[0].stats)
    ctxs[0].mw_relay_copy_index_next(recs[0], kids[0].table, kids[0].stats, ctxs[1], recs[1], kids[1].table, T, kids[1].stats)
    B.mw_relay_batch(jobs[1:2], jobs[2:4])
    B.mw_relay_batch(jobs[2:4], [])
    for i, c in enumerate(ctxs):
        relay.check_children(kids[i], c.mw_get_relay_stats(kids[i].stats), parents[i], *tables[i % 2], w.row_bytes)
        c.close()


@pytest.mark.parametrize("T,hidden,fmt", RELAYED)
def test_relays_of_packets(T, hidden, fmt):
    print("row stores, packets relayed", T, hidden, fmt, flush=True)
    w = _workload("stores", T, hidden, fmt)
    tables = [((np.arange(16) * 5 // 16).astype(np.int32), 5), ((np.arange(16) % 7).astype(np.int32), 7)]
    ctxs = [packets._relay_ctx(w, 0, 8) for _ in range(2)]
    sent, parents, kids, child_tables, recs, stats = [], [], [], [], [], []
    for i, c in enumerate(ctxs):
        c.mw_set_forwarding(*tables[i])
        tk = W.topk_ids(w, 9 + i, i)
        x, sc = W.payload_rows(w, 9 + i, i)
        sent.append(packets.GpuPackets(ctxs[0], tk, x, sc))
        parents.append(H.oracle_packets(w, tk, x, sc))
        kids.append([torch.zeros((T, sent[i].packets.shape[1]), dtype=torch.uint8, device=H.DEV) for _ in range(tables[i][1])])
        child_tables.append(torch.tensor([k.data_ptr() for k in kids[i]], dtype=torch.int64, device=H.DEV))
        recs.append(B.packets_table([sent[i].packets], [sent[i].N], H.DEV))
        stats.append(torch.zeros(B.RELAY_STATS_BYTES, dtype=torch.uint8, device=H.DEV))
    ctxs[0].mw_relay_packets_index(recs[0], T, stats[0])
    ctxs[0].mw_relay_packets_copy_index_next(recs[0], child_tables[0], stats[0], ctxs[1], recs[1], T, stats[1])
    ctxs[1].mw_relay_packets_copy(recs[1], child_tables[1], stats[1])
    for i, c in enumerate(ctxs):
        st = c.mw_get_relay_stats(stats[i])
        assert int(st["error_flags"]) == 0
        for h in range(tables[i][1]):
            want = ref.relay_packets_child(parents[i], *tables[i], h)[0]
            assert int(st["rows_per_hop"][h]) == len(want)
            H.assert_same_bytes(H.host(kids[i][h])[: len(want)], want, "buffer %d child %d" % (i, h))
            assert not H.host(kids[i][h])[len(want):].any(), "packets behind the last one were written"
        c.close()


@pytest.mark.parametrize("T,hidden,fmt", [(1500, 328, "bf16"), (1500, 600, "bf16"), (1500, 992, "bf16"), (1500, 640, "bf16"), (1200, 3584, "fp8")])
def test_steps(T, hidden, fmt):
    """A step with movers that outlast its riders: this rank's tokens packed, the received rows expanded."""
    print("row stores, steps", T, hidden, fmt, flush=True)
    w, me = _workload("stores", T, hidden, fmt, ranks=8), 3
    ctx, nxt = H.make_ctx(w, me), H.make_ctx(w, me)
    toks, recs = [], []
    for p in range(w.n_ranks):
        tk = W.topk_ids(w, 12, p)
        x, sc = W.payload_rows(w, 12, p)
        g = H.GpuSend(ctx, tk, x, sc)
        toks.append((tk, x, sc))
        recs.append(H.shrink(g.deliver(me)))
    tk, x, sc = toks[me]
    g = H.GpuSend(ctx, tk, x, sc, prefill=0x5c)
    cap = sum(r["n_rows"] for r in recs) * w.top_k
    table, rv, rv2, send2 = B.peers_table(recs, H.DEV), B.RecvBuffers(ctx, cap), B.RecvBuffers(nxt, cap), B.SendBuffers(nxt, T)
    ctx.mw_unpack_index(table, len(recs), cap, rv.expert_offsets, rv.stats)
    g.buf.packed.fill_(0x5c)
    ctx.mw_stream_step(g.x_d, g.s_d, g.topk_d, g.buf.perm, g.buf.stats, g.buf.packed, g.buf.row_src_token, g.buf.row_topk, len(recs),
                       rv.out_rows, rv.out_scales, cap, rv.out_src_peer, rv.out_src_token, nxt, table, len(recs), cap, rv2.expert_offsets,
                       rv2.stats, g.topk_d, send2.mask, send2.perm, send2.desc, send2.stats)
    torch.cuda.synchronize()
    H.check_send(w, g, tk, x, sc)
    gu = H.GpuUnpack.__new__(H.GpuUnpack)
    gu.ctx, gu.buf, gu.stats = ctx, rv, ctx.mw_get_recv_stats(rv.stats)
    gu.Q = int(gu.stats["n_out_rows"])
    H.check_unpack(gu, ref.dispatch_plain(toks, W.expert_to_rank(w), me, cap), "step")
    ctx.close(), nxt.close()
