"""GPU parity of mw_unpack of a few hundred rows, where index and expander are one launch: rows of one segment of 64 chunks, of
one chunk more, of many; fp8 rows; as many rows as lanes and one more than expected; peers of no row; more ids than
eight; regions that are damaged, compared with the two halves (mw_unpack_index, mw_unpack_expand) flag by flag; what it leaves for a
second expander and for the way back; and an output that is too short.  Bit-exact."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2605_22428_amd import binding as B

import gpu_harness as H

pytestmark = pytest.mark.gpu


def _regions(rng, R, E, K, counts, hidden, fmt, ctx, e2r, my_rank):
    mine = np.nonzero(e2r == my_rank)[0]
    toks, recs = [], []
    for n in counts:
        tk = np.argsort(rng.random((n, E)), axis=1)[:, :K].astype(np.int32) if n else np.zeros((0, K), np.int32)
        tk[np.arange(n), rng.integers(0, K, n)] = rng.choice(mine, n)
        tk[rng.random((n, K)) < 0.05] = -1
        if fmt == "bf16":
            x, sc = rng.integers(0, 1 << 16, size=(n, hidden), dtype=np.uint16), None
        else:
            x, sc = rng.integers(0, 256, size=(n, hidden), dtype=np.uint8), rng.random((n, hidden // 128), dtype=np.float32)
        toks.append((tk, x, sc))
        recs.append(H.shrink(H.GpuSend(ctx, tk, x, sc).deliver(my_rank)))
    return toks, recs


def _halves(ctx, recs, cap):
    gu = H.GpuUnpack.__new__(H.GpuUnpack)
    gu.ctx, gu.buf = ctx, B.RecvBuffers(ctx, cap)
    table, b = B.peers_table(recs, H.DEV), gu.buf
    ctx.mw_unpack_index(table, len(recs), cap, b.expert_offsets, b.stats)
    ctx.mw_unpack_expand(len(recs), b.out_rows, b.out_scales, cap, b.out_src_peer, b.out_src_token)
    gu.stats = ctx.mw_get_recv_stats(b.stats)
    gu.Q = int(gu.stats["n_out_rows"])
    return gu


@pytest.mark.parametrize("R,E,K,T,hidden,fmt", [
    (8, 16, 2, 60, 8, "bf16"), (8, 16, 2, 64, 512, "bf16"), (8, 16, 2, 64, 520, "bf16"), (4, 64, 12, 100, 1032, "bf16"),
    (16, 64, 8, 30, 7168, "bf16"), (16, 64, 8, 32, 1024, "fp8"), (8, 512, 8, 50, 3584, "fp8"), (130, 260, 8, 3, 64, "bf16"),
    (256, 512, 4, 2, 256, "bf16"), (1, 64, 64, 512, 64, "bf16"), (3, 1200, 5, 90, 256, "bf16"), (1, 1, 1, 1, 8, "bf16")])
def test_small_unpack(R, E, K, T, hidden, fmt):
    print("small unpack", R, E, K, T, hidden, fmt, flush=True)
    rng = np.random.default_rng(R * E + T)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    my_rank = R // 2
    code = B.MW_ROW_BF16 if fmt == "bf16" else B.MW_ROW_FP8_E4M3_BLOCK128
    ctx = B.Context(R, E, K, my_rank, hidden, code, T, R * T, e2r, device=H.DEV)
    for turn in range(3):
        counts = [T if turn == 2 else (p + turn) % 3 * T // 3 + (p == 0) * (T > 2) for p in range(R)]
        counts = [min(c, T) for c in counts]
        toks, recs = _regions(rng, R, E, K, counts, hidden, fmt, ctx, e2r, my_rank)
        m = sum(r["n_rows"] for r in recs)
        cap = max(1, m * min(K, int((e2r == my_rank).sum())))
        want = ref.dispatch_plain(toks, e2r, my_rank, cap)
        H.check_unpack(H.GpuUnpack(ctx, recs, cap), want, "turn %d" % turn)
        gu = H.GpuUnpack(ctx, recs, cap)                     # (the row count is known now)
        H.check_unpack(gu, want, "turn %d again" % turn)
        second = H.GpuUnpack.__new__(H.GpuUnpack)            # what it left in the context serves a second expander
        second.ctx, second.buf, second.stats, second.Q = ctx, B.RecvBuffers(ctx, cap), gu.stats, gu.Q
        second.buf.expert_offsets.copy_(gu.buf.expert_offsets)
        ctx.mw_unpack_expand(R, second.buf.out_rows, second.buf.out_scales, cap, second.buf.out_src_peer, second.buf.out_src_token)
        torch.cuda.synchronize()
        H.check_unpack(second, want, "second expander")
        if gu.Q > 1:                                         # an output that ends in the middle
            short = gu.Q // 2
            b = B.RecvBuffers(ctx, cap)
            b.out_rows.fill_(0x5a)
            ctx.mw_unpack(B.peers_table(recs, H.DEV), R, b.out_rows, b.out_scales, short, b.out_src_peer, b.out_src_token,
                          b.expert_offsets, b.stats)
            st = ctx.mw_get_recv_stats(b.stats)
            assert int(st["error_flags"]) == B.MW_FLAG_OUT_CAPACITY and int(st["n_out_rows"]) == gu.Q
            H.assert_same_bytes(H.host(b.out_rows)[:short], want[0][:short], "rows in front of the capacity")
            assert (H.host(b.out_rows)[short:].view(np.uint8) == 0x5a).all()
    ctx.close()


@pytest.mark.parametrize("damage", ["id", "token", "offset", "count", "mask", "many", "none_here", "twice"])
def test_damaged_regions_match_the_two_halves(damage):
    print("damage", damage, flush=True)
    R, E, K, T, hidden, my_rank = 8, 32, 4, 60, 64, 5
    rng = np.random.default_rng(7)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    ctx, other = (B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, T, R * T - 100, e2r, device=H.DEV) for _ in range(2))
    toks, recs = _regions(rng, R, E, K, [20] * R, hidden, "bf16", ctx, e2r, my_rank)
    cap = 4 * R * T
    H.check_unpack(H.GpuUnpack(ctx, recs, cap), ref.dispatch_plain(toks, e2r, my_rank, cap), "sound")
    rec = {k: v.clone() if torch.is_tensor(v) else v for k, v in recs[3].items()}
    desc = H.host(rec["desc"]).copy().reshape(-1).view(B.DESC_DTYPE)
    if damage == "id":
        rec["row_topk"][4, 1] = E + 3
    elif damage == "token":
        rec["row_src_token"][2] = T
    elif damage == "offset":
        desc["row_offset"][1] = 1000
    elif damage == "count":
        desc["row_count"][0] = 1 << 20
    elif damage == "mask":
        desc["mask"][2] = 0
    elif damage == "many":
        rec["n_rows"] = rec["n_rows"] - 3
    elif damage == "none_here":
        rec["row_topk"][5] = 0
    elif damage == "twice":
        rec["row_src_token"][1] = rec["row_src_token"][0]
        rec["row_topk"][1] = rec["row_topk"][0]
    rec["desc"] = H.dev(desc.view(np.uint8))
    broken = recs[:3] + [rec] + recs[4:]
    a, b = H.GpuUnpack(ctx, broken, cap), _halves(other, broken, cap)
    for f in ("n_recv_rows", "n_out_rows", "error_flags", "n_rows_seen"):
        assert int(a.stats[f]) == int(b.stats[f]), f
    assert (int(a.stats["error_flags"]) != 0) == (damage != "mask")
    if damage != "twice":                                    # (two rows for one place: either is there)
        for x, y, what in zip(a.host_out(), b.host_out(), ("rows", "scales", "peer", "token", "offsets")):
            if x is not None:
                H.assert_same_bytes(x, y, what)
    H.check_unpack(H.GpuUnpack(ctx, recs, cap), ref.dispatch_plain(toks, e2r, my_rank, cap), "sound again")


def test_events_bracket_the_kernels_they_name():
    """With events set for the receive index mw_unpack of a small batch is two launches again: the index of 12800 rows where 64
    were seen last takes one workgroup tens of microseconds, an empty bracket three."""
    print("timing events", flush=True)
    R, E, K, T, hidden, my_rank = 64, 256, 8, 256, 8, 5
    rng = np.random.default_rng(11)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    ctx = B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, T, R * T, e2r, device=H.DEV)
    _, few = _regions(rng, R, E, K, [1] * R, hidden, "bf16", ctx, e2r, my_rank)
    toks, recs = _regions(rng, R, E, K, [200] * R, hidden, "bf16", ctx, e2r, my_rank)
    cap = sum(r["n_rows"] for r in recs) * 4
    want = ref.dispatch_plain(toks, e2r, my_rank, cap)
    for timed in (False, True, False):
        H.GpuUnpack(ctx, few, cap)                           # (its statistics are read: the next batch is expected to be as small)
        ev = [[torch.cuda.Event(enable_timing=True) for _ in range(2)] for _ in range(2)]
        if timed:
            for kernel, (a, b) in zip((B.MW_KERNEL_RECV_INDEX, B.MW_KERNEL_EXPAND), ev):
                for e in (a, b):
                    e.record()
                ctx.mw_ctx_set_timing_events(kernel, a, b)
        H.check_unpack(H.GpuUnpack(ctx, recs, cap), want, "timed" if timed else "not timed")
        if timed:
            for kernel in (B.MW_KERNEL_RECV_INDEX, B.MW_KERNEL_EXPAND):
                ctx.mw_ctx_set_timing_events(kernel, None, None)
            index, expand = (1e3 * a.elapsed_time(b) for a, b in ev)
            print("index %.1f us, expander %.1f us" % (index, expand), flush=True)
            assert index > 30.0 and expand > 0.0


@pytest.mark.parametrize("hidden", [64, 2048])
def test_a_captured_small_batch_replayed_on_a_larger_one(hidden):
    """A graph captured when the context expected a few rows, replayed on region tables of none, of as many and of a hundred times
    as many."""
    print("captured small unpack", hidden, flush=True)
    R, E, K, T, my_rank = 16, 64, 4, 512, 7
    rng = np.random.default_rng(hidden)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    ctx = B.Context(R, E, K, my_rank, hidden, B.MW_ROW_BF16, T, R * T, e2r, device=H.DEV)
    batches = []
    for n in (3, 0, T, 1):
        toks, recs = _regions(rng, R, E, K, [n] * R, hidden, "bf16", ctx, e2r, my_rank)
        cap = max(1, sum(r["n_rows"] for r in recs) * 4)
        batches.append((recs, B.peers_table(recs, H.DEV), ref.dispatch_plain(toks, e2r, my_rank, cap)))
    buf = B.RecvBuffers(ctx, max(1, 4 * R * T))
    table = batches[0][1].clone()

    def unpack():
        ctx.mw_unpack(table, R, buf.out_rows, buf.out_scales, buf.capacity, buf.out_src_peer, buf.out_src_token, buf.expert_offsets, buf.stats)
    unpack()
    ctx.mw_get_recv_stats(buf.stats)
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        unpack()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=side):
        unpack()
    for recs, other, want in batches + batches[::-1]:
        table.copy_(other)
        buf.out_rows.fill_(0)
        graph.replay()
        torch.cuda.synchronize()
        gu = H.GpuUnpack.__new__(H.GpuUnpack)
        gu.ctx, gu.buf = ctx, buf
        gu.stats = H.host(buf.stats).view(B.RECV_STATS_DTYPE)[0]
        gu.Q = int(gu.stats["n_out_rows"])
        H.check_unpack(gu, want, "replay")
