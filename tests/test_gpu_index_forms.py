"""GPU parity of the receive index where its form changes: experts spread over several workgroups a
peer and over several passes of one, id lists that are not whole 16-byte units or do not start on
one, more than eight ids, more than 64 local experts, more experts than the table in LDS holds, the
largest batch; on its own, riding beside the expander, from packets, and dropping repeated rows.
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
    "parts_and_passes": (2, 128, 8, 8192, 1),      # riding: more chunks of experts than workgroups a peer
    "sixty_four_local": (4, 256, 8, 300, 2),
    "sixty_five_local": (1, 65, 8, 400, 0),        # no 64-bit set of experts
    "nine_ids": (8, 64, 9, 700, 7),
    "six_ids": (8, 64, 6, 700, 0),                 # ids word by word
    "one_id": (16, 64, 1, 333, 5),
    "table_in_memory": (100, 3000, 4, 300, 99),    # riding: no room for the table of slots in LDS
    "many_local": (2, 2000, 4, 500, 1),            # slots do not fit a byte
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
        H.check_unpack(gu, want, "riding")

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
