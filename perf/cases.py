"""What a rank of a MultiWrite job has this library do, as timed cases.

listed() names the cases, draw() gives more of the same ranges, prepare() makes what a program holds
before the call (inputs and received regions on the GPU, contexts, output buffers), run() is one
pass through the public entry points, work() the bytes a pass cannot do without, tolerance() how far
another correct implementation may be off, exact() the floating results in 64 bits.

Inputs are drawn on the GPU with plain torch: router scores per peer and token, top-k of them as the
expert ids, N(0, 1) rows (fp8 rows are such rows quantised per 128 elements).  A peer's received region
is what the network would leave: the peer's tokens whose destination set names this rank, ordered by
(bitmap, token), one descriptor per distinct bitmap.

Kinds of cases
  decode        mw_plan_pack + mw_unpack: a batch of at most 256 tokens, one in flight
  dispatch      mw_plan + mw_pack + mw_unpack: one batch in flight
  step          two mw_stream_step calls: a steady stream of batches, one launch a batch
  packets       mw_plan + mw_pack_packets + mw_unpack_packets: the bitmap in front of every row
  quantize      mw_plan + mw_pack_quantize: bf16 in, fp8 rows out
  combine       mw_combine_gather: the way back of a dispatch
  relay         mw_relay of a whole sender buffer over a two-level topology (8 ranks a server)
  relay_stream  two mw_relay_copy_index_next calls: one buffer after the other
  relay_packets mw_relay_packets of a sender's packets
  allgather     mw_plan_allgather + mw_pack_allgather + mw_unpack_allgather
  ag_step       mw_allgather_step: the same for a stream, one launch
  ag_split      mw_plan_allgather_split + mw_pack_allgather + mw_unpack_allgather_split
"""
import math

import numpy as np
import torch

from paper_2605_22428_amd import binding as B

DEV = "cuda:0"
SERVER = 8                     # ranks of one server (relay topology, group-limited routing)
LARGEST_BYTES = 2.0e9          # a drawn case moves no more than the largest listed one
LARGEST_SCORES = 256 * 8192 * 256


def _case(name, kind, ranks, experts, top_k, tokens, hidden, fmt="bf16", routing="uniform", line_stride=False,
          stats=True, padded=0):
    return dict(name=name, kind=kind, ranks=ranks, experts=experts, top_k=top_k, tokens=tokens, hidden=hidden,
                format=fmt, routing=routing, line_stride=line_stride, stats=stats, padded=padded)


def _gather_case(name, kind, ranks, shard_bytes):
    return dict(name=name, kind=kind, ranks=ranks, shard_bytes=shard_bytes)


def listed():
    return [
        # the smallest call: 8 ranks, 16 experts, top-2, 128 tokens of 512 bytes; launches and latency
        _case("decode_ep8_tiny", "decode", 8, 16, 2, 128, 256),
        # token generation with 64 tokens a rank over 64 ranks, as a steady stream of micro-batches
        _case("step_ep64_64tok", "step", 64, 256, 8, 64, 7168, routing="nodes"),
        # the paper's dispatch workload (16 devices, 64 experts, top-8) at a ragged thousand fp8 tokens; a
        # program that never reads the statistics back
        _case("dispatch_ep16_1000tok_fp8", "dispatch", 16, 64, 8, 1000, 4096, "fp8", stats=False),
        # prefill over 64 ranks with fp8 rows a whole number of cache lines apart, one batch in flight
        _case("dispatch_ep64_4096tok_fp8", "dispatch", 64, 256, 8, 4096, 7168, "fp8", "nodes", line_stride=True),
        # prefill over 64 ranks, bf16, steady stream: the largest
        _case("step_ep64_4096tok", "step", 64, 256, 8, 4096, 7168, routing="nodes"),
        # one node of 8 GPUs, 32 experts on each: few peers, many rows from each, several experts a row
        _case("step_ep8_2048tok", "step", 8, 256, 8, 2048, 7168),
        # 256 ranks, one expert each, skewed popularity: four-word bitmaps
        _case("dispatch_ep256_8192tok_zipf", "dispatch", 256, 256, 8, 8192, 7168, routing="zipf"),
        # self-describing rows (bitmap and ids in a header), the paper's 2k batch
        _case("packets_ep16_2048tok", "packets", 16, 64, 8, 2048, 4096),
        # the way back on one node of 8 GPUs: several expert outputs summed into one returned row
        _case("combine_ep8_4096tok", "combine", 8, 256, 8, 4096, 7168),
        # the send side with quantisation to fp8 inside the packer
        _case("quantize_ep64_4096tok", "quantize", 64, 256, 8, 4096, 7168, "fp8", "nodes"),
        # a relay node: a whole sender buffer split over 15 next hops
        _case("relay_ep64_4096tok", "relay", 64, 256, 8, 4096, 7168, routing="nodes"),
        # AllGather of 16 MiB a rank on one node of 8, as a stream
        _gather_case("ag_step_8x16MiB", "ag_step", 8, 16 << 20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choice(["decode", "decode", "dispatch", "dispatch", "dispatch", "step", "step", "step", "packets", "quantize",
                       "combine", "relay", "relay_stream", "relay_packets", "gather"])
    if kind == "gather":
        ranks = rng.choice([2, 4, 8, 8, 16, 64, 128])
        shard = _log_int(rng, 4 << 10, 200 << 20) // 16 * 16
        return dict(kind=rng.choice(["allgather", "ag_step", "ag_split"]), ranks=ranks, shard_bytes=shard)
    if kind.startswith("relay"):
        ranks = rng.choice([16, 16, 32, 64, 64, 128])
    else:
        ranks = rng.choice([4, 8, 8, 8, 12, 16, 16, 24, 32, 48, 64, 64, 72, 96, 128, 144, 256])
    experts = rng.choice([e for e in (16, 60, 64, 128, 160, 256, 384) if e >= ranks] or [ranks])
    top_k = rng.choice([k for k in (1, 2, 4, 6, 8, 8, 8, 9, 12) if k <= experts])
    fmt = "fp8" if kind == "quantize" or (kind != "combine" and rng.random() < 0.4) else "bf16"
    hidden = rng.choice([1024, 2048, 4096, 5120, 6144, 7168, 8192] + ([512, 3584] if fmt == "fp8" else [2880, 328]))
    tokens = _log_int(rng, 1, 256) if kind == "decode" else _log_int(rng, 16, 8192 if kind == "step" else 16384)
    routing = rng.choice(["uniform", "uniform", "zipf", "nodes"])
    if routing == "nodes" and (ranks % SERVER or ranks < 16 or experts % ranks or top_k > 8):
        routing = "uniform"
    return dict(kind=kind, ranks=ranks, experts=experts, top_k=top_k, tokens=tokens, hidden=hidden, format=fmt,
                routing=routing, line_stride=fmt == "fp8" and rng.random() < 0.5, stats=rng.random() < 0.7,
                padded=rng.choice([0, 0, 0, 10]))


def draw(rng):
    while True:
        c = _draw_once(rng)
        if work(c)["bytes"] > LARGEST_BYTES:
            continue
        if "tokens" in c and _peers(c) * c["tokens"] * c["experts"] > LARGEST_SCORES:
            continue
        if c["kind"].startswith("relay") and _relay_hops(c)[1] * c["tokens"] * _rows(c)[2] > LARGEST_BYTES:
            continue                                 # a child buffer for a whole batch on every hop
        return c


# ---- what a case consists of -------------------------------------------------------------------
def _peers(c):
    """Simulated senders: all ranks where this rank receives, itself alone where it only sends or relays."""
    return 1 if c["kind"] == "quantize" or c["kind"].startswith("relay") else c["ranks"]


def _rows(c):
    """(bytes of a row's values, bytes of its scales, bytes from row to row)."""
    h = c["hidden"]
    x, s = (2 * h, 0) if c["format"] == "bf16" else (h, 4 * (h // 128))
    stride = -(-(x + s) // 128) * 128 if c["line_stride"] else x + s
    return x, s, stride


def _placement(c):
    """Rank of every expert: contiguous, as even as the counts allow."""
    return np.arange(c["experts"], dtype=np.int64) * c["ranks"] // c["experts"]


def _popularity(c):
    """log weight of every expert (zipf routing): i^-1.1 over a fixed order."""
    e = c["experts"]
    order = np.argsort(np.sin(np.arange(e) * 12.9898 + 4.1414) * 43758.5453 % 1.0, kind="stable")
    logw = np.empty(e)
    logw[order] = -1.1 * np.log(np.arange(1, e + 1))
    return logw, order


def _my_rank(c):
    if c["routing"] == "zipf":                       # the rank of the expert of median popularity
        return int(_placement(c)[_popularity(c)[1][c["experts"] // 2 - 1]])
    return c["ranks"] // 2


def _expected(c):
    """(packed rows, received rows, output rows) this rank handles, in expectation."""
    e, k, p = c["experts"], c["top_k"], _peers(c)
    t = c["tokens"] - c["tokens"] * c["padded"] // 100
    place = _placement(c)
    mine = np.nonzero(place == _my_rank(c))[0]
    if c["routing"] == "zipf":
        w = np.exp(_popularity(c)[0])
        lo, hi = 0.0, 1e12
        for _ in range(200):                         # exponential clocks stopped when k have rung
            mid = (lo + hi) / 2
            lo, hi = (mid, hi) if (1 - np.exp(-w * mid)).sum() < k else (lo, mid)
        pi = 1 - np.exp(-w * lo)
        return t, p * t * (1 - np.prod(1 - pi[mine])), p * t * pi[mine].sum()
    l = len(mine)
    none = math.comb(e - l, k) / math.comb(e, k) if e - l >= k else 0.0
    return t, p * t * (1 - none), p * t * k * l / e


def _capacity(rows):
    """Rows a program makes room for where it expects `rows`."""
    return int(rows * 1.125 + 8 * math.sqrt(rows)) + 64


def _relay_hops(c):
    """Next hop of every rank for a node of server 0: the ranks of its own server one by one, the others by server."""
    r = np.arange(c["ranks"])
    hop = np.where(r // SERVER == 0, r, SERVER + r // SERVER - 1)
    return hop.astype(np.int32), int(hop.max()) + 1


def work(case):
    c = case
    if "shard_bytes" in c:
        s, r = c["shard_bytes"], c["ranks"]
        return {"bytes": 2.0 * s * r + 2.0 * s, "flops": 0}
    x, s, _ = _rows(c)
    rb, k, t = x + s, c["top_k"], c["tokens"]
    n, m, q = _expected(c)
    meta = 4 + 4 * k
    plan = t * 4 * k + t * 32 + n * 4 + n * 48
    if c["kind"] == "quantize":
        return {"bytes": plan + n * (2 * c["hidden"] + rb + meta), "flops": 4.0 * n * c["hidden"]}
    if c["kind"] == "combine":
        return {"bytes": q * x + m * x + m * 32, "flops": float(q) * c["hidden"]}
    if c["kind"].startswith("relay"):
        hops = _relay_hops(c)[0]
        per = np.bincount(hops, minlength=hops.max() + 1) * (c["experts"] / c["ranks"])     # experts behind a hop
        e = c["experts"]
        copies = sum(1 - math.exp(math.lgamma(e - v + 1) - math.lgamma(e - v - k + 1) - math.lgamma(e + 1) +
                                  math.lgamma(e - k + 1)) if e - v >= k else 1.0 for v in per if v > 0)
        if c["routing"] == "nodes":                  # at most four servers a token, k / 4 experts on each
            nodes = c["ranks"] // SERVER
            few = min(4, nodes)
            copies = few * (nodes - 1) / nodes + few / nodes * SERVER * (1 - (1 - 1 / SERVER) ** (k / few))
        one = n * (1 + copies) * (rb + meta + 48)
        return {"bytes": one * (2 if c["kind"] == "relay_stream" else 1), "flops": 0}
    recv = m * (rb + meta + 48) + q * (rb + 8)
    one = plan + n * (2 * rb + meta) + recv
    if c["kind"] == "packets":
        one = plan + n * (2 * rb + B.mw_packet_header_bytes(k)) + m * (rb + B.mw_packet_header_bytes(k)) + q * (rb + 8)
    return {"bytes": one * (2 if c["kind"] == "step" else 1), "flops": 0}


def tolerance(case):
    # rows, indices and codes are moved or decided in whole bytes; the combine's sums and the scales
    # have a fixed order and one rounding per operation, so every correct result has the same bits
    return "exact"


# ---- inputs -------------------------------------------------------------------------------------
def _generator(seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1000003 + tag) % (1 << 62))
    return g


def _ids(c, seed, batch):
    """int32 [peers][tokens][top_k]: every peer's expert ids as its gate emits them (-1: padded token)."""
    p, t, e, k = _peers(c), c["tokens"], c["experts"], c["top_k"]
    g = _generator(seed, 11 + batch)
    out = torch.empty((p, t, k), dtype=torch.int32, device=DEV)
    flat, step = out.view(p * t, k), max(1, (1 << 26) // e)
    for lo in range(0, p * t, step):
        n = min(step, p * t - lo)
        score = torch.randn((n, e), generator=g, device=DEV)
        if c["routing"] == "zipf":
            score = torch.rand((n, e), generator=g, device=DEV).clamp_(1e-7, 1 - 1e-7)
            score = torch.from_numpy(_popularity(c)[0]).float().to(DEV) - torch.log(-torch.log(score))
        elif c["routing"] == "nodes":                # at most four servers a token, by their two best experts
            nodes = c["ranks"] // SERVER
            prob = torch.softmax(score, 1).view(n, nodes, e // nodes)
            best = prob.topk(2, dim=2).values.sum(2).topk(min(4, nodes), dim=1).indices
            allowed = torch.zeros((n, nodes), dtype=torch.bool, device=DEV).scatter_(1, best, True)
            score = torch.where(allowed[:, :, None], prob, -1.0).view(n, e)
        flat[lo:lo + n] = score.topk(k, dim=1).indices.int()
    pad = t * c["padded"] // 100
    if pad:
        out[:, t - pad:] = -1
    return out


def _masks(c, ids):
    """int64 [peers][tokens][4]: the destination bitmaps, and whether a token has any destination."""
    place = torch.from_numpy(_placement(c)).to(DEV)
    rank = torch.where(ids >= 0, place[ids.clamp(min=0).long()], -1)
    m = torch.zeros((ids.shape[0], ids.shape[1], 4), dtype=torch.int64, device=DEV)
    for j in range(ids.shape[2]):
        r = rank[:, :, j]
        bit = torch.where(r >= 0, torch.ones_like(r) << (r & 63), 0)
        for w in range((c["ranks"] + 63) // 64):
            m[:, :, w] |= torch.where(r >> 6 == w, bit, 0)
    return m


def _packed_order(c, mask):
    """[peers][tokens]: the tokens in (bitmap as an unsigned number, token) order."""
    order = torch.arange(mask.shape[1], device=DEV).expand(mask.shape[0], -1)
    for w in range((c["ranks"] + 63) // 64):
        key = mask[:, :, w].gather(1, order) ^ torch.iinfo(torch.int64).min
        order = order.gather(1, key.sort(dim=1, stable=True).indices)
    return order


def _values(c, seed, tag, n):
    """n rows of N(0, 1) values: (uint8 [n][value bytes], float32 [n][hidden / 128] or None)."""
    g, h = _generator(seed, tag), c["hidden"]
    if c["format"] == "bf16":
        return torch.randn((n, h), generator=g, dtype=torch.bfloat16, device=DEV).view(torch.uint8), None
    codes = torch.empty((n, h), dtype=torch.uint8, device=DEV)
    scales = torch.empty((n, h // 128), dtype=torch.float32, device=DEV)
    step = max(1, (1 << 27) // h)
    for lo in range(0, n, step):
        v = torch.randn((min(step, n - lo), h // 128, 128), generator=g, device=DEV)
        s = v.abs().amax(2).clamp_(min=1e-6) / 448.0
        scales[lo:lo + step] = s
        codes[lo:lo + step] = (v / s[:, :, None]).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8).view(-1, h)
    return codes, scales


def _wire_rows(c, values, scales):
    """Rows as they lie in a packed buffer: values, then scales, then the gap to the next row."""
    x, s, stride = _rows(c)
    if scales is None and stride == x:
        return values
    rows = torch.zeros((values.shape[0], stride), dtype=torch.uint8, device=DEV)
    rows[:, :x] = values
    if scales is not None:
        rows[:, x:x + s] = scales.view(torch.uint8)
    return rows


class _Region:
    """The rows of every peer's packed order that `keep` [peers][tokens] selects, with their metadata."""

    def __init__(self, c, seed, batch, ids, mask, keep):
        order = _packed_order(c, mask)
        kept = keep.gather(1, order)
        self.peer, pos = kept.nonzero(as_tuple=True)
        self.token = order[self.peer, pos]
        self.counts = kept.sum(1).tolist()
        n = len(self.peer)
        self.mask = mask[self.peer, self.token]
        self.topk = ids[self.peer, self.token].contiguous()
        self.src_token = self.token.int()
        self.values, self.scales = _values(c, seed, 31 + batch, n)
        first = torch.ones(n, dtype=torch.bool, device=DEV)
        if n > 1:
            first[1:] = (self.mask[1:] != self.mask[:-1]).any(1) | (self.peer[1:] != self.peer[:-1])
        start = first.nonzero().view(-1)
        length = torch.diff(start, append=torch.tensor([n], device=DEV))
        base = torch.zeros(len(self.counts) + 1, dtype=torch.int64, device=DEV)
        base[1:] = torch.tensor(self.counts, device=DEV).cumsum(0)
        desc = torch.zeros((max(len(start), 1), 6), dtype=torch.int64, device=DEV)
        if n:
            g_peer = self.peer[start]
            place = torch.from_numpy(_placement(c)).to(DEV)
            ranks = place[self.topk[start].long()].sort(1).values
            n_dest = 1 + (ranks[:, 1:] != ranks[:, :-1]).sum(1)
            desc[:, :4] = self.mask[start]
            desc[:, 4] = (start - base[g_peer]) | (length << 32)
            desc[:, 5] = n_dest
            self.groups = torch.bincount(g_peer, minlength=len(self.counts)).tolist()
        else:
            self.groups = [0] * len(self.counts)
        self.desc = desc.view(torch.uint8)

    def records(self, c):
        rows = _wire_rows(c, self.values, self.scales)
        self.rows = rows if len(rows) else torch.zeros((1, _rows(c)[2]), dtype=torch.uint8, device=DEV)
        out, g, r = [], 0, 0
        for n_desc, n_rows in zip(self.groups, self.counts):
            out.append(dict(desc=self.desc[g:], n_desc=n_desc, n_rows=n_rows, rows=self.rows[r:],
                            row_src_token=self.src_token[r:], row_topk=self.topk[r:]))
            g, r = g + n_desc, r + n_rows
        return out

    def packets(self, c):
        x, s, _ = _rows(c)
        hb, k, n = B.mw_packet_header_bytes(c["top_k"]), c["top_k"], len(self.peer)
        pk = torch.zeros((max(n, 1), hb + x + s), dtype=torch.uint8, device=DEV)
        if n:
            head = torch.zeros((n, hb // 4), dtype=torch.int32, device=DEV)
            head[:, :8] = self.mask.view(torch.int32)
            head[:, 8], head[:, 9], head[:, 10:10 + k] = self.src_token, k, self.topk
            pk[:, :hb], pk[:, hb:hb + x] = head.view(torch.uint8), self.values
            if s:
                pk[:, hb + x:] = self.scales.view(torch.uint8)
        return pk


def _output_rows(c, region):
    """Where the receive side puts the rows: (output row, region row) of every (row, local expert) pair."""
    mine = torch.zeros(c["experts"] + 1, dtype=torch.bool, device=DEV)
    mine[:-1] = torch.from_numpy(_placement(c) == _my_rank(c)).to(DEV)
    row, col = mine[region.topk.long()].nonzero(as_tuple=True)      # (id -1 looks at the last entry)
    expert = region.topk[row, col].long()
    key = (expert * c["ranks"] + region.peer[row]) * 65536 + region.token[row]
    order = key.argsort()
    return row[order]


def _context(c, max_hops=0):
    fmt = B.MW_ROW_BF16 if c["format"] == "bf16" else B.MW_ROW_FP8_E4M3_BLOCK128
    return B.Context(c["ranks"], c["experts"], c["top_k"], 0 if max_hops else _my_rank(c), c["hidden"], fmt, c["tokens"],
                     _peers(c) * c["tokens"], _placement(c).astype(np.int32), device=DEV, max_hops=max_hops,
                     row_stride=_rows(c)[2])


class _Batch:
    """One batch of this rank: its own tokens to send and, where it receives, the peers' regions."""

    def __init__(self, c, seed, batch, ctx, receives=True, packets=False):
        ids = _ids(c, seed, batch)
        own = _my_rank(c) if len(ids) > 1 else 0
        self.topk = ids[own].clone()
        self.x, self.scales = _values(c, seed, 21 + batch, c["tokens"])
        self.send = B.SendBuffers(ctx, c["tokens"])
        if not receives:
            return
        mask, me = _masks(c, ids), _my_rank(c)
        self.region = _Region(c, seed, batch, ids, mask, (mask[:, :, me >> 6] >> (me & 63)) & 1 == 1)
        if packets:
            pk = self.region.packets(c)
            first = np.concatenate([[0], np.cumsum(self.region.counts)])
            self.table = B.packets_table([pk[min(int(f), len(pk) - 1):] for f in first[:-1]], self.region.counts, DEV)
            self.keep = pk
        else:
            self.table = B.peers_table(self.region.records(c), DEV)
        self.capacity = _capacity(_expected(c)[2])
        self.recv = B.RecvBuffers(ctx, self.capacity)

    def sent(self):
        s = self.send
        return dict(mask=s.mask, perm=s.perm, desc=s.desc, send_stats=s.stats, packed=s.packed.view(torch.int32),
                    row_src_token=s.row_src_token, row_topk=s.row_topk)

    def received(self):
        r = self.recv
        out = dict(rows=r.out_rows.view(torch.int32), peer=r.out_src_peer, token=r.out_src_token, offsets=r.expert_offsets,
                   recv_stats=r.stats)
        if r.out_scales is not None:
            out["scales"] = r.out_scales.view(torch.int32)
        return out


def _read_back(c, ctx, batch):
    """A program that reads an earlier batch's statistics (row counts) has done so before this one."""
    ctx.mw_unpack_index(batch.table, c["ranks"], batch.capacity, batch.recv.expert_offsets, batch.recv.stats)
    if c["stats"]:
        ctx.mw_get_recv_stats(batch.recv.stats)


# ---- states -------------------------------------------------------------------------------------
def prepare(case, seed):
    c = case
    kind = c["kind"]
    if "shard_bytes" in c:
        return _prepare_gather(c, seed)
    if kind.startswith("relay"):
        return _prepare_relay(c, seed)
    if kind == "quantize":
        ctx = _context(c)
        b = _Batch(dict(c, format="bf16"), seed, 0, ctx, receives=False)
        return dict(kind=kind, ctx=ctx, b=b, codes=b.send.packed[:, :c["hidden"]],
                    scales=b.send.packed[:, c["hidden"]:c["hidden"] + c["hidden"] // 32].view(torch.float32))
    if kind == "step":
        ctxs = [_context(c), _context(c)]
        bs = [_Batch(c, seed, i, ctxs[i]) for i in range(2)]
        for ctx, b in zip(ctxs, bs):
            _read_back(c, ctx, b)
        s = bs[0].send
        ctxs[0].mw_plan(bs[0].topk, s.mask, s.perm, s.desc, s.stats)
        calls = []
        for i in range(2):
            b, n, nc = bs[i], bs[1 - i], ctxs[1 - i]
            s, r = b.send, b.recv
            calls.append((ctxs[i], B.send_batch(b.x, b.scales, b.topk, s.perm, s.stats, s.packed, s.row_src_token, s.row_topk),
                          B.recv_batch(c["ranks"], r.out_rows, r.out_scales, b.capacity, r.out_src_peer, r.out_src_token),
                          B.next_batch(nc, n.table, c["ranks"], n.capacity, n.recv.expert_offsets, n.recv.stats, n.topk,
                                       n.send.mask, n.send.perm, n.send.desc, n.send.stats)))
        return dict(kind=kind, calls=calls, bs=bs)
    ctx = _context(c)
    b = _Batch(c, seed, 0, ctx, packets=kind == "packets")
    st = dict(kind=kind, ctx=ctx, b=b, ranks=c["ranks"])
    if kind == "packets":
        st["packets"] = torch.zeros((c["tokens"], B.mw_packet_header_bytes(c["top_k"]) + ctx.row_bytes), dtype=torch.uint8,
                                    device=DEV)
        if c["stats"]:
            _unpack_packets(st)
            ctx.mw_get_recv_stats(b.recv.stats)
        return st
    _read_back(c, ctx, b)
    if kind == "combine":
        st["y"] = _values(c, seed, 41, b.capacity)[0]
        st["ret"] = torch.zeros((_capacity(_expected(c)[1]), c["hidden"]), dtype=torch.bfloat16, device=DEV)
    return st


def _prepare_gather(c, seed):
    r, n = c["ranks"], c["shard_bytes"]
    ctx = B.Context(r, 0, 1, 0, 0, B.MW_ROW_BYTES, 1, 1, None, row_bytes=16, device=DEV)
    g = _generator(seed, 51)

    def shard(size):
        return torch.randn(max(size // 2, 8), generator=g, dtype=torch.bfloat16, device=DEV).view(torch.int16)

    def table(ts):
        return torch.tensor([t.data_ptr() for t in ts], dtype=torch.int64, device=DEV)

    st = dict(kind=c["kind"], ctx=ctx, n=n, own=shard(n), send=torch.zeros(n // 2, dtype=torch.int16, device=DEV),
              desc=torch.zeros((2, B.DESC_BYTES), dtype=torch.uint8, device=DEV),
              stats=torch.zeros(B.SEND_STATS_BYTES, dtype=torch.uint8, device=DEV),
              out=torch.zeros((r, n // 2), dtype=torch.int16, device=DEV))
    if c["kind"] == "ag_split":                      # the relayed half crosses a link as fast as the direct one
        st["direct"] = B.mw_allgather_split_point(n, 1.0, 1.0, 1)
        st["keep"] = [[shard(st["direct"]) for _ in range(r)], [shard(n - st["direct"]) for _ in range(r)]]
        st["tables"] = [table(t) for t in st["keep"]]
    else:
        st["keep"] = [shard(n) for _ in range(r)]
        st["table"] = table(st["keep"])
    return st


def _prepare_relay(c, seed):
    hops, n_hops = _relay_hops(c)
    x, s, stride = _rows(c)
    packets = c["kind"] == "relay_packets"
    jobs = []
    for i in range(2 if c["kind"] == "relay_stream" else 1):
        ctx = _context(c, max_hops=n_hops)
        ctx.mw_set_forwarding(hops, n_hops)
        ids = _ids(c, seed, i)
        mask = _masks(c, ids)
        region = _Region(c, seed, i, ids, mask, (mask != 0).any(2))
        stats = torch.zeros(B.RELAY_STATS_BYTES, dtype=torch.uint8, device=DEV)
        t, k = c["tokens"], c["top_k"]
        if packets:
            pk = region.packets(c)
            out = dict(packets=torch.zeros((n_hops, t, pk.shape[1]), dtype=torch.uint8, device=DEV))
            record = B.packets_table([pk], region.counts, DEV)
            table = torch.tensor([o.data_ptr() for o in out["packets"]], dtype=torch.int64, device=DEV)
        else:
            pk = region.records(c)
            record = B.peers_table(pk, DEV)
            out = dict(desc=torch.zeros((n_hops, t, B.DESC_BYTES), dtype=torch.uint8, device=DEV),
                       rows=torch.zeros((n_hops, t, stride), dtype=torch.uint8, device=DEV),
                       row_src_token=torch.full((n_hops, t), -1, dtype=torch.int32, device=DEV),
                       row_topk=torch.zeros((n_hops, t, k), dtype=torch.int32, device=DEV))
            host = np.zeros(n_hops, dtype=B.RELAY_CHILD_DTYPE)
            for h in range(n_hops):
                host[h] = tuple(out[f][h].data_ptr() for f in ("desc", "rows", "row_src_token", "row_topk"))
            table = torch.from_numpy(host.view(np.uint8).reshape(-1)).to(DEV)
        jobs.append(dict(ctx=ctx, record=record, table=table, cap=t, stats=stats, out=out, keep=(region, pk)))
    if len(jobs) == 2:
        a = jobs[0]
        a["ctx"].mw_relay_index(a["record"], a["table"], a["cap"], a["stats"])
    return dict(kind=c["kind"], jobs=jobs)


# ---- one pass -----------------------------------------------------------------------------------
def _unpack(st):
    b, r = st["b"], st["b"].recv
    st["ctx"].mw_unpack(b.table, st["ranks"], r.out_rows, r.out_scales, b.capacity, r.out_src_peer, r.out_src_token,
                        r.expert_offsets, r.stats)


def _unpack_packets(st):
    b, r = st["b"], st["b"].recv
    st["ctx"].mw_unpack_packets(b.table, st["ranks"], r.out_rows, r.out_scales, b.capacity, r.out_src_peer,
                                r.out_src_token, r.expert_offsets, r.stats)


def run(state):
    st, kind = state, state["kind"]
    if kind == "step":
        for ctx, send, recv, nxt in st["calls"]:
            ctx.mw_stream_step_records(send, recv, nxt)
        return [dict(b.sent(), **b.received()) for b in st["bs"]]
    if kind in ("relay", "relay_packets", "relay_stream"):
        a = st["jobs"][0]
        if kind == "relay":
            a["ctx"].mw_relay(a["record"], a["table"], a["cap"], a["stats"])
        elif kind == "relay_packets":
            a["ctx"].mw_relay_packets(a["record"], a["table"], a["cap"], a["stats"])
        else:
            for a, n in (st["jobs"], st["jobs"][::-1]):
                a["ctx"].mw_relay_copy_index_next(a["record"], a["table"], a["stats"], n["ctx"], n["record"], n["table"],
                                                  n["cap"], n["stats"])
        return [dict({name: o.view(torch.int32) for name, o in j["out"].items()}, stats=j["stats"]) for j in st["jobs"]]
    ctx = st["ctx"]
    if kind == "allgather":
        ctx.mw_plan_allgather(st["n"], st["desc"], st["stats"])
        ctx.mw_pack_allgather(st["own"], st["n"], st["send"])
        ctx.mw_unpack_allgather(st["table"], st["n"], st["out"])
        return [st["desc"], st["stats"], st["send"], st["out"]]
    if kind == "ag_step":
        ctx.mw_allgather_step(st["own"], st["n"], st["send"], st["desc"], st["stats"], st["table"], st["out"])
        return [st["desc"], st["stats"], st["send"], st["out"]]
    if kind == "ag_split":
        ctx.mw_plan_allgather_split(st["n"], st["direct"], st["desc"], st["stats"])
        ctx.mw_pack_allgather(st["own"], st["n"], st["send"])
        ctx.mw_unpack_allgather_split(st["tables"][0], st["tables"][1], st["n"], st["direct"], st["out"])
        return [st["desc"], st["stats"], st["send"], st["out"]]
    b = st["b"]
    s = b.send
    if kind == "combine":
        ctx.mw_combine_gather(st["ranks"], st["y"], b.capacity, st["ret"], st["ret"].shape[0])
        return dict(ret=st["ret"])
    if kind == "decode":
        ctx.mw_plan_pack(b.topk, b.x, b.scales, s.mask, s.perm, s.desc, s.stats, s.packed, s.row_src_token, s.row_topk)
        _unpack(st)
        return dict(b.sent(), **b.received())
    ctx.mw_plan(b.topk, s.mask, s.perm, s.desc, s.stats)
    if kind == "quantize":
        ctx.mw_pack_quantize(b.x, b.topk, s.perm, s.stats, s.packed, s.row_src_token, s.row_topk)
        out = b.sent()
        del out["packed"]
        return dict(out, codes=st["codes"], scales=st["scales"])
    if kind == "packets":
        ctx.mw_pack_packets(b.x, b.scales, b.topk, s.mask, s.perm, s.stats, st["packets"])
        _unpack_packets(st)
        out = dict(b.sent(), **b.received())
        for name in ("packed", "row_src_token", "row_topk"):
            del out[name]
        return dict(out, packets=st["packets"].view(torch.int32))
    ctx.mw_pack(b.x, b.scales, b.topk, s.perm, s.stats, s.packed, s.row_src_token, s.row_topk)
    _unpack(st)
    return dict(b.sent(), **b.received())


def exact(case, seed):
    c = case
    if c["kind"] == "combine":
        ids = _ids(c, seed, 0)
        mask, me = _masks(c, ids), _my_rank(c)
        region = _Region(c, seed, 0, ids, mask, (mask[:, :, me >> 6] >> (me & 63)) & 1 == 1)
        row = _output_rows(c, region)
        y = _values(c, seed, 41, _capacity(_expected(c)[2]))[0].view(torch.bfloat16)[: len(row)]
        out = torch.zeros((_capacity(_expected(c)[1]), c["hidden"]), dtype=torch.float64, device=DEV)
        return dict(ret=out.index_add_(0, row, y.double()))
    if c["kind"] == "quantize":
        ids = _ids(c, seed, 0)
        mask = _masks(c, ids)
        order = _packed_order(c, mask)[0]
        order = order[(mask != 0).any(2)[0][order]]
        x = _values(dict(c, format="bf16"), seed, 21, c["tokens"])[0].view(torch.bfloat16).double()
        scale = x.view(len(x), -1, 128).abs().amax(2).clamp(min=2.0 ** -20) / 448.0
        out = torch.zeros_like(scale)
        out[: len(order)] = scale[order]
        return dict(mask=None, perm=None, desc=None, send_stats=None, row_src_token=None, row_topk=None, codes=None,
                    scales=out)
    return None
