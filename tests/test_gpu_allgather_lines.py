"""GPU parity of the AllGather copies with shards that are no whole number of cache lines: pieces begin on the destination's lines, so
every shard after the first, and a send buffer anywhere, has a short first piece.  Around a piece's 64 chunks, in one call, as a
step and from two pieces; what lies in front of and behind the destination stays as it is."""
import pytest
import torch

from paper_2605_22428_amd import binding as B

import gpu_harness as H

pytestmark = pytest.mark.gpu
GUARD = 64                                           # chunks in front of and behind a destination


def _between(n, first):
    """A destination of n chunks that begins `first` chunks into a cache line, and all of its allocation."""
    whole = torch.full(((n + 2 * GUARD + 8), 16), 0xa5, dtype=torch.uint8, device=H.DEV)
    at = GUARD + (first - (whole.data_ptr() // 16 + GUARD)) % 8
    return whole, at


def _check(whole, at, want, what):
    n = want.shape[0]
    assert torch.equal(whole[at: at + n], want), what
    assert bool((whole[:at] == 0xa5).all()) and bool((whole[at + n:] == 0xa5).all()), what + ": bytes outside were written"


@pytest.mark.parametrize("R", [1, 3, 9])
@pytest.mark.parametrize("chunks", [1, 7, 8, 56, 57, 58, 63, 64, 65, 120, 121, 128, 1001])
def test_shards_of_any_length(R, chunks):
    print("allgather lines", R, chunks, flush=True)
    g = torch.Generator(device=H.DEV).manual_seed(chunks * 16 + R)
    ctx = B.Context(R, 0, 1, 0, 0, B.MW_ROW_BYTES, 1, 1, None, row_bytes=16, device=H.DEV)
    shards = [torch.randint(0, 256, (chunks, 16), generator=g, dtype=torch.uint8, device=H.DEV) for _ in range(R)]
    own = torch.randint(0, 256, (chunks, 16), generator=g, dtype=torch.uint8, device=H.DEV)
    table = torch.tensor([s.data_ptr() for s in shards], dtype=torch.int64, device=H.DEV)
    desc, stats = (torch.zeros((2, B.DESC_BYTES), dtype=torch.uint8, device=H.DEV), torch.zeros(B.SEND_STATS_BYTES, dtype=torch.uint8, device=H.DEV))
    want, n = torch.cat(shards), 16 * chunks
    ctx.mw_plan_allgather(n, desc, stats)
    plan = (desc.clone(), stats.clone())
    for first in (0, 1, 5, 7):
        out, at = _between(R * chunks, first)
        send, sat = _between(chunks, (first * 3) % 8)
        ctx.mw_unpack_allgather(table, n, out[at:])
        ctx.mw_pack_allgather(own, n, send[sat:])
        _check(out, at, want, "assembly")
        _check(send, sat, own, "copy")
        out, at = _between(R * chunks, first)
        send, sat = _between(chunks, (first * 3) % 8)
        desc.zero_(), stats.zero_()
        ctx.mw_allgather_step(own, n, send[sat:], desc, stats, table, out[at:])
        _check(out, at, want, "step, assembly")
        _check(send, sat, own, "step, copy")
        assert torch.equal(desc, plan[0]) and torch.equal(stats, plan[1]), "step, plan"
        d = chunks // 3
        pieces = [[s[:d].contiguous() if d else own for s in shards], [s[d:].contiguous() for s in shards]]
        tables = [torch.tensor([t.data_ptr() for t in p], dtype=torch.int64, device=H.DEV) for p in pieces]
        out, at = _between(R * chunks, first)
        ctx.mw_unpack_allgather_split(tables[0], tables[1], n, 16 * d, out[at:])
        _check(out, at, want, "two pieces")
    ctx.close()
