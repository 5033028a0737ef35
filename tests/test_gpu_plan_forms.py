"""GPU parity of mw_plan where its form changes: one, two, four, six and eight tokens a lane, keys made in the
same launch or in one of their own, tokens compared with all others or searched for in sorted chunks, one-word and
byte keys, the batch beyond; empty tokens, one bitmap throughout, few bitmaps, every bit set; an id
outside the range.  Every output against the oracle, bit-exact."""
import numpy as np
import pytest

from oracle import ref
from paper_2605_22428_amd import binding as B

import gpu_harness as H

pytestmark = pytest.mark.gpu

SIZES = [1, 64, 255, 257, 513, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193]
# ranks, experts, top_k: few and many possible destination sets, one-word and byte keys, a byte key's first
# position at 255, one id, more than eight ids with one word, ids that are not whole 16-byte units
SHAPES = [(8, 256, 8), (12, 60, 4), (13, 26, 6), (24, 96, 8), (25, 50, 3), (64, 256, 8), (64, 64, 64), (65, 130, 8),
          (256, 256, 8), (200, 400, 5), (7, 7, 1)]


def _tokens(rng, kind, T, E, K):
    if kind == "same":
        return np.tile(rng.permutation(E)[:K].astype(np.int32), (T, 1))
    if kind == "every":
        return np.argsort(rng.random((T, E)), axis=1)[:, :K].astype(np.int32)
    if kind == "few":
        pool = rng.integers(0, E, size=(5, K)).astype(np.int32)
        return pool[rng.integers(0, 5, size=T)]
    if kind == "ends":                                       # first and last ranks only: shortest and longest keys
        tk = np.where(rng.random((T, K)) < 0.5, 0, E - 1).astype(np.int32)
        tk[rng.random((T, K)) < 0.3] = -1
        return tk
    tk = rng.integers(0, E, size=(T, K)).astype(np.int32)
    tk[rng.random((T, K)) < 0.15] = -1
    tk[rng.random(T) < 0.05] = -1
    if kind == "empty":
        tk[:] = -1
    if kind == "outside":
        tk[T // 2, K - 1] = E
    return tk


@pytest.mark.parametrize("T", SIZES)
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "R%d_E%d_K%d" % s)
def test_plan_forms(shape, T):
    R, E, K = shape
    print("plan form", shape, T, flush=True)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    ctx = B.Context(R, E, K, 0, 8, B.MW_ROW_BF16, T, 1, e2r, device=H.DEV)
    buf = B.SendBuffers(ctx, T)
    rng = np.random.default_rng(T * 1000 + R)
    kinds = ["random", "same", "few", "ends", "empty", "outside", "random"] if T <= 4097 else ["random", "few", "same"]
    if K == E:
        kinds.append("every")
    for kind in kinds:
        tk = _tokens(rng, kind, T, E, K)
        buf.perm.fill_(-7)
        ctx.mw_plan(H.dev(tk), buf.mask, buf.perm, buf.desc, buf.stats)
        st = ctx.mw_get_send_stats(buf.stats)
        outside = (tk < -1) | (tk >= E)
        assert int(st["error_flags"]) == (B.MW_FLAG_BAD_EXPERT if outside.any() else 0), kind
        mask, perm, desc, want = ref.plan(np.where(outside, -1, tk), e2r, R, 16)
        N, G = len(perm), len(desc)
        for f in ("n_rows", "n_groups", "multicast_bytes", "unicast_bytes"):
            assert int(st[f]) == int(want[f]), (kind, f)
        H.assert_same_bytes(st["rows_per_dest"], want["rows_per_dest"], kind + " rows_per_dest")
        H.assert_same_bytes(H.host(buf.mask).view(np.uint64)[:T], mask, kind + " mask")
        got = H.host(buf.perm)
        H.assert_same_bytes(got[:N], perm, kind + " perm")
        assert (got[N:] == -7).all(), kind + ": perm behind the last packed row was written"
        H.assert_same_bytes(H.host(buf.desc).reshape(-1).view(B.DESC_DTYPE)[:G].view(np.uint8), desc.view(np.uint8), kind + " desc")


@pytest.mark.parametrize("T", [1025, 1100, 1300, 1700, 2047])
@pytest.mark.parametrize("R,E,K", [(1, 2, 2), (2, 64, 8), (8, 64, 8), (9, 27, 6), (22, 44, 2), (23, 46, 2), (64, 64, 1), (65, 65, 1),
                                   (256, 512, 1)])
def test_plan_of_few_destination_sets(R, E, K, T):
    """1025 to 2048 tokens around the rule of 256 possible destination sets (8 ranks, eight ids: 255; 22 ranks, two ids: 253; 23:
    276), five to eight tokens a workgroup, which then lie in one wave's 64 tokens or in two; a third of the tokens go nowhere."""
    print("few sets", R, E, K, T, flush=True)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    ctx = B.Context(R, E, K, 0, 8, B.MW_ROW_BF16, T, 1, e2r, device=H.DEV)
    buf = B.SendBuffers(ctx, T)
    rng = np.random.default_rng(T + R)
    for kind in ("random", "some", "ends"):
        tk = _tokens(rng, kind, T, E, K)
        if kind == "some":
            tk[rng.random(T) < 0.3] = -1
        buf.perm.fill_(-7)
        ctx.mw_plan(H.dev(tk), buf.mask, buf.perm, buf.desc, buf.stats)
        st = ctx.mw_get_send_stats(buf.stats)
        mask, perm, desc, want = ref.plan(tk, e2r, R, 16)
        assert (int(st["n_rows"]), int(st["n_groups"]), int(st["error_flags"])) == (len(perm), len(desc), 0)
        H.assert_same_bytes(st["rows_per_dest"], want["rows_per_dest"], "rows_per_dest")
        H.assert_same_bytes(H.host(buf.mask).view(np.uint64)[:T], mask, "mask")
        got = H.host(buf.perm)
        H.assert_same_bytes(got[: len(perm)], perm, "perm")
        assert (got[len(perm):] == -7).all(), "perm behind the last packed row was written"
        H.assert_same_bytes(H.host(buf.desc).reshape(-1).view(B.DESC_DTYPE)[: len(desc)].view(np.uint8), desc.view(np.uint8), "desc")


@pytest.mark.parametrize("T", [2049, 2176, 4095, 6144, 6145, 8065, 8192])
@pytest.mark.parametrize("R,E,K", [(64, 64, 64), (256, 256, 8), (17, 34, 4), (18, 36, 4), (19, 38, 4), (64, 128, 2), (256, 256, 2),
                                   (256, 256, 1), (72, 144, 2)])
def test_plan_of_sorted_chunks(R, E, K, T):
    """Chunks of 128 tokens, a lane's four, six or eight tokens, the last chunk partly filled; keys that appear exactly twice,
    anywhere; every rank named (the largest one-word key) among tokens without a destination; most tokens of two keys.  The
    ranks up to which a bitmap has a bit of its own are 17 (up to 4096 tokens) and 18."""
    print("sorted chunks", R, E, K, T, flush=True)
    e2r = (np.arange(E) * R // E).astype(np.int32)
    ctx = B.Context(R, E, K, 0, 8, B.MW_ROW_BF16, T, 1, e2r, device=H.DEV)
    buf = B.SendBuffers(ctx, T)
    rng = np.random.default_rng(T + R)
    half = np.argsort(rng.random(((T + 1) // 2, E)), axis=1)[:, :K].astype(np.int32)
    twice = np.concatenate([half, half])[rng.permutation(2 * len(half))[:T]]
    if K == E:
        twice[rng.random((T, K)) < 0.5] = -1
    ends = np.tile(np.arange(K, dtype=np.int32) if K == E else np.arange(E - K, E, dtype=np.int32), (T, 1))
    ends[rng.random(T) < 0.4] = -1
    two = np.argsort(rng.random((T, E)), axis=1)[:, :K].astype(np.int32)
    two[rng.random(T) < 0.6] = two[0]
    two[rng.random(T) < 0.3] = two[1]
    for tk in (twice, ends, two):
        ctx.mw_plan(H.dev(tk), buf.mask, buf.perm, buf.desc, buf.stats)
        st = ctx.mw_get_send_stats(buf.stats)
        mask, perm, desc, want = ref.plan(tk, e2r, R, 16)
        assert (int(st["n_rows"]), int(st["n_groups"]), int(st["error_flags"])) == (len(perm), len(desc), 0)
        H.assert_same_bytes(st["rows_per_dest"], want["rows_per_dest"], "rows_per_dest")
        H.assert_same_bytes(H.host(buf.mask).view(np.uint64)[:T], mask, "mask")
        H.assert_same_bytes(H.host(buf.perm)[: len(perm)], perm, "perm")
        H.assert_same_bytes(H.host(buf.desc).reshape(-1).view(B.DESC_DTYPE)[: len(desc)].view(np.uint8), desc.view(np.uint8), "desc")
