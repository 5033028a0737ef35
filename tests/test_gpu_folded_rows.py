"""GPU parity of the packer and the expander where a row's last few chunks go to the lanes of its first wave: one chunk and
sixteen too many for whole waves, seventeen (a wave of their own), ten waves and a few (not folded), the largest row of one workgroup
and the first beyond; fp8 rows, whose scales are those chunks; and the same widths in steps of a stream too short to fold them
(folded beside riders: test_gpu_riding_index.py).  Bit-exact."""
import numpy as np
import pytest

from oracle import ref
from paper_2605_22428_amd import workloads as W

import gpu_harness as H
import test_gpu_index_forms as forms

pytestmark = pytest.mark.gpu


def _dispatch(w, my_rank):
    e2r, ctx = W.expert_to_rank(w), H.make_ctx(w, my_rank)
    toks, recs = [], []
    for p in range(w.n_ranks):
        tk = W.topk_ids(w, 3, p)
        x, sc = W.payload_rows(w, 3, p)
        g = H.GpuSend(ctx, tk, x, sc, prefill=0x5c)
        H.check_send(w, g, tk, x, sc)
        toks.append((tk, x, sc))
        recs.append(H.shrink(g.deliver(my_rank)))
    cap = max(1, sum(r["n_rows"] for r in recs) * w.top_k)
    want = ref.dispatch_plain(toks, e2r, my_rank, cap)
    H.check_unpack(H.GpuUnpack(ctx, recs, cap), want, "unpack")
    ctx.close()


@pytest.mark.parametrize("chunks", [64, 65, 80, 81, 128, 129, 144, 145, 257, 264, 272, 273, 330, 513, 528, 641, 655, 1024, 1025, 1039, 1041])
def test_rows_of_whole_waves_and_a_few_chunks(chunks):
    print("folded rows", chunks, flush=True)
    _dispatch(W.DispatchWorkload("fold", 76, 4, 16, 4, 150, 8 * chunks, "bf16", "uniform"), 1)


@pytest.mark.parametrize("hidden", [512, 1024, 2048, 3584, 4096, 5120, 7168, 8192])
def test_fp8_rows(hidden):
    print("folded fp8 rows", hidden, flush=True)
    _dispatch(W.DispatchWorkload("fold8", 77, 4, 16, 4, 150, hidden, "fp8", "uniform"), 2)


@pytest.mark.parametrize("chunks", [132, 257, 272, 273, 527])
@pytest.mark.parametrize("R,E,K", [(4, 16, 4), (4, 16, 9), (130, 260, 8)])
def test_stream_steps(chunks, R, E, K):
    forms.test_stream_steps_with_riders_and_without(R, E, 300, K, 8 * chunks, True)
