"""What a context's workspace holds: the arrays of the large-batch plans only where a batch can need them.  No GPU needed."""
import ctypes as C

import numpy as np

from paper_2605_22428_amd import binding as B


def _bytes(max_tokens):
    e2r = np.arange(16, dtype=np.int32) // 2
    cfg = B.MwConfig(8, 16, 2, 0, 256, B.MW_ROW_BF16, 0, max_tokens, 0, 1024, e2r.ctypes.data, 0)
    need = C.c_int64(0)
    assert B.load().mw_workspace_bytes(C.byref(cfg), C.byref(need)) == B.MW_OK
    return need.value


def test_large_batch_arrays_begin_where_batches_need_them():
    # a token more costs its counters, its row map and (up to 8192) its key, each aligned: under 1 KiB without new arrays
    for last in (4096, 8191, 24574):
        assert _bytes(last + 1) - _bytes(last) <= 1024, last
    assert _bytes(8193) - _bytes(8192) >= 9216 * 12             # sorted chunks: key and second word, whole chunks
    assert _bytes(24576) - _bytes(24575) >= 24576 * 9           # counters and start byte of every packed row
