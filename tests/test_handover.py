"""The hand-over of drawn blocks between two wavefronts (rewl_handover.h, built
for the host): between two barriers no record is both written and read, and the
block read from a record is the last one written there before the last barrier."""
import ctypes

import numpy as np
import pytest


@pytest.mark.parametrize("n", [0, 1, 63, 64, 65, 128, 129, 192, 193, 256, 1000, 10_000])
def test_records_are_read_before_they_are_written_again(kernel_arith, n):
    blocks = (n + 63) // 64
    room = blocks + 4
    written, read = np.zeros((room, 3), dtype=np.int64), np.zeros((room, 3), dtype=np.int64)
    out = np.zeros(4, dtype=np.int64)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    kernel_arith.handover_trace.argtypes = [ctypes.c_int64, ctypes.c_size_t] + [ctypes.c_void_p] * 3
    kernel_arith.handover_trace.restype = None
    kernel_arith.handover_trace(n, room, p(written), p(read), p(out))
    written, read = written[:out[0]], read[:out[1]]
    assert out[2] == out[3]                                  # both sides meet at every barrier
    assert sorted(written[:, 2]) == list(range(blocks))      # each block is drawn once
    last = {}
    order = sorted([(t, 0, s, b) for t, s, b in written.tolist()] + [(t, 1, s, b) for t, s, b in read.tolist()])
    busy = {(t, s) for t, s, _ in written.tolist()}
    for t, is_read, s, b in order:
        if not is_read:
            last[s] = (t, b)
            continue
        assert (t, s) not in busy, (n, t, s, b)              # never in the same interval
        if b < blocks:
            assert last[s][1] == b and last[s][0] < t, (n, t, s, b)
    assert [b for _, _, b in read.tolist() if b < blocks] == list(range(blocks))
