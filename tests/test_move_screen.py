"""The 16-bit partner screens of the continuous models (rewl_moves.h, built for
the host) keep every partner within the cut-off of a bead's old or new place,
in boxes of every accepted size: partners are put just inside the cut-off along
the move, where the screen has the least room."""
import ctypes

import numpy as np
import pytest


def screen(lib, box, count, seed):
    rng = np.random.default_rng(seed)
    f32 = np.float32
    box = f32(box)
    o = (rng.random((count, 3)) * float(box)).astype(f32)
    o[o >= box] = 0
    r, r2 = (rng.integers(0, 2**32, (count, 3), dtype=np.uint32) for _ in range(2))
    # displacement of a word: 0.1 (2 u - 1), u of 23 bits
    d = 0.1 * ((r >> 9) * 2.0**-22 - 1.0)
    along = d / np.maximum(np.linalg.norm(d, axis=1, keepdims=True), 1e-9)
    turn = rng.normal(size=(count, 3)) * rng.choice([0.0, 0.02, 3.0], (count, 1))
    u = along + turn
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    from_new = rng.random((count, 1)) < 0.7
    away = 2.5 * (1.0 - np.exp(rng.uniform(np.log(1e-7), np.log(1e-2), (count, 1))))
    q = np.mod(o + np.where(from_new, d, 0.0) + away * u, float(box)).astype(f32)
    q[q >= box] = 0
    kept = np.zeros(count, dtype=np.uint8)
    p = lambda a: np.ascontiguousarray(a).ctypes.data_as(ctypes.c_void_p)
    lib.screen_all.argtypes = [ctypes.c_size_t] + [ctypes.c_void_p] * 4 + [ctypes.c_float, ctypes.c_void_p]
    lib.screen_all.restype = None
    lib.screen_all(count, p(o), p(r), p(q), p(r2), float(box), p(kept))
    return [((kept >> b) & 1).astype(bool) for b in range(6)]


@pytest.mark.parametrize("box", [2.6, 6.0, 10.0, 60.0, 98.0, 200.0, 400.0, 1000.0, 1e4, 1e5, 9.9e5])
def test_no_partner_within_the_cut_off_is_screened_out(kernel_arith, box):
    near_old, near_new, kept, kept_rep, close, near_moved = screen(kernel_arith, box, 2_000_000, 51)
    assert near_old.sum() > 100_000 and near_new.sum() > 100_000
    assert not np.any((near_old | near_new) & ~kept), box
    assert not np.any(near_old & ~kept_rep), box
    assert not np.any((near_old | near_new | near_moved) & ~close), box


@pytest.mark.parametrize("waves", [1, 2, 4, 8, 16])
def test_corrections_are_read_inside_their_table(kernel_arith, waves):
    last = ctypes.c_int64()
    kernel_arith.correction_read.restype = ctypes.c_int64
    for lane in range(64):
        for r in range(16):
            v = kernel_arith.correction_read(lane, waves, r, ctypes.byref(last))
            assert last.value < 16 * waves
            if lane < waves:
                assert v == 16 * lane + r + 1
