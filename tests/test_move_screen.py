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
            assert last.value < kernel_arith.correction_entries(waves)
            if lane < waves:
                assert v == lane * waves + r + 1


LDS = 160 * 1024


def workgroup(lib, used, per_wave, particles, walkers):
    out = (ctypes.c_int64 * 3)()
    lib.move_workgroup.argtypes = [ctypes.c_size_t, ctypes.c_size_t, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    lib.move_workgroup.restype = None
    lib.move_workgroup(used, per_wave, particles, walkers, out)
    return tuple(out)


@pytest.mark.parametrize("particles,walkers,window,waves,grid", [
    (192, 1, 267, 16, 1), (192, 64, 267, 16, 1), (192, 256, 267, 16, 1),
    (192, 257, 267, 8, 1), (192, 512, 267, 8, 1), (192, 513, 267, 4, 1), (192, 1024, 267, 4, 1),
    (192, 1025, 267, 2, 1), (192, 65535, 267, 2, 1),
    (9, 64, 60, 8, 1), (63, 64, 60, 8, 1), (64, 64, 60, 16, 1), (12, 1024, 60, 4, 1),
    (192, 1024, 8000, 16, 1),             # the LDS holds one walker whatever its wavefronts
    (192, 1024, 4500, 8, 1),              # two
    (192, 64, 13000, 8, 0), (48, 64, 13440, 4, 0),
])
def test_workgroups_of_the_continuous_models(kernel_arith, particles, walkers, window, waves, grid):
    used = -(-12 * particles // 256) * 256 + -(-window // 64) * 64 * 12
    got = workgroup(kernel_arith, used, 0, particles, walkers)
    assert got[:2] == (waves, grid) and got[2] <= LDS


def test_every_accepted_size_has_a_workgroup_that_fits(kernel_arith):
    # what creation accepts: state and window beside the buffers of one attempt
    # shared by the wavefronts (512 bytes and more for 64 particles)
    rng = np.random.default_rng(61)
    for _ in range(20_000):
        particles = int(np.exp(rng.uniform(np.log(3), np.log(4096))))
        lipid = rng.random() < 0.5
        chunks = (particles + 63) // 64
        state = -(-((16 if lipid else 0) + (21 if lipid else 12) * particles) // 256) * 256
        room = LDS - state - chunks * 64 * 8 * (1 if lipid else 2) - (chunks * 16 if lipid else 0)
        if room < 768:
            continue
        window = (room // 768 if rng.random() < 0.5 else rng.integers(1, room // 768 + 1)) * 64
        used = state + int(window) * 12 + (chunks * 16 if lipid else 0)
        waves, grid, lds = workgroup(kernel_arith, used, 8 if lipid else 0, particles, int(rng.integers(1, 65536)))
        assert waves in (1, 2, 4, 8, 16) and lds <= LDS, (particles, lipid, window)
