"""The kernels' closed forms for repeated additions of ln f to one ln g value
(rewl_replay.h, built for the host) against the additions made one by one, bit
for bit: ln f = W/t of the 1/t schedule, whose significand is full, and
significands of a few bits, which fall half-way between two values of the sum's
binade; sums that enter a binade with the first addition."""
import ctypes

import numpy as np
import pytest


def ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def call(fn, n, *arrays):
    fn.restype = ctypes.c_size_t
    fn.argtypes = [ctypes.c_size_t] + [ctypes.c_void_p] * (len(arrays) + 1)
    return fn(len(n), *[ptr(a) for a in arrays], ptr(n))


def two_sum(h, l, x):
    s = h + x
    bb = s - h
    return s, l + ((h - (s - bb)) + (x - bb))


def steps(kind, count, rng, dtype):
    """ln f below 2^-7: W/t, significands whose last 1 .. 8 bits are zero, or a few bits wide."""
    if kind == "W/t":
        f = rng.integers(8, 6000, count) / np.exp(rng.uniform(np.log(1e6), np.log(1e11), count))
        return np.minimum(f, 2.0**-7).astype(dtype)
    bits = 24 if dtype is np.float32 else 53
    width = bits - rng.integers(1, 9, count) if kind == "zeros" else rng.integers(1, 9, count)
    sig = rng.integers(2.0**(width - 1), 2.0**width) | 1
    return np.ldexp(sig.astype(np.float64), (-width - rng.integers(7, 34, count)).astype(np.int32)).astype(dtype)


@pytest.mark.parametrize("kind", ["W/t", "zeros", "short"])
def test_pair(kernel_arith, kind):
    # bins of ln g 50 .. 3000 as a binary64 value split, visited 1 .. 12 times a block for 60 blocks
    rng = np.random.default_rng(41)
    bins = 20_000
    g = rng.uniform(50.0, 3000.0, bins)
    hi = g.astype(np.float32)
    lo = (g - hi.astype(np.float64)).astype(np.float32)
    f = steps(kind, bins, rng, np.float32)
    for _ in range(60):
        n = rng.integers(1, 13, bins).astype(np.uint32)
        rh, rl = hi, lo
        for k in range(12):
            h, l = two_sum(rh, rl, f)
            rh, rl = np.where(k < n, h, rh), np.where(k < n, l, rl)
        call(kernel_arith.replay_pair_all, n, hi, lo, f)
        bad = np.flatnonzero((hi.view(np.int32) != rh.view(np.int32)) | (lo.view(np.int32) != rl.view(np.int32)))
        assert len(bad) == 0, (len(bad), hi[bad[0]], lo[bad[0]], rl[bad[0]], f[bad[0]], n[bad[0]])


@pytest.mark.parametrize("lnf", [461 / 1.18e9, 461 / 4.3e10, 2.0**-21])
def test_pair_late_in_a_run_takes_closed_forms(kernel_arith, lnf):
    # low words of either sign against an ln f that the high word ignores
    rng = np.random.default_rng(43)
    g = rng.uniform(200.0, 3000.0, 20_000)
    hi = g.astype(np.float32)
    lo = (g - hi.astype(np.float64)).astype(np.float32)
    f = np.full(len(g), lnf, dtype=np.float32)
    single = total = 0
    for _ in range(40):
        n = rng.integers(1, 13, len(g)).astype(np.uint32)
        single += call(kernel_arith.replay_pair_all, n, hi, lo, f)
        total += int(n.sum())
    assert single < 0.2 * total


def test_pair_that_enters_a_binade_on_an_odd_value(kernel_arith):
    # ln f half-way between two spacings of the binade it enters; 10 visits
    hi = np.array([float.fromhex("0x1.41c00cp+11")], dtype=np.float32)
    lo = np.array([float.fromhex("0x1.764888p-20")], dtype=np.float32)
    f = np.array([float.fromhex("0x1.3899b8p-22")], dtype=np.float32)
    call(kernel_arith.replay_pair_all, np.array([10], dtype=np.uint32), hi, lo, f)
    assert float(hi[0]) == float.fromhex("0x1.41c00cp+11") and float(lo[0]) == float.fromhex("0x1.20f238p-18")


@pytest.mark.parametrize("kind", ["W/t", "zeros", "short"])
def test_binary64(kernel_arith, kind):
    # values just below a power of two, as many of ln f's half spacings as it takes to cross
    rng = np.random.default_rng(42)
    count = 200_000
    f = steps(kind, count, rng, np.float64)
    top = np.ldexp(1.0, rng.integers(-3, 13, count).astype(np.int32))
    near = rng.random(count) < 0.5
    x = np.where(near, top - f * rng.uniform(0.0, 2.0, count), top * rng.uniform(0.5, 1.0, count))
    # half of ln f's to end on half a spacing of that binade
    spacing = np.spacing(top)
    tie = rng.random(count) < 0.5
    f = np.where(tie & (f > 4 * spacing), np.floor(f / spacing) * spacing + 0.5 * spacing, f)
    n = rng.integers(1, 65, count).astype(np.uint32)
    ref = x
    for k in range(64):
        ref = np.where(k < n, ref + f, ref)
    got = x.copy()
    closed = call(kernel_arith.replay_binary64_all, n, got, f)
    bad = np.flatnonzero(got != ref)
    assert len(bad) == 0, (len(bad), x[bad[0]].hex(), f[bad[0]].hex(), n[bad[0]])
    assert closed > 0.3 * count


def test_margin_of_pairs_refuses_what_lies_outside_the_window(kernel_arith):
    f = kernel_arith.pair_decision_margin
    f.restype, f.argtypes = ctypes.c_double, [ctypes.c_double, ctypes.c_double, ctypes.c_float]
    inf = float("inf")
    assert f(0.01, -40.0, -0.5) == 0.01 + 40.5 * 2.0**-18
    assert -inf < -f(0.01, -inf, 0.0)        # t = d = -inf lies below the margin: no exact evaluation
    assert not -inf < -f(inf, -inf, 0.0)     # ln g of the current energy infinite: evaluated exactly
    assert not -inf < -f(0.01, -inf, inf)
