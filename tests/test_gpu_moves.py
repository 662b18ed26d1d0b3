"""GPU parity of the block-wise displacement attempts (rewl_moves.h) where
their launch or their arithmetic takes another path: workgroups cut down by the
LDS, places without their 16-bit copies, boxes smaller than the cut-off or far
larger than it, particles drawn several times in a block, weights of minus
infinity, energies more than 2^20 bins away.  Integers and binary64 bits equal
the oracle's."""
import numpy as np
import pytest

import oracle
import workloads
from statecmp import assert_same_state
from test_gpu_lipid import assert_same_lipids
from test_gpu_lipid import make_pair as lipid_pair
from test_gpu_trimer import assert_same_energies
from test_gpu_trimer import make_pair as trimer_pair

pytestmark = pytest.mark.gpu

TRIMERS = [
    # (nmol, box, e_min, bin_w, bins, h, m, attempts, precision)
    (16, 7.0, -40.0, 0.05, 13440, 1, 2, 1500, 0),   # two or four wavefronts beside 158 KiB of window
    (16, 7.0, -40.0, 0.05, 12800, 1, 2, 1500, 1),   # sixteen wavefronts, no room for the 16-bit places
    (2, 2.6, -10.0, 0.5, 400, 1, 3, 2000, 0),       # half the box below the cut-off, six beads for sixteen attempts
    (21, 60.0, -40.0, 0.5, 600, 2, 2, 1500, 0),     # 63 beads: one partner short of a chunk
    (43, 9.0, -60.0, 0.5, 600, 2, 2, 1200, 1),      # 129 beads: one partner in the third chunk
]


@pytest.mark.parametrize("nmol,box,e_min,bin_w,bins,h,m,attempts,precision", TRIMERS)
def test_trimer_blocks(nmol, box, e_min, bin_w, bins, h, m, attempts, precision):
    g, o = trimer_pair(nmol, box, e_min, bin_w, bins, h, m, lnf_init=0.05, fixed_lnf=1, sync_attempts=499,
                       precision=precision, seed=5)
    g.run(attempts)
    o.run(attempts)
    assert_same_state(g, o)
    assert_same_energies(g, o)


LIPIDS = [
    # (nlip, nsol, box, e_min, bin_w, bins, h, m, attempts, rep_prob)
    (4, 20, 4.3, 150.0, 0.05, 13440, 1, 1, 600, 0.2),       # two or four wavefronts
    (125, 625, None, 7000.0, 0.1, 11200, 1, 1, 300, 0.2),   # sixteen wavefronts, no 16-bit places
]


@pytest.mark.parametrize("nlip,nsol,box,e_min,bin_w,bins,h,m,attempts,rep_prob", LIPIDS)
def test_lipid_blocks(nlip, nsol, box, e_min, bin_w, bins, h, m, attempts, rep_prob):
    g, o = lipid_pair(nlip, nsol, box or workloads.LIPID["box"], e_min, bin_w, bins, h, m, rep_prob=rep_prob,
                      lnf_init=0.05, fixed_lnf=1, sync_attempts=199, seed=6)
    g.run(attempts)
    o.run(attempts)
    assert_same_state(g, o)
    assert_same_lipids(g, o)


def test_weights_of_minus_infinity():
    # unvisited bins of a finished piece, read back and set as weights
    g, o = trimer_pair(8, 5.0, -30.0, 0.5, 160, 1, 2, lnf_init=0.25, fixed_lnf=1, sync_attempts=300, seed=3)
    g.run(600)
    o.run(600)
    for w in range(2):
        lng = np.where(g.walker(w)["H"] > 0, g.walker(w)["lng"], -np.inf)
        g.set_lng(w, lng)
        o.set_lng(w, lng)
    g.run(900)
    o.run(900)
    assert_same_state(g, o)
    assert_same_energies(g, o)


def test_moves_beyond_a_million_bins():
    x = workloads.init_trimers(8, 5.0, 1, 1)
    o = oracle.Rewl.trimer(8, 5.0, -1000.0, 1.0, 4000, 1, 0.75, 1, x)
    args = (8, 5.0, o.energy(0) - 0.006, 1e-6, 12000, 1, 1)
    g, o = trimer_pair(*args, lnf_init=0.05, fixed_lnf=1, sync_attempts=1000, seed=3)
    g.run(3000)
    o.run(3000)
    assert_same_state(g, o)
    assert_same_energies(g, o)


@pytest.mark.parametrize("bin_w,precision", [(4096.0, 0), (4096.0, 1), (4097.0, 0), (4097.0, 1)])
def test_widest_bins_of_the_quick_decisions(bin_w, precision):
    # 2^44 units of energy a bin, and a unit of energy more: exact rounds only
    g, o = trimer_pair(8, 5.0, -5.0 * bin_w, bin_w, 10, 1, 2, lnf_init=0.05, fixed_lnf=1, sync_attempts=300,
                       precision=precision, seed=7)
    g.run(900)
    o.run(900)
    assert_same_state(g, o)
    assert_same_energies(g, o)


@pytest.mark.parametrize("box", [250.0, 1000.0])
def test_droplets_in_large_boxes(box):
    # a dense cluster in the middle of a box a hundred times its size: places
    # 0.004 and 0.015 apart on the screens' 16-bit grid
    import paper_1312_3004_amd as pk

    x = workloads.init_trimers(64, 10.0, 3, 2).reshape(3, 64, 3, 3).astype(np.float64)
    for b in (1, 2):                                   # molecules in one piece
        d = x[:, :, b] - x[:, :, b - 1]
        x[:, :, b] -= 10.0 * np.rint(d / 10.0)
    x = (x.reshape(3, 192, 3) + box / 2).astype(np.float32)
    opts = dict(lnf_init=0.05, fixed_lnf=1, sync_attempts=499, seed=9)
    args = (64, box, -300.0, 0.5, 2400, 1, 0.75, 3, x)
    print(f"[case] droplet of 64 trimers, box {box}", flush=True)
    g, o = pk.Rewl.trimer(*args, **opts), oracle.Rewl.trimer(*args, threads=8, **opts)
    g.run(4000)
    o.run(4000)
    assert_same_state(g, o)
    assert_same_energies(g, o)

    x = workloads.init_lipids(6, 106, 5.0, 3, 2).astype(np.float64)
    x = (np.where(x > 4.5, x - 5.0, x) + box / 2).astype(np.float32)
    start = oracle.Rewl.lipid(6, 106, box, 0.0, 1.0, 100, 1, 0.75, 3, x, rep_prob=0.4)
    e = [start.energy(w) for w in range(3)]
    args = (6, 106, box, min(e) - 200.0, 0.5, int(2 * (max(e) - min(e) + 400.0)), 1, 0.75, 3, x)
    g, o = pk.Rewl.lipid(*args, rep_prob=0.4, **opts), oracle.Rewl.lipid(*args, rep_prob=0.4, threads=8, **opts)
    g.run(3000)
    o.run(3000)
    assert_same_state(g, o)
    assert_same_lipids(g, o)


@pytest.mark.parametrize("nmol,box,h,m,attempts,precision", [
    (4, 5.0, 1, 1024, 150, 0),        # four, as many walkers a CU
    (16, 7.0, 1, 512, 150, 1),        # eight, two walkers a CU
    (8, 5.0, 2, 650, 100, 0),         # two, up to eight walkers a CU
])
def test_trimer_workgroups_of_fewer_wavefronts(nmol, box, h, m, attempts, precision):
    g, o = trimer_pair(nmol, box, -40.0, 0.5, 400, h, m, lnf_init=0.05, fixed_lnf=1, sync_attempts=49,
                       precision=precision, seed=11)
    g.run(attempts)
    o.run(attempts)
    assert_same_state(g, o)
    assert_same_energies(g, o)


@pytest.mark.parametrize("h,m", [(1, 300), (1, 700), (2, 550)])   # eight, four and two wavefronts
def test_lipid_workgroups_of_fewer_wavefronts(h, m):
    g, o = lipid_pair(6, 60, 5.0, 300.0, 0.5, 800, h, m, rep_prob=0.3, lnf_init=0.05, fixed_lnf=1, sync_attempts=49,
                      seed=12)
    g.run(100)
    o.run(100)
    assert_same_state(g, o)
    assert_same_lipids(g, o)


@pytest.mark.parametrize("nmol,box,m,attempts,precision", [
    (1, 3.0, 2, 3001, 0), (1, 3.0, 2, 3001, 1), (2, 2.6, 3, 2000, 1), (2, 4.0, 1024, 130, 0), (2, 14.0, 2, 63, 0),
    (2, 14.0, 2, 1, 1),
])
@pytest.mark.parametrize("infinite", [False, True])
def test_trimers_of_few_beads(nmol, box, m, attempts, precision, infinite):
    # one wavefront, attempts one after the other; unvisited bins at minus infinity
    g, o = trimer_pair(nmol, box, -20.0, 0.5, 200, 1, m, lnf_init=0.25, fixed_lnf=1, sync_attempts=97,
                       precision=precision, seed=13)
    g.run(attempts)
    o.run(attempts)
    if infinite:
        for w in range(min(m, 3)):
            lng = np.where(g.walker(w)["H"] > 0, g.walker(w)["lng"], -np.inf)
            g.set_lng(w, lng)
            o.set_lng(w, lng)
    g.run(attempts)
    o.run(attempts)
    assert_same_state(g, o)
    assert_same_energies(g, o)
