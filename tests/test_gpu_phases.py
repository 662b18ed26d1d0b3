"""GPU parity at the edges of the attempt kernel's rules: ln f on either side
of the line between its two decision phases, blocks of one attempt more or less
than a wavefront, walkers with and without a drawing wavefront beside them,
infinite ln g, and walkers per window around the exchange kernel's workgroup."""
import numpy as np
import pytest

from statecmp import assert_same_state
from test_gpu_parity import make_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,q,h,m,sync,precision,lnf", [
    (4, 2, 2, 3, 333, 0, 1.0),            # 16 sites: nearly every attempt touches an earlier one
    (4, 2, 2, 3, 333, 1, 0.3),
    (8, 10, 4, 1, 63, 0, 1.0),            # blocks of 63, 64 and 65 attempts
    (8, 10, 4, 1, 64, 1, 1.0),
    (8, 10, 4, 1, 65, 0, 2.0**-6),
    (32, 10, 16, 4, 1000, 0, 2.0**-6),     # last halving from event to event
    (32, 10, 16, 4, 1000, 1, 2.0**-6),
    (32, 10, 16, 4, 1000, 0, 2.0**-7),     # first that guesses
    (32, 10, 16, 4, 1000, 1, 2.0**-7),
    (12, 3, 4, 384, 500, 0, 1.0),         # six walkers a compute unit: with a drawing wavefront
    (12, 3, 4, 385, 500, 0, 1.0),         # more: without
    (12, 3, 4, 385, 500, 1, 1.0),
    (12, 3, 4, 385, 500, 0, 2.0**-7),
])
def test_decision_phases_bitexact(L, q, h, m, sync, precision, lnf):
    g, o = make_pair(L, q, h, m, lnf_init=lnf, fixed_lnf=1, sync_attempts=sync, exchange=1, precision=precision, seed=23)
    for n in (sync, 3 * sync + 1):
        g.run(n)
        o.run(n)
    assert_same_state(g, o)


@pytest.mark.parametrize("precision,lnf", [(0, 0.5), (1, 0.5), (0, 2.0**-9), (1, 2.0**-9)])
def test_infinite_weights_bitexact(precision, lnf):
    # bins no walker may enter (+inf) and bins every proposal is accepted into (-inf)
    g, o = make_pair(8, 3, 1, 4, lnf_init=lnf, fixed_lnf=1, sync_attempts=500, precision=precision, seed=29)
    for w in range(4):
        lng = 0.25 * np.arange(g.W, dtype=np.float64)
        lng[w::9] = np.inf if w % 2 else -np.inf
        g.set_lng(w, lng)
        o.set_lng(w, lng)
    g.run(3001)
    o.run(3001)
    assert_same_state(g, o)


@pytest.mark.parametrize("m", [1, 2, 17, 64, 65])
def test_exchange_and_flatness_over_walkers_per_window(m):
    g, o = make_pair(6, 3, 3, m, lnf_init=1.0, flat=(1, 2), sync_attempts=300, exchange=1, seed=31)
    g.run(6000)
    o.run(6000)
    assert_same_state(g, o)


@pytest.mark.parametrize("precision", [0, 1])
def test_lnf_of_the_one_over_t_schedule_bitexact(precision):
    # ln f = W/t has a full significand; weights as a long run leaves them
    g, o = make_pair(8, 10, 4, 8, lnf_init=461 / 1.6e9, fixed_lnf=1, sync_attempts=4000, precision=precision, seed=37)
    rng = np.random.default_rng(37)
    for w in range(32):
        lng = rng.uniform(50.0, 3000.0) + np.cumsum(rng.uniform(-0.5, 0.7, g.W))
        g.set_lng(w, lng)
        o.set_lng(w, lng)
    g.run(60_000)
    o.run(60_000)
    assert_same_state(g, o)


def test_more_runs_at_once_than_slots_for_their_flags():
    # 70 runs of different lengths, alive together: each reads its own flag and
    # stop point, with a pinned slot or without; destroyed runs' slots are used again
    for turn in range(2):
        pairs = [make_pair(3, 2, 1, 1, lnf_init=1.0, lnf_final=2.0**-(1 + i % 7), flat=(0, 1), sync_attempts=50 + i,
                           seed=turn * 100 + i) for i in range(70)]
        for g, o in pairs:
            assert g.run(400) == o.run(400)
        for g, o in pairs:
            assert g.run(300) == o.run(300)
            assert g.progress()[:2] == (o.step, o.round)
            assert_same_state(g, o)
