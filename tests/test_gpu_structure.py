"""GPU parity of the structural observables of the lipid model (Sec. 3.2,
Eqs. 6-8) with the oracle: cluster count, largest-cluster size and the axis
of S_mol exact; S_mol, Q_ii and the prolateness to rounding (the kernel sums
across lanes in butterfly order, the oracle with numpy)."""
import sys

import numpy as np
import pytest

import oracle
import workloads
from oracle import structure as S

pytestmark = pytest.mark.gpu

RTOL, ATOL = 1e-10, 1e-12


def _pk():
    import paper_1312_3004_amd as pk
    return pk


def gpu_records(coords, lips, box):
    import torch

    x = torch.from_numpy(np.ascontiguousarray(coords, dtype=np.float32)).cuda()
    lp = torch.from_numpy(np.ascontiguousarray(lips, dtype=np.int32)).cuda()
    out = _pk().lipid_structure(x, lp, box)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def assert_same_record(got, ref, what):
    # integers: cluster count and largest size exact
    assert got[2] == ref[2] and got[3] == ref[3], (what, got[:4], ref[:4])
    # the axis is decided in binary64 on both sides; accept a different axis only on a near tie
    if got[1] != ref[1]:
        assert abs(got[0] - ref[0]) <= 1e-12, (what, got[:2], ref[:2])
    np.testing.assert_allclose(got[[0, 4, 5, 6]], ref[[0, 4, 5, 6]], rtol=RTOL, atol=ATOL, err_msg=what)
    # P = 9 sum (Q - lambda)^3 / tr^3: absolute rounding scale 1
    np.testing.assert_allclose(got[7], ref[7], rtol=1e-9, atol=1e-11, err_msg=what)


def random_configs(nconf, M, nsol, box, seed, bond=0.97):
    rng = np.random.default_rng(seed)
    np_ = 3 * M + nsol
    xs = rng.uniform(0, box, (nconf, np_, 3))
    lips = np.zeros((nconf, M, 3), dtype=np.int32)
    for c in range(nconf):
        perm = rng.permutation(np_)[:3 * M].reshape(M, 3)   # lipid beads scattered over the indices
        o = rng.uniform(0, box, (M, 3))
        v = rng.normal(size=(M, 3))
        v /= np.linalg.norm(v, axis=1)[:, None]
        w = rng.normal(size=(M, 3))
        w /= np.linalg.norm(w, axis=1)[:, None]
        xs[c, perm[:, 0]] = o
        xs[c, perm[:, 1]] = o + bond * v
        xs[c, perm[:, 2]] = o + bond * v + bond * w
        lips[c] = perm
    return (xs % box).astype(np.float32), lips


@pytest.mark.parametrize("nconf,M,nsol,box,seed", [
    (3, 1, 5, 6.0, 0),        # one lipid
    (4, 20, 30, 8.0, 1),      # sparse: many small clusters
    (5, 63, 10, 6.0, 2),      # one mask word, dense
    (5, 64, 0, 6.5, 3),       # exactly one word
    (4, 65, 7, 7.0, 4),       # ragged second word
    (3, 128, 20, 8.0, 7),     # exactly two words
    (3, 129, 20, 8.0, 8),     # one lipid in the third word
    (3, 200, 100, 9.0, 5),    # four words, percolating
    (2, 512, 64, 11.0, 6),    # the maximum: LDS beyond 64 KiB
])
def test_random_configurations(nconf, M, nsol, box, seed):
    print(f"[case] structure random nconf={nconf} M={M} nsol={nsol} box={box} seed={seed}", flush=True)
    sys.stdout.flush()
    xs, lips = random_configs(nconf, M, nsol, box, seed)
    got = gpu_records(xs, lips, box)
    for c in range(nconf):
        assert_same_record(got[c], S.structure(xs[c], lips[c], box), f"conf {c}")


@pytest.mark.parametrize("M,box,shift,seed", [
    (70, 7.0, 1.0, 10),       # places outside [0, box): the binary32 screen
    (256, 9.0, 0.4, 11),      # the last size with its rows in registers
    (257, 9.0, 0.0, 12),      # the first that reads them from LDS
    (40, 2.5, 0.0, 13),       # contact radius beyond half the box: all touch
    (40, 0.5, 0.0, 14),       # beyond the box: the limits' upper end
    (40, 3.0e5, 0.0, 15),     # contact radius below the grid's step: every pair exact
])
def test_screen_and_row_forms(M, box, shift, seed):
    print(f"[case] structure screen M={M} box={box} shift={shift} seed={seed}", flush=True)
    xs, lips = random_configs(3, M, 9, min(box, 9.0), seed)
    xs = (xs % np.float32(box)).astype(np.float32)
    xs[1:] += np.float32(shift * box) * np.random.default_rng(seed).integers(-1, 2, xs[1:].shape).astype(np.float32)
    got = gpu_records(xs, lips, box)
    for c in range(3):
        assert_same_record(got[c], S.structure(xs[c], lips[c], box), f"conf {c}")


def test_rods_and_hand_built_clusters():
    # a ring of 10 lipids closing through the boundary, and a straight rod
    K, s = 10, 0.6
    box = 3 * K * s
    beads = np.zeros((K, 3, 3))
    beads[:, :, 0] = (s * np.arange(3 * K)).reshape(K, 3)
    beads[:, :, 1:] = 5.0
    ring = beads.reshape(-1, 3).astype(np.float32)
    lip = np.arange(3 * K, dtype=np.int32).reshape(K, 3)
    print("[case] structure ring", flush=True)
    got = gpu_records(ring[None], lip[None], box)[0]
    ref = S.structure(ring, lip, box)
    assert_same_record(got, ref, "ring")
    assert got[3] == K and got[4] == pytest.approx(s * s * ((3 * K) ** 2 - 1) / 12, rel=1e-5)


def test_bad_index_gives_nan_record_and_others_unaffected():
    xs, lips = random_configs(3, 10, 5, 6.0, 9)
    lips = lips.copy()
    lips[1, 4, 2] = 35  # np = 35: one past the end
    print("[case] structure bad index", flush=True)
    got = gpu_records(xs, lips, 6.0)
    assert np.all(np.isnan(got[1]))
    for c in (0, 2):
        assert_same_record(got[c], S.structure(xs[c], lips[c], 6.0), f"conf {c}")


def test_empty_batch_and_argument_errors():
    import torch

    pk = _pk()
    x = torch.zeros((0, 30, 3), dtype=torch.float32, device="cuda")
    lp = torch.zeros((0, 10, 3), dtype=torch.int32, device="cuda")
    assert pk.lipid_structure(x, lp, 5.0).shape == (0, 8)
    x = torch.zeros((1, 30, 3), dtype=torch.float32, device="cuda")
    lp = torch.zeros((1, 11, 3), dtype=torch.int32, device="cuda")
    with pytest.raises(pk.RewlError):
        pk.lipid_structure(x, lp, 5.0)   # np < 3 nlip


def test_run_walkers_on_the_paper_system():
    # the paper's system (125 lipids, 625 solvent, density 0.8): every walker's
    # configuration after a short run, against the oracle run's own states
    c = workloads.LIPID
    h, m = 4, 2
    x0 = workloads.init_lipids(c["nlip"], c["nsol"], c["box"], h * m, 1)
    print("[case] structure on lipid runs (125 lipids, 8 walkers)", flush=True)
    g = _pk().Rewl.lipid(c["nlip"], c["nsol"], c["box"], c["e_min"], c["bin_w"], c["bins"], h, 0.75, m, x0,
                         lnf_init=1.0, sync_attempts=400, seed=c["seed"])
    o = oracle.Rewl.lipid(c["nlip"], c["nsol"], c["box"], c["e_min"], c["bin_w"], c["bins"], h, 0.75, m, x0,
                          threads=8, lnf_init=1.0, sync_attempts=400, seed=c["seed"])
    g.run(1200)
    o.run(1200)
    got = g.structure()
    for w in range(h * m):
        xw, _, lw = o.lipid_state(w)
        assert_same_record(got[w], S.structure(xw, lw, c["box"]), f"walker {w}")


def oracle_obs(o, nlip, box, obs_bins, hist, sums, cnt):
    """Add every walker's sample at a sync point: O = lipids in the largest cluster."""
    for w in range(o.nw):
        xw, _, lw = o.lipid_state(w)
        O = int(S.structure(xw, lw, box)[3])
        b = o.walker(w)["E"] - int(o.starts[w // o.m])
        if 0 <= b < o.W:
            hist[w, b, O * obs_bins // (nlip + 1)] += 1
            sums[w, b] += O
            cnt[w, b] += 1


@pytest.mark.parametrize("nlip,nsol,box,e_min,bins,h,m,S_att,syncs,rep_prob,obs_bins", [
    (6, 60, 5.0, 300.0, 320, 3, 2, 300, 8, 0.3, 7),
    (10, 40, 5.0, 300.0, 400, 2, 2, 250, 8, 0.5, 4),
])
def test_lipid_production_h_of_e_and_largest_cluster(nlip, nsol, box, e_min, bins, h, m, S_att, syncs, rep_prob,
                                                     obs_bins):
    # H(E, O) of the production phase (Sec. 3.2) against the oracle run's own
    # states, sampled by the oracle's structure() at each sync point
    x0 = workloads.init_lipids(nlip, nsol, box, h * m, 2)
    print(f"[case] lipid production H(E, O) nlip={nlip} nsol={nsol} h={h} m={m} obs_bins={obs_bins}", flush=True)
    opts = dict(rep_prob=rep_prob, lnf_init=0.05, fixed_lnf=1, sync_attempts=S_att, exchange=1, seed=4)
    g = _pk().Rewl.lipid(nlip, nsol, box, e_min, 0.5, bins, h, 0.75, m, x0, obs_bins=obs_bins, **opts)
    o = oracle.Rewl.lipid(nlip, nsol, box, e_min, 0.5, bins, h, 0.75, m, x0, threads=8, **opts)
    g.run(2 * S_att)
    o.run(2 * S_att)
    g.begin_production()
    o.begin_production()
    nw, W = h * m, o.W
    hist = np.zeros((nw, W, obs_bins), dtype=np.uint32)
    sums = np.zeros((nw, W), dtype=np.uint64)
    cnt = np.zeros((nw, W), dtype=np.uint32)
    for _ in range(syncs):
        o.run(S_att)
        oracle_obs(o, nlip, box, obs_bins, hist, sums, cnt)
    g.run(syncs * S_att)
    for w in range(nw):
        gh, gs, gc = g.obs(w)
        assert np.array_equal(gh, hist[w]), f"H(E, O) of walker {w}"
        assert np.array_equal(gs, sums[w]) and np.array_equal(gc, cnt[w]), f"sum/count of walker {w}"
    assert cnt.sum() == nw * syncs  # walkers never leave their windows
    mean, c = g.obs_micro()
    assert c.sum() == cnt.sum()


def test_lipid_obs_bins_limits():
    pk = _pk()
    x = workloads.init_lipids(4, 20, 4.3, 2, 1)
    with pytest.raises(pk.RewlError):
        pk.Rewl.lipid(4, 20, 4.3, 200.0, 0.5, 160, 1, 0.75, 2, x, obs_bins=4097)   # more than 4096 bins


def test_lipid_production_h_of_e_on_the_paper_system():
    # 125 lipids in 625 solvent particles: H(E, O) over three production sync
    # intervals, O = lipids in the largest cluster in all 126 bins
    c = workloads.LIPID
    h, m, S_att, syncs = 4, 2, 400, 3
    nlip, box, obs_bins = c["nlip"], c["box"], c["nlip"] + 1
    x0 = workloads.init_lipids(nlip, c["nsol"], box, h * m, 3)
    print("[case] lipid production H(E, O) on the paper system", flush=True)
    opts = dict(lnf_init=1.0, sync_attempts=S_att, seed=c["seed"])
    g = _pk().Rewl.lipid(nlip, c["nsol"], box, c["e_min"], c["bin_w"], c["bins"], h, 0.75, m, x0,
                         obs_bins=obs_bins, **opts)
    o = oracle.Rewl.lipid(nlip, c["nsol"], box, c["e_min"], c["bin_w"], c["bins"], h, 0.75, m, x0, threads=8,
                          **opts)
    g.run(S_att)
    o.run(S_att)
    g.begin_production()
    o.begin_production()
    hist = np.zeros((h * m, o.W, obs_bins), dtype=np.uint32)
    sums = np.zeros((h * m, o.W), dtype=np.uint64)
    cnt = np.zeros((h * m, o.W), dtype=np.uint32)
    for _ in range(syncs):
        o.run(S_att)
        oracle_obs(o, nlip, box, obs_bins, hist, sums, cnt)
    g.run(syncs * S_att)
    for w in range(h * m):
        gh, gs, gc = g.obs(w)
        assert np.array_equal(gh, hist[w]) and np.array_equal(gs, sums[w]) and np.array_equal(gc, cnt[w]), w
    assert cnt.sum() == h * m * syncs


def binned(v, lo, hi, bins):
    t = (v - lo) / (hi - lo) * bins
    q = int(t) if 0.0 <= t < bins else (bins - 1 if t >= bins else 0)
    return q, abs(t - round(t)) if 0.0 < t < bins else 1.0


@pytest.mark.parametrize("field,lo,hi,obs_bins", [(0, -0.5, 1.0, 12), (7, -0.25, 2.0, 9), (4, 0.0, 3.0, 10)])
def test_lipid_h_of_e_for_a_floating_point_field(field, lo, hi, obs_bins):
    # H(E, O) over S_mol, the prolateness or Q_xx in obs_bins bins over [lo, hi)
    nlip, nsol, box, e_min, bins, h, m, S_att, syncs = 6, 60, 5.0, 300.0, 320, 3, 2, 300, 8
    x0 = workloads.init_lipids(nlip, nsol, box, h * m, 2)
    print(f"[case] lipid production H(E, O) field={field} range=[{lo}, {hi}) bins={obs_bins}", flush=True)
    opts = dict(rep_prob=0.3, lnf_init=0.05, fixed_lnf=1, sync_attempts=S_att, exchange=1, seed=4)
    g = _pk().Rewl.lipid(nlip, nsol, box, e_min, 0.5, bins, h, 0.75, m, x0, obs_bins=obs_bins, **opts)
    o = oracle.Rewl.lipid(nlip, nsol, box, e_min, 0.5, bins, h, 0.75, m, x0, threads=8, **opts)
    g.lipid_obs_field(field, lo, hi)
    g.run(2 * S_att)
    o.run(2 * S_att)
    g.begin_production()
    o.begin_production()
    nw, W = h * m, o.W
    hist = np.zeros((nw, W, obs_bins), dtype=np.uint32)
    sums = np.zeros((nw, W), dtype=np.uint64)
    edge = 1.0
    for _ in range(syncs):
        o.run(S_att)
        for w in range(nw):
            xw, _, lw = o.lipid_state(w)
            q, e = binned(S.structure(xw, lw, box)[field], lo, hi, obs_bins)
            edge = min(edge, e)
            b = o.walker(w)["E"] - int(o.starts[w // m])
            hist[w, b, q] += 1
            sums[w, b] += q
    g.run(syncs * S_att)
    got = np.stack([g.obs(w)[0] for w in range(nw)])
    gsum = np.stack([g.obs(w)[1] for w in range(nw)])
    if edge > 1e-9:   # no sample within rounding of a bin edge: the histograms agree exactly
        assert np.array_equal(got, hist) and np.array_equal(gsum, sums)
    else:
        assert np.abs(got.astype(np.int64) - hist).sum() <= 2 and got.sum() == hist.sum()
    assert hist.sum() == nw * syncs and len(np.unique(np.nonzero(hist)[2])) >= 2


def test_lipid_obs_field_argument_errors():
    pk = _pk()
    x = workloads.init_lipids(4, 20, 4.3, 2, 1)
    g = pk.Rewl.lipid(4, 20, 4.3, 200.0, 0.5, 160, 1, 0.75, 2, x, obs_bins=5)
    for args in [(1, 0.0, 1.0), (8, 0.0, 1.0), (0, 1.0, 1.0), (0, 0.0, float("inf"))]:
        with pytest.raises(pk.RewlError):
            g.lipid_obs_field(*args)
    g.lipid_obs_field(3)
    g2 = pk.Rewl.lipid(4, 20, 4.3, 200.0, 0.5, 160, 1, 0.75, 2, x)
    with pytest.raises(pk.RewlError):
        g2.lipid_obs_field(0, -0.5, 1.0)   # no observable sampling


def test_contacts_within_ulps_of_the_threshold():
    # 100 isolated pairs of lipids on the x axis whose tail gap steps through
    # float32 values around 1.4: the kernel's binary32 screen leaves those near
    # 1.4 to its binary64 test, and every decision must equal the definition
    K = 100
    base = np.float32(3.4)
    # the float32 grid around 3.4: base moved by -50 .. +49 ulps
    grid = [base]
    lo, hi = base, base
    for _ in range(50):
        lo = np.nextafter(lo, np.float32(0))
        grid.insert(0, lo)
    for _ in range(49):
        hi = np.nextafter(hi, np.float32(10))
        grid.append(hi)
    assert len(grid) == K
    beads = np.zeros((2 * K, 3, 3), dtype=np.float32)
    for k, xc in enumerate(grid):
        y, z = np.float32(5 * (k % 10) + 2), np.float32(5 * (k // 10) + 2)
        beads[2 * k] = [[0.0, y, z], [1.0, y, z], [2.0, y, z]]            # A: head, centre, end at x = 2
        beads[2 * k + 1] = [[xc + np.float32(2.0), y, z], [xc + np.float32(1.0), y, z], [xc, y, z]]  # B: end at xc
    x = beads.reshape(-1, 3)
    lip = np.arange(6 * K, dtype=np.int32).reshape(2 * K, 3)
    box = 60.0
    gap = np.array([np.float64(np.float32(xc - np.float32(2.0))) for xc in grid])
    contacts = int(np.sum(gap * gap < 1.96))
    assert 0 < contacts < K
    print(f"[case] structure threshold pairs: {contacts} of {K} touch", flush=True)
    got = gpu_records(x[None], lip[None], box)[0]
    ref = S.structure(x, lip, box)
    assert ref[2] == 2 * K - contacts
    assert_same_record(got, ref, "threshold pairs")
