"""The work a user of this package has it do, as cases that can be timed and compared.

A case is a dict of plain values.  ``prepare`` builds what a program holds
before the call (a run with walkers in their windows and weights of the phase
the case stands for, a batch, a set of configurations), ``run`` is one pass
through the public entry points and returns what it computed.  Runs return
their device workspace: it holds every walker's configuration, energy, ln g
and H, the windows' state and the observable record.

Phases of a run are pinned by ``fixed_lnf`` (sync points then leave ln f
alone), so that a pass costs the same however often it is repeated.  Weights
of a small ln f come from a quick descent: ln f halved at every sync point.
"""
import math

import numpy as np
import torch

import paper_1312_3004_amd as pk

DEVICE = "cuda:0"
TEMPERATURES = 201


def listed():
    return [
        # The smallest call: 8 x 8 lattice, four walkers, one sync interval of
        # the default 1,000 attempts.  Launches and waiting count.
        dict(name="potts_L8_call", kind="potts", L=8, q=10, windows=4, walkers=1, lnf_log2=-10, precision=0,
             obs_bins=0, sync=1000, attempts=1000),
        # The 32 x 32 benchmark system (16 windows x 4 walkers, sync every
        # 10^4 attempts) right after the walk-in, ln f = 1.
        dict(name="potts_L32_first", kind="potts", L=32, q=10, windows=16, walkers=4, lnf_log2=0, precision=0,
             obs_bins=0, sync=10000, attempts=20000),
        # The same while ln f halves.
        dict(name="potts_L32_halving", kind="potts", L=32, q=10, windows=16, walkers=4, lnf_log2=-10, precision=0,
             obs_bins=0, sync=10000, attempts=50000),
        # The same where most of a run's attempts are spent: ln f near 1e-6.
        dict(name="potts_L32_late", kind="potts", L=32, q=10, windows=16, walkers=4, lnf_log2=-21, precision=0,
             obs_bins=0, sync=10000, attempts=50000),
        # The same with ln g kept as a binary32 (hi, lo) pair.
        dict(name="potts_L32_pair", kind="potts", L=32, q=10, windows=16, walkers=4, lnf_log2=-21, precision=1,
             obs_bins=0, sync=10000, attempts=50000),
        # The 80 x 80 system: 64 windows x 16 walkers, every CU holds several.
        dict(name="potts_L80_late", kind="potts", L=80, q=10, windows=64, walkers=16, lnf_log2=-20, precision=0,
             obs_bins=0, sync=10000, attempts=20000),
        # 256 independent runs of mixed sizes advanced together (8,192 walkers).
        dict(name="batch_256", kind="batch", instances=256, windows=8, walkers=4, L_max=48, lnf_log2=0, sweeps=100),
        # 64 amphiphilic trimers per walker, single-bead displacements.
        dict(name="trimer_64", kind="trimer", nmol=64, box=10.0, e_min=-460.0, bin_w=0.5, bins=1000, windows=16,
             walkers=4, precision=0, sync=2000, attempts=2000),
        # Lipids in explicit solvent at the size of the paper (N = 1000),
        # recording the largest cluster at every sync point.
        dict(name="lipid_1000", kind="lipid", nlip=125, nsol=625, e_min=7000.0, bins=800, windows=16, walkers=4,
             obs_bins=25, sync=1000, attempts=1000),
        # Structural observables of a stored trajectory of that system.
        dict(name="structure_4096", kind="structure", nconf=4096, nlip=125, nsol=625),
        # Starting a run: creation from random lattices and the walk-in.
        dict(name="start_L32", kind="start", L=32, q=10, windows=16, walkers=4),
        # Error bars over 64 independent runs: 1,000 resamples, each joined anew.
        dict(name="bootstrap_64", kind="bootstrap", L=8, q=10, windows=4, runs=64, nboot=1000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["potts", "potts", "potts", "potts", "batch", "trimer", "lipid", "structure", "start", "bootstrap"])
    if kind == "potts":
        L = _log_int(rng, 8, 80)
        windows = rng.randint(1, 4) if L < 16 else rng.randint(4, 16)
        walkers = rng.randint(1, 8)
        precision = int(rng.random() < 0.25)
        obs = rng.choice([0, 0, 0, rng.randint(5, 65)])
        sync = _log_int(rng, 500, 10000)
        return dict(kind=kind, L=L, q=rng.randint(2, 12), windows=windows, walkers=walkers,
                    lnf_log2=-rng.randint(0, 22), precision=precision, obs_bins=obs, sync=sync,
                    attempts=sync * rng.randint(1, 4) + rng.choice([0, 0, rng.randint(1, sync)]))
    if kind == "batch":
        return dict(kind=kind, instances=_log_int(rng, 8, 48), windows=rng.randint(2, 8), walkers=rng.randint(1, 4),
                    L_max=rng.choice([16, 24, 32, 48]), lnf_log2=-rng.randint(0, 16), sweeps=_log_int(rng, 10, 100))
    if kind == "trimer":
        nmol = _log_int(rng, 6, 96)
        attempts = _log_int(rng, 300, 2000)
        return dict(kind=kind, nmol=nmol, box=round(10.0 * (nmol / 64) ** (1 / 3) * rng.uniform(1.0, 1.3), 3),
                    e_min=-3.0 * nmol, bin_w=0.5, bins=12 * nmol + 60, windows=rng.randint(1, 8),
                    walkers=rng.randint(1, 8), precision=int(rng.random() < 0.25), sync=attempts, attempts=attempts)
    if kind == "lipid":
        n = rng.randint(5, 10)
        total = n ** 3
        nlip = max(3, int(total * rng.uniform(0.03, 0.14)))
        attempts = _log_int(rng, 200, 1000)
        # the band about the energy of the lattice starts, as in the listed case
        f = nlip / total
        start = total * (-4.75 + 105.0 * f - 60.0 * f * f)
        return dict(kind=kind, nlip=nlip, nsol=total - 3 * nlip, e_min=round(start - 0.45 * total),
                    bins=max(40, int(0.8 * total)), windows=rng.randint(1, 8), walkers=rng.randint(1, 8),
                    obs_bins=rng.choice([0, nlip + 1]), sync=attempts, attempts=attempts)
    if kind == "structure":
        nlip = _log_int(rng, 8, 250)
        return dict(kind=kind, nconf=_log_int(rng, 16, 2000), nlip=nlip, nsol=rng.randint(nlip, 5 * nlip))
    if kind == "start":
        return dict(kind=kind, L=_log_int(rng, 8, 30), q=rng.randint(2, 12), windows=rng.randint(2, 8),
                    walkers=rng.randint(1, 4))
    return dict(kind="bootstrap", L=rng.randint(4, 8), q=rng.randint(2, 10), windows=rng.randint(1, 4),
                runs=_log_int(rng, 8, 64), nboot=_log_int(rng, 50, 1000))


# ---------------------------------------------------------------------------
# Inputs.

def _lattices(L, q, starts, W, walkers, rng):
    """One lattice per walker near its window: some rows in one state, the
    others random, the share of ordered rows set by the window's energy."""
    N = L * L
    out = rng.integers(0, q, size=(len(starts) * walkers, L, L), dtype=np.int8)
    for k, e0 in enumerate(starts):
        share = ((e0 + W / 2) / (-2.0 * N) - 1.0 / q) / (1.0 - 1.0 / q)
        rows = int(round(min(max(share, 0.0), 1.0) * L))
        for j in range(walkers):
            out[k * walkers + j, :rows] = rng.integers(0, q)
    return out.reshape(len(out), N)


def _potts_run(c, seed):
    rng = np.random.default_rng(seed)
    L, q, h, m = c["L"], c["q"], c["windows"], c["walkers"]
    W, starts = pk.window_layout(L, h, 0.75)
    spins = _lattices(L, q, starts, W, m, rng)
    lnf = 2.0 ** c["lnf_log2"]
    weights = None
    if lnf < 1.0:
        a = pk.Rewl(L, q, h, 0.75, m, spins, device=DEVICE, seed=seed + 1, flat=(0, 1), lnf_final=1.5 * lnf,
                    sync_attempts=min(max(400 * L * L, 10000), 400000))
        while a.run(10 * a.opts.sync_attempts) != pk.CONVERGED:
            pass
        state = [a.state(w) for w in range(h * m)]
        spins = np.stack([s["spins"] for s in state])
        weights = [s["lng"] for s in state]
    r = pk.Rewl(L, q, h, 0.75, m, spins, device=DEVICE, seed=seed, lnf_init=lnf, fixed_lnf=1,
                sync_attempts=c["sync"], precision=c["precision"], obs_bins=min(c["obs_bins"], L * L + 1))
    r.walkin()
    if weights is None:
        r.run((100000 // c["sync"] + 1) * c["sync"])
    else:
        for w, g in enumerate(weights):
            r.set_lng(w, g)
    return r


def _batch_instances(c, seed):
    mix = np.random.default_rng(c["instances"])   # the systems belong to the case, their starts to the seed
    sizes = [L for L in (16, 24, 32, 48) if L <= c["L_max"]]
    geo = [dict(L=int(mix.choice(sizes)), q=int(mix.choice((2, 4, 8, 10))), windows=c["windows"], overlap=0.75,
                walkers=c["walkers"]) for _ in range(c["instances"])]
    rng = np.random.default_rng(seed)
    spins = []
    for g in geo:
        W, starts = pk.window_layout(g["L"], g["windows"], 0.75)
        spins.append(_lattices(g["L"], g["q"], starts, W, g["walkers"], rng))
    return geo, spins


def _batch(c, seed):
    geo, spins = _batch_instances(c, seed)
    lnf = 2.0 ** c["lnf_log2"]
    weights = None
    if lnf < 1.0:
        a = pk.Batch([dict(g, seed=seed, instance=1000 + i, flat=(0, 1), lnf_final=1.5 * lnf,
                           sync_attempts=50 * g["L"] ** 2) for i, g in enumerate(geo)], spins, device=DEVICE)
        while a.run(8) != pk.CONVERGED:
            pass
        state = [[a.instance(i).state(w) for w in range(g["windows"] * g["walkers"])] for i, g in enumerate(geo)]
        spins = [np.stack([s["spins"] for s in st]) for st in state]
        weights = [[s["lng"] for s in st] for st in state]
    b = pk.Batch([dict(g, seed=seed, instance=i, lnf_init=lnf, fixed_lnf=1, sync_attempts=c["sweeps"] * g["L"] ** 2)
                  for i, g in enumerate(geo)], spins, device=DEVICE)
    b.walkin()
    if weights is None:
        b.run(2)
    else:
        for i, st in enumerate(weights):
            for w, g in enumerate(st):
                b.instance(i).set_lng(w, g)
    return b


def _batch_states(b):
    """The instances' state: the workspace behind the batch's own tables
    (which hold addresses and queue counters)."""
    tail = 0
    for geo, opts in b._desc:
        n = pk.workspace_bytes(geo["L"], geo["q"], geo["windows"], geo["overlap"], geo["walkers"], opts)
        tail += (n + 255) // 256 * 256
    return b.workspace[b.workspace.numel() - tail:]


def _trimers(nmol, box, walkers, seed, min_dist=0.85):
    """Trimers without overlaps: heads uniform, tails at unit distance along
    random directions, a molecule redrawn while a bead is too close to one of
    another molecule; all walkers at once."""
    rng = np.random.default_rng(seed)
    out = np.zeros((walkers, 3 * nmol, 3))
    for i in range(nmol):
        todo = np.arange(walkers)
        while len(todo):
            v = rng.normal(size=(2, len(todo), 3))
            v /= np.linalg.norm(v, axis=2, keepdims=True)
            head = rng.uniform(0.0, box, size=(len(todo), 3))
            beads = np.mod(np.stack([head, head + v[0], head + v[0] + v[1]], axis=1), box)
            ok = np.linalg.norm(v[0] + v[1], axis=1) > min_dist
            if i:
                d = np.abs(beads[:, :, None, :] - out[todo][:, None, :3 * i, :])
                d = np.minimum(d, box - d)
                ok &= (np.sum(d * d, axis=3).reshape(len(todo), -1).min(axis=1) >= min_dist ** 2)
            out[todo[ok], 3 * i:3 * i + 3] = beads[ok]
            todo = todo[~ok]
    x = out.astype(np.float32)
    x[x >= np.float32(box)] = 0.0
    return x


def _lipid_box(c):
    return float(np.float32(((3 * c["nlip"] + c["nsol"]) / 0.8) ** (1 / 3)))


def _lipids(nlip, nsol, box, nconf, seed, device):
    """Lipids and solvent on a jittered cubic lattice, each lipid on three
    consecutive sites of a row: float32 [nconf, np, 3] on `device`."""
    g = torch.Generator(device=device).manual_seed(seed)
    total = 3 * nlip + nsol
    n = math.ceil(total ** (1 / 3) - 1e-9)
    while n ** 3 < total or nlip > n * n * (n // 3):
        n += 1
    a = box / n
    per_row = n // 3
    slots = torch.rand(nconf, n * n * per_row, generator=g, device=device).argsort(dim=1)[:, :nlip]
    first = (slots // per_row) * n + 3 * (slots % per_row)
    sites = first[:, :, None] + torch.arange(3, device=device)
    turn = torch.rand(nconf, nlip, 1, generator=g, device=device) < 0.5
    sites = torch.where(turn, sites.flip(2), sites).reshape(nconf, 3 * nlip)
    key = torch.rand(nconf, n ** 3, generator=g, device=device)
    key.scatter_(1, sites, 2.0)
    sites = torch.cat([sites, key.argsort(dim=1)[:, :nsol]], dim=1)
    x = torch.stack([sites % n, (sites // n) % n, sites // (n * n)], dim=2).double() * a
    x = x + (torch.rand(x.shape, generator=g, device=device, dtype=torch.float64) - 0.5) * (0.1 * a)
    x = torch.remainder(x, box).float()
    return torch.where(x >= np.float32(box), torch.zeros_like(x), x)


def _structure_inputs(c, seed):
    """Configurations whose lipids sit denser in one half of the box, so that
    clusters of many sizes occur; lipid rows name the particles."""
    box = _lipid_box(c)
    x = _lipids(c["nlip"], c["nsol"], box, c["nconf"], seed, DEVICE)
    order = x[:, 0:3 * c["nlip"]:3, 2].argsort(dim=1)
    rows = (3 * order[:, :, None] + torch.arange(3, device=DEVICE)).to(torch.int32).contiguous()
    return x.contiguous(), rows, box


def _bootstrap_batch(c, seed):
    rng = np.random.default_rng(seed)
    W, starts = pk.window_layout(c["L"], c["windows"], 0.75)
    inst = [dict(L=c["L"], q=c["q"], windows=c["windows"], overlap=0.75, walkers=1, seed=seed, instance=i,
                 flat=(0, 1), lnf_final=1e-4, sync_attempts=100 * c["L"] ** 2) for i in range(c["runs"])]
    b = pk.Batch(inst, [_lattices(c["L"], c["q"], starts, W, 1, rng) for _ in inst], device=DEVICE)
    while b.run(16) != pk.CONVERGED:
        pass
    return b


def prepare(case, seed):
    c = case
    if c["kind"] == "potts":
        return c, _potts_run(c, seed)
    if c["kind"] == "batch":
        return c, _batch(c, seed)
    if c["kind"] == "trimer":
        x = _trimers(c["nmol"], c["box"], c["windows"] * c["walkers"], seed)
        r = pk.Rewl.trimer(c["nmol"], c["box"], c["e_min"], c["bin_w"], c["bins"], c["windows"], 0.75, c["walkers"],
                           x, device=DEVICE, seed=seed, lnf_init=2.0 ** -6, fixed_lnf=1, sync_attempts=c["sync"],
                           precision=c["precision"])
        r.walkin()
        return c, r
    if c["kind"] == "lipid":
        box = _lipid_box(c)
        x = _lipids(c["nlip"], c["nsol"], box, c["windows"] * c["walkers"], seed, "cpu").numpy()
        r = pk.Rewl.lipid(c["nlip"], c["nsol"], box, c["e_min"], 1.0, c["bins"], c["windows"], 0.75, c["walkers"], x,
                          device=DEVICE, seed=seed, lnf_init=2.0 ** -6, fixed_lnf=1, sync_attempts=c["sync"],
                          obs_bins=c["obs_bins"])
        r.walkin()
        return c, r
    if c["kind"] == "structure":
        return c, _structure_inputs(c, seed)
    if c["kind"] == "start":
        rng = np.random.default_rng(seed)
        return c, (rng.integers(0, c["q"], size=(c["windows"] * c["walkers"], c["L"] ** 2), dtype=np.int8), seed)
    return c, (_bootstrap_batch(c, seed), np.linspace(0.5, 1.5, TEMPERATURES))


def run(state):
    c, r = state
    if c["kind"] in ("potts", "trimer", "lipid"):
        r.run(c["attempts"])
        return r.workspace
    if c["kind"] == "batch":
        r.run(1)
        return _batch_states(r)
    if c["kind"] == "structure":
        return pk.lipid_structure(*r)
    if c["kind"] == "start":
        spins, seed = r
        new = pk.Rewl(c["L"], c["q"], c["windows"], 0.75, c["walkers"], spins, device=DEVICE, seed=seed)
        new.walkin()
        return new.workspace
    batch, temperatures = r
    return batch.bootstrap(c["nboot"], 7, temperatures)


# ---------------------------------------------------------------------------
# What a pass cannot do without.

def work(case):
    c = case
    if c["kind"] == "potts":
        W = math.ceil((2 * c["L"] ** 2 + 1) / (1 + 0.25 * (c["windows"] - 1)))
        nw = c["windows"] * c["walkers"]
        # 205 32-bit operations an attempt, nearly all of them the random words,
        # the energy change and the decision; every walker's rows in and out
        return dict(bytes=2 * nw * (c["L"] ** 2 + 12 * W), flops=205 * nw * c["attempts"])
    if c["kind"] == "batch":
        sizes = [L for L in (16, 24, 32, 48) if L <= c["L_max"]]
        N = sum(L * L for L in sizes) / len(sizes)
        nw = c["instances"] * c["windows"] * c["walkers"]
        W = 2 * N / (1 + 0.25 * (c["windows"] - 1))
        return dict(bytes=2 * nw * (N + 12 * W), flops=205 * nw * c["sweeps"] * N)
    if c["kind"] in ("trimer", "lipid"):
        nb = 3 * c["nmol"] if c["kind"] == "trimer" else 3 * c["nlip"] + c["nsol"]
        nw = c["windows"] * c["walkers"]
        W = c["bins"] / (1 + 0.25 * (c["windows"] - 1))
        row = 12 * nb + (0 if c["kind"] == "trimer" else 5 * nb + 12 * c["nlip"])
        # squared distances of a moved particle to all others, old and new place
        return dict(bytes=2 * nw * (row + 12 * W), flops=2 * (nb - 1) * 8 * nw * c["attempts"])
    if c["kind"] == "structure":
        M = c["nlip"]
        return dict(bytes=c["nconf"] * (36 * M + 12 * M + 64), flops=c["nconf"] * M * (M - 1) / 2 * 4 * 8)
    if c["kind"] == "start":
        N, nw = c["L"] ** 2, c["windows"] * c["walkers"]
        return dict(bytes=nw * (N + 4 * (2 * N + 1)) * 2, flops=205 * nw * N)
    B = 2 * c["L"] ** 2 + 1
    W = math.ceil(B / (1 + 0.25 * (c["windows"] - 1)))
    return dict(bytes=c["runs"] * c["windows"] * W * 8 + 16 * B + 32 * TEMPERATURES,
                flops=c["nboot"] * (c["runs"] * c["windows"] * W + 3 * 20 * B * TEMPERATURES))


# ---------------------------------------------------------------------------
# Outputs in 64 bits from the definition.

def _image(a, b, box):
    """b - a, the nearest image per axis (one wrap), taken in binary32."""
    box = np.float32(box)
    d = b - a
    d = np.where(d > box / 2, d - box, np.where(d < -box / 2, d + box, d))
    return d.astype(np.float64)


def _contacts(x, box):
    """Which lipids touch (a tail bead of each within 1.4), bool [nconf, M, M];
    x float32 [nconf, M, 3 beads, 3] on the GPU."""
    out = []
    for part in x.split(64):
        tails = part[:, :, 1:].flatten(1, 2)
        d = tails[:, None] - tails[:, :, None]
        d = torch.where(d > box / 2, d - box, torch.where(d < -box / 2, d + box, d)).double()
        near = (d * d).sum(dim=3) < 1.96
        M = part.shape[1]
        touch = near.view(-1, M, 2, M, 2).any(dim=4).any(dim=2)
        out.append(touch & ~torch.eye(M, dtype=torch.bool, device=x.device))
    return torch.cat(out).cpu().numpy()


def _record(x, touch, box):
    """Structural record of one configuration; x float32 [M, 3 beads, 3]."""
    M = len(x)
    bond = _image(x[:, 0], x[:, 1], box)
    cos2 = np.mean(bond ** 2 / np.sum(bond ** 2, axis=1, keepdims=True), axis=0)
    order = 1.5 * cos2 - 0.5
    axis = int(np.argmax(order))
    free = np.ones(M, dtype=bool)
    clusters, best = 0, []
    for r in range(M):
        if not free[r]:
            continue
        clusters += 1
        free[r] = False
        level, tree = [r], [(r, -1)]
        while level:
            rows = touch[level] & free
            found = np.flatnonzero(rows.any(axis=0))
            tree += [(int(j), level[int(np.argmax(rows[:, j]))]) for j in found]
            free[found] = False
            level = [int(j) for j in found]
        if len(tree) > len(best):
            best = tree
    u = np.zeros((M, 3, 3))
    for j, p in best:
        if p < 0:
            u[j, 0] = x[j, 0]
            known = 0
        else:
            for a, b in ((1, 1), (1, 2), (2, 1), (2, 2)):
                d = _image(x[p, a], x[j, b], box)
                if d @ d < 1.96:
                    u[j, b] = u[p, a] + d
                    known = b
                    break
        for a, b in {0: ((0, 1), (1, 2)), 1: ((1, 0), (1, 2)), 2: ((2, 1), (1, 0))}[known]:
            u[j, b] = u[j, a] + _image(x[j, a], x[j, b], box)
    beads = u[[j for j, _ in best]].reshape(-1, 3)
    Q = np.mean((beads - beads.mean(axis=0)) ** 2, axis=0)
    e = Q - Q.mean()
    return [order[axis], axis, clusters, len(best), *Q, 9.0 * np.sum(e ** 3) / np.sum(Q) ** 3]


def exact(case, seed):
    # The other outputs are a run's state (whole numbers and the weights its
    # own decisions led to) or averages over such runs.
    if case["kind"] != "structure" or case["nconf"] * case["nlip"] ** 2 > 4096 * 125 ** 2:
        return None
    x, rows, box = _structure_inputs(case, seed)
    x = torch.stack([p[r.long()] for p, r in zip(x, rows)])
    touch = _contacts(x, box)
    x = x.cpu().numpy()
    return np.array([_record(x[i], touch[i], box) for i in range(len(x))])
