"""GPU pair-interaction kernel (the collapsed-polymer force field of Sec. II:
rest-length harmonic backbone springs with the signed Eq. 4 force, LJ
self-association between non-adjacent beads) against the oracle on the same
seeds and counters."""
import numpy as np
import pytest

from gpu_util import announce, rel_err, require_gpu, run_gpu, run_oracle
from paper_2206_05851_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _paper_group(N, R, flow=wl.SHEAR, rate=30.0, **kw):
    return wl.group(N, R, 1e-5, wl.HARMONIC, 400.0, 0.0, flow, rate, rest_length=2.0, lj_eps=1.0,
                    lj_rmin=2.0, **kw)


CASES = [
    ("paper N=50 shear", lambda: _paper_group(50, 6)),
    ("paper N=12 quiescent, 5 replicas per wave", lambda: _paper_group(12, 13, wl.QUIESCENT, 0.0)),
    ("FENE + LJ N=20 planar", lambda: wl.group(20, 7, 1e-4, wl.FENE, 1.0, 50.0, wl.PLANAR, 0.5, lj_eps=0.5,
                                               lj_rmin=1.2)),
    ("Hookean + LJ N=8", lambda: wl.group(8, 17, 1e-4, wl.HOOKEAN, 2.0, 0.0, wl.UNIAXIAL, 0.3, lj_eps=0.3,
                                          lj_rmin=1.0)),
    ("harmonic, no LJ, N=64", lambda: wl.group(64, 3, 1e-5, wl.HARMONIC, 400.0, 0.0, wl.SHEAR, 30.0,
                                               rest_length=2.0)),
    # each non-bonded pair is evaluated once, from the bead that reaches its
    # partner in at most N/2 steps around the segment: odd N, a full
    # wavefront (N = 64, the pairs at N/2 met from both ends), and the
    # shortest chains (N = 3: one pair, reached across the wrap-around;
    # N = 2: none)
    ("paper N=13 odd, 4 replicas per wave", lambda: _paper_group(13, 9)),
    ("paper N=64, full wavefront", lambda: _paper_group(64, 3)),
    ("Hookean + LJ N=3", lambda: wl.group(3, 11, 1e-4, wl.HOOKEAN, 2.0, 0.0, wl.SHEAR, 1.0, lj_eps=0.5,
                                          lj_rmin=1.0)),
    ("Hookean + LJ N=2", lambda: wl.group(2, 40, 1e-4, wl.HOOKEAN, 2.0, 0.0, wl.SHEAR, 1.0, lj_eps=0.5,
                                          lj_rmin=1.0)),
]


def _parent(g, seed):
    if g["spring"] == wl.HARMONIC or (g["lj_eps"] > 0 and g["lj_rmin"] >= 2.0):
        return wl.collapsed_parent(g["n_beads"], seed=seed)
    return wl.collapsed_parent(g["n_beads"], seed=seed, spacing=g["lj_rmin"] * 1.1, jitter=0.02)


def _floor(g):
    # signed spring forces cross zero: errors are taken relative to the
    # thermal force scale sqrt(H kT) where the force is smaller than it
    return float(np.sqrt(g["H"] * g["kT"]))


@pytest.mark.parametrize("name,mk", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("precision", [32, 64])
def test_pair_kernel_matches_oracle(name, mk, precision):
    g = mk()
    p = _parent(g, 3)
    steps, S = 300, 50
    announce("pair %s precision %d" % (name, precision))
    rep = run_gpu([g], [p], 7, steps, S, precision=precision, tsf=True)
    assert rep.kernel_family() == 2
    smp, tsf = rep.samples(tsf=True)
    bonds = rep.bonds()[0].cpu().numpy()
    rep.sync_status()
    o = run_oracle([g], [p], 7, steps, S, tsf=True)
    osmp, otsf = o.samples(tsf=True)
    obonds = np.diff(o.positions()[0], axis=1)
    tol = 1e-4 if precision == 32 else 1e-9
    fl = _floor(g)
    e = [rel_err(smp[0].cpu().numpy(), osmp[0], fl), rel_err(tsf[0].cpu().numpy(), otsf[0], fl),
         np.max(np.abs(bonds - obonds))]
    announce("samples %.2e tsf %.2e bonds abs %.2e" % tuple(e))
    assert e[0] < tol and e[1] < tol and e[2] < tol
    if g["spring"] == wl.HARMONIC:
        assert np.min(smp[0].cpu().numpy()) < 0.0   # signed spring force (Eq. 4)


def test_pair_batch_invariance_and_graph():
    gs = [dict(_paper_group(50, 5), stream_id=4), dict(_paper_group(9, 20, wl.QUIESCENT, 0.0), stream_id=8)]
    ps = [_parent(gs[0], 1), _parent(gs[1], 2)]
    both = run_gpu(gs, ps, 3, 200, 40, use_graph=True)
    a = both.samples()
    alone = [run_gpu([g], [p], 3, 200, 40).samples()[0] for g, p in zip(gs, ps)]
    for x, y in zip(a, alone):
        assert np.array_equal(x.cpu().numpy(), y.cpu().numpy())


def test_pair_rsf_cycle_matches_oracle():
    from oracle import ora
    from paper_2206_05851_amd import ra
    g = _paper_group(50, 12)
    p = _parent(g, 5)
    S, P, W = 60, 40, 3
    par = ra.Replicas([dict(g, n_replicas=1)], 9, sample_every=P, max_windows=W, tsf=True, noise_tag=1)
    par.init_chains([p])
    rep = ra.Replicas([g], 9, sample_every=S, max_windows=W)
    rep.rsf_cycle(par, W, P)
    isf, _, tsf, _ = [t.cpu().numpy() for t in par.average_forces(tsf=True)]
    rsf, rstd = [t.cpu().numpy() for t in rep.average_forces()]
    dbar, rg2, srg2 = [t.cpu().numpy() for t in rep.conformation()]
    op = ora.Oracle([dict(g, n_replicas=1)], 9, P, W, tsf=True)
    op.set_tag(ora.TAG_PARENT)
    op.init_chains([p])
    orr = ora.Oracle([g], 9, S, W)
    orr.rsf_cycle(op, W, P)
    oisf, _, otsf, _ = op.average_forces(tsf=True)
    orsf, orstd = orr.average_forces()
    odbar, org2, osrg2 = orr.conformation()
    fl = _floor(g)
    e = [rel_err(isf, oisf, fl), rel_err(tsf, otsf, fl), rel_err(rsf, orsf, fl), rel_err(rstd, orstd, fl),
         rel_err(dbar, odbar, 1e-2), rel_err(rg2, org2, 1e-2), rel_err(srg2, osrg2, 1e-2)]
    announce("pair rsf: " + " ".join("%.1e" % x for x in e))
    assert max(e) < 1e-4


def test_pair_full_size_collapsed50_first_window_per_replica():
    # The collapsed50 workload in full (1000 replicas, 20 windows of 750
    # steps); the oracle replays the parent and replicas 0..3 of the first
    # window with the same counters.
    from oracle import ora
    from paper_2206_05851_amd import ra
    groups, parents, run = wl.collapsed50()
    g = groups[0]
    S, P, W = run["sample_every"], run["parent_steps"], run["n_windows"]
    announce("collapsed50 full size")
    par = ra.Replicas([dict(g, n_replicas=1)], run["seed"], sample_every=P, max_windows=W, tsf=True, noise_tag=1)
    par.init_chains(parents)
    rep = ra.Replicas(groups, run["seed"], sample_every=S, max_windows=W, use_graph=True)
    rep.rsf_cycle(par, W, P)
    smp = rep.samples()[0].cpu().numpy()
    rsf, _ = rep.average_forces()
    rsf = rsf.cpu().numpy()
    par.sync_status()
    rep.sync_status()
    assert np.all(np.isfinite(rsf)) and smp.shape == (W, 1000, 49)
    op = ora.Oracle([dict(g, n_replicas=1)], run["seed"], P, 1, tsf=True)
    op.set_tag(ora.TAG_PARENT)
    op.init_chains(parents)
    orr = ora.Oracle(groups, run["seed"], S, 1)
    orr.set_replicas(0, 0, 4)
    orr.rsf_cycle(op, 1, P)
    err = rel_err(smp[0, :4], orr.samples()[0][0], _floor(g))
    announce("collapsed50 window 0 replicas 0-3 rel err %.2e" % err)
    assert err < 1e-4


@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("N", [2, 3, 4, 5, 7, 8, 12, 32, 33, 50, 63, 64])
def test_pair_wavefronts_per_item_keep_the_bits(N, precision):
    # four, two and one wavefronts per work item (up to 512, up to 1280 or 768, and
    # more items): the first replicas agree to the bit. Calls of 1-9 steps end
    # inside and at the edges of a round of shared noise.
    from paper_2206_05851_amd import ra
    spring, H, b = [(wl.HARMONIC, 50.0, 0.0), (wl.FENE, 3.0, 20.0), (wl.HOOKEAN, 2.0, 0.0)][N % 3]
    P = 64 // N
    few = 2 * P + 1
    out = []
    for items in (3, 600, 1300):
        R = few if items == 3 else items * P
        g = wl.group(N, R, 1e-5, spring, H, b, wl.SHEAR, 5.0, rest_length=2.0 if spring == wl.HARMONIC else 0.0,
                     lj_eps=0.7, lj_rmin=2.0 if spring == wl.HARMONIC else 1.0, stream_id=3)
        p = _parent(g, 11)
        announce("pair wavefronts N=%d precision=%d items=%d" % (N, precision, items))
        rep = ra.Replicas([g], 13, precision=precision, sample_every=7, max_windows=5, tsf=True)
        rep.init_chains([p])
        for c in (1, 2, 3, 4, 5, 9, 8, 3):   # 35
            rep.step(c)
        smp, tsf = rep.samples(tsf=True)
        out.append([x.cpu().numpy() for x in (smp[0][:, :few], tsf[0][:, :few], rep.bonds()[0][:few])])
        rep.sync_status()
        assert np.all(np.isfinite(out[-1][2]))
    for other in out[1:]:
        for x, y in zip(out[0], other):
            assert np.array_equal(x, y)


@pytest.mark.parametrize("N", [2, 9, 12, 13])
def test_pair_short_chains_share_fewer_wavefronts_with_the_same_bits(N):
    # up to 12 beads two wavefronts step an item up to 768 items, above that one, longer
    # chains up to 1280; two beads have no pair: the same bits as without LJ
    from paper_2206_05851_amd import ra
    P = 64 // N
    out = []
    for items, eps in ((700, 0.7), (1000, 0.7), (1290, 0.7)) + (((700, 0.0),) if N == 2 else ()):
        g = wl.group(N, items * P, 1e-5, wl.HARMONIC, 50.0, 0.0, wl.SHEAR, 5.0, rest_length=2.0, lj_eps=eps, lj_rmin=2.0,
                     stream_id=3)
        announce("pair short chains N=%d items=%d" % (N, items))
        rep = ra.Replicas([g], 13, sample_every=7, max_windows=3)
        rep.init_chains([_parent(g, 11)])
        for c in (1, 4, 9, 7):   # 21
            rep.step(c)
        out.append(rep.bonds()[0][:5 * P].cpu().numpy())
        rep.sync_status()
    for other in out[1:]:
        assert np.array_equal(out[0], other)
