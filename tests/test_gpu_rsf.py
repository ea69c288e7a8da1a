"""GPU RSF sampling cycle (Sec. II re-clone from a parent trajectory), block
spread sigma(N_R), MFTU and the Eq. 5 fidelity / radius-of-gyration
diagnostics, against the oracle on the same seeds and counters."""
import numpy as np
import pytest

from gpu_util import announce, rel_err, require_gpu
from paper_2206_05851_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _gpu_pair(groups, parents, seed, S, P, W, precision=32, two_streams=False, use_graph=False, noise_map=0):
    import torch
    from paper_2206_05851_amd import ra
    pstream = torch.cuda.Stream() if two_streams else None
    par = ra.Replicas([dict(g, n_replicas=1) for g in groups], seed, precision=precision, sample_every=P,
                      max_windows=W, tsf=True, noise_tag=1, stream=pstream, use_graph=use_graph,
                      noise_map=noise_map)
    par.init_chains(parents)
    rep = ra.Replicas(groups, seed, precision=precision, sample_every=S, max_windows=W, use_graph=use_graph,
                      noise_map=noise_map)
    return par, rep


def _oracle_pair(groups, parents, seed, S, P, W, ranges=None, noise_map=0):
    from oracle import ora
    par = ora.Oracle([dict(g, n_replicas=1) for g in groups], seed, P, W, tsf=True, noise_map=noise_map)
    par.set_tag(ora.TAG_PARENT)
    par.init_chains(parents)
    rep = ora.Oracle(groups, seed, S, W, noise_map=noise_map)
    for g, r in (ranges or {}).items():
        rep.set_replicas(g, *r)
    return par, rep


def _run_both(groups, parents, seed, S, P, W, **kw):
    import torch
    gp, gr = _gpu_pair(groups, parents, seed, S, P, W, **kw)
    gr.rsf_cycle(gp, W, P)
    isf, _, tsf, _ = gp.average_forces(tsf=True)
    rsf, rstd = gr.average_forces()
    torch.cuda.synchronize()
    gp.sync_status()
    gr.sync_status()
    op, orr = _oracle_pair(groups, parents, seed, S, P, W, noise_map=kw.get("noise_map", 0))
    orr.rsf_cycle(op, W, P)
    oisf, _, otsf, _ = op.average_forces(tsf=True)
    orsf, orstd = orr.average_forces()
    return (gp, gr, isf.cpu().numpy(), tsf.cpu().numpy(), rsf.cpu().numpy(), rstd.cpu().numpy()), \
           (op, orr, oisf, otsf, orsf, orstd)


@pytest.mark.parametrize("two_streams,noise_map", [(False, 0), (True, 0), (False, 1), (True, 1)])
def test_rsf_cycle_matches_oracle(two_streams, noise_map):
    gs = [wl.group(24, 48, 1e-4, wl.FENE, 1.0, 60.0, wl.SHEAR, wl.wi_to_rate(40.0, 24), stream_id=3),
          wl.group(10, 20, 1e-3, wl.HOOKEAN, 1.0, 0.0, wl.UNIAXIAL, wl.wi_to_rate(0.4, 10), stream_id=9)]
    ps = [wl.equilibrium_parent(24, wl.FENE, 1.0, 60.0, seed=5), wl.equilibrium_parent(10, seed=6)]
    S, P, W = 40, 30, 5
    announce("rsf cycle two_streams=%s noise_map=%d" % (two_streams, noise_map))
    (gp, gr, isf, tsf, rsf, rstd), (op, orr, oisf, otsf, orsf, orstd) = _run_both(gs, ps, 11, S, P, W,
                                                                                   two_streams=two_streams,
                                                                                   noise_map=noise_map)
    e = [rel_err(isf, oisf, 1e-3), rel_err(tsf, otsf, 1e-3), rel_err(rsf, orsf, 1e-3), rel_err(rstd, orstd, 1e-3)]
    announce("isf %.2e tsf %.2e rsf %.2e std %.2e" % tuple(e))
    assert max(e) < 1e-4
    # MFTU of each estimate through the parent context (window = parent_steps)
    import torch
    for prof, oprof in ((isf, oisf), (tsf, otsf), (rsf, orsf)):
        _, rs = gp.bell_rates(torch.from_numpy(prof).cuda(), 1e-3, 0.1)
        m = gp.mftu(rs).cpu().numpy()
        _, ors = op.bell_rates(oprof, 1e-3, 0.1)
        assert rel_err(m, op.mftu(ors)) < 1e-5


def test_rsf_cycle_fp64_matches_oracle_tightly():
    gs = [wl.group(10, 32, 1e-3, wl.HOOKEAN, 1.0, 0.0, wl.PLANAR, 0.2)]
    ps = [wl.equilibrium_parent(10, seed=1)]
    announce("rsf cycle fp64")
    (_, _, isf, tsf, rsf, rstd), (_, _, oisf, otsf, orsf, orstd) = _run_both(gs, ps, 3, 50, 20, 4, precision=64)
    assert max(rel_err(isf, oisf), rel_err(tsf, otsf), rel_err(rsf, orsf), rel_err(rstd, orstd)) < 1e-10


def test_rsf_cycle_graph_replay_is_bitwise_eager():
    gs = [wl.group(30, 40, 1e-4, wl.FENE, 1.0, 80.0, wl.PLANAR, 0.5)]
    ps = [wl.equilibrium_parent(30, wl.FENE, 1.0, 80.0, seed=2)]
    out = []
    for graph in (False, True):
        gp, gr = _gpu_pair(gs, ps, 4, 25, 25, 6, use_graph=graph, two_streams=graph)
        gr.rsf_cycle(gp, 3, 25)
        gr.rsf_cycle(gp, 3, 25)
        out.append((gp.average_forces(tsf=True)[2].cpu().numpy(), gr.average_forces()[0].cpu().numpy()))
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1])


def test_block_sigma_definition_and_oracle():
    import torch
    gs = [wl.group(12, 200, 1e-3, wl.FENE, 1.0, 50.0, wl.UNIAXIAL, 0.1)]
    ps = [wl.equilibrium_parent(12, wl.FENE, 1.0, 50.0, seed=8)]
    (gp, gr, *_), (op, orr, *_) = _run_both(gs, ps, 21, 30, 30, 3)
    smp = gr.samples()[0].cpu().numpy()          # [W][R][N-1]
    for nr in (10, 20, 40, 64, 200, 300):
        sig = gr.block_sigma(nr).cpu().numpy()
        torch.cuda.synchronize()
        B = 200 // nr
        if B >= 2:
            bm = smp[:, :B * nr].reshape(3, B, nr, 11).mean(axis=2)
            assert rel_err(sig, bm.std(axis=1, ddof=1), 1e-12) < 1e-12
        else:
            assert np.all(sig == 0.0)
        assert rel_err(sig, orr.block_sigma(nr), 1e-3) < 1e-4


def test_mftu_events_matches_oracle():
    # first windows bit-exact (the event decisions are FP64 on both sides from
    # the same counters) and the censored mean; two groups, one of them longer
    # than a wavefront of springs; a short cap so some trials are censored
    import torch
    from oracle import ora
    from paper_2206_05851_amd import ra
    gs = [wl.group(12, 4, 1e-2, stream_id=3), wl.group(90, 4, 1e-2, stream_id=8)]
    S, W = 10, 6
    rng = np.random.default_rng(5)
    mean = rng.uniform(0.0, 20.0, size=(W, 11 + 89))
    o = ora.Oracle(gs, 21, S, W)
    rates, _ = o.bell_rates(mean, k0=2e-3, x_dagger=0.1)
    announce("MFTU by event sampling: 500 trials, caps 40 and 4000")
    rep = ra.Replicas(gs, 21, sample_every=S, max_windows=W)
    for cap in (40, 4000):
        m_ref, f_ref = o.mftu_events(rates, 500, cap)
        m, f = rep.mftu_events(torch.from_numpy(rates).cuda(), 500, cap)
        f = f.cpu().numpy()
        assert np.array_equal(f, f_ref)
        assert np.allclose(m.cpu().numpy(), m_ref, rtol=1e-13, atol=0)
        if cap == 40:
            assert np.any(f < 0) and np.any(f >= 0)
    rep.close()


def test_mftu_events_threshold_edges_and_wide_chain_match_oracle():
    # The event test as an integer threshold on the 52-bit uniform: rates of
    # 0, below one 2^-53 step, ordinary, and large enough that 1 - exp(-k S dt)
    # rounds to 1 (every draw an event), against the oracle's FP64 test on the
    # same counters; and a chain whose per-window thresholds (599 springs x 8
    # windows) exceed the LDS table, which takes the per-draw FP64 path.
    import torch
    from oracle import ora
    from paper_2206_05851_amd import ra
    S, W = 10, 8
    rng = np.random.default_rng(11)
    gs = [wl.group(9, 2, 1e-2, stream_id=4)]
    rates = rng.uniform(0.0, 0.3, size=(W, 8))
    rates[:, 0] = 0.0
    rates[:, 1] = 1e-20
    rates[3, 2] = 1e3
    rates[5, :] = 1e-3
    o = ora.Oracle(gs, 31, S, W)
    rep = ra.Replicas(gs, 31, sample_every=S, max_windows=W)
    announce("MFTU by events: threshold edges")
    m_ref, f_ref = o.mftu_events(rates, 300, 50)
    m, f = rep.mftu_events(torch.from_numpy(rates).cuda(), 300, 50)
    assert np.array_equal(f.cpu().numpy(), f_ref)
    assert np.allclose(m.cpu().numpy(), m_ref, rtol=1e-13, atol=0)
    assert np.all(f_ref <= 3)   # window 3 holds a certain event
    rep.close()
    gw = [wl.group(600, 2, 1e-2, stream_id=9)]
    rates = rng.uniform(0.0, 2e-3, size=(W, 599))
    o = ora.Oracle(gw, 32, S, W)
    rep = ra.Replicas(gw, 32, sample_every=S, max_windows=W)
    announce("MFTU by events: 599 springs, per-draw path")
    m_ref, f_ref = o.mftu_events(rates, 24, 40)
    m, f = rep.mftu_events(torch.from_numpy(rates).cuda(), 24, 40)
    assert np.array_equal(f.cpu().numpy(), f_ref)
    assert np.allclose(m.cpu().numpy(), m_ref, rtol=1e-13, atol=0)
    assert np.any(f_ref >= 0)
    rep.close()


@pytest.mark.parametrize("cap,trials,rate", [(1, 1, 0.5), (511, 3, 2e-3), (513, 40, 4e-4), (32769, 5, 2e-5),
                                             (70000, 9, 1e-5)])
def test_mftu_events_at_the_edges_of_rounds_and_segments(cap, trials, rate):
    # caps about the 512 windows of a round and the segments that a ticket takes
    # (one round up to 65536 windows, two above), few and many trials, two groups;
    # whole numbers: the windows are equal
    import torch
    from oracle import ora
    from paper_2206_05851_amd import ra
    gs = [wl.group(3, 2, 1e-2, stream_id=6), wl.group(6, 2, 1e-2, stream_id=2)]
    S, W = 10, 3
    rates = np.random.default_rng(cap).uniform(0.0, rate, size=(W, 7))
    o = ora.Oracle(gs, 77, S, W)
    rep = ra.Replicas(gs, 77, sample_every=S, max_windows=W)
    announce("MFTU by events: cap %d, %d trials" % (cap, trials))
    m_ref, f_ref = o.mftu_events(rates, trials, cap)
    m, f = rep.mftu_events(torch.from_numpy(rates).cuda(), trials, cap)
    assert np.array_equal(f.cpu().numpy(), f_ref)
    assert np.allclose(m.cpu().numpy(), m_ref, rtol=1e-13, atol=0)
    rep.close()


@pytest.mark.parametrize("cap,trials", [(4095, 300), (4096, 3), (4097, 300), (4096 + 512, 65), (9000, 600)])
def test_mftu_events_of_many_groups_match_oracle(cap, trials):
    # 40 groups, each with rates of its own from certain to none over the head, the
    # queue's segments and the cap, chains of one to seven springs: workgroups go from
    # group to group, claims hold up to `trials` tickets, more than a workgroup's threads
    import torch
    from oracle import ora
    from paper_2206_05851_amd import ra
    ng = 40
    groups = [wl.group(2 + g % 7, 1, 1e-3, stream_id=100 + g) for g in range(ng)]
    mean = [0.3 * 10.0 ** (g % 6) for g in range(ng)]               # windows to an event
    S = 10
    rates = np.concatenate([np.full((3, g["n_beads"] - 1), 0.0 if i % 13 == 12 else 1.0 / (mean[i] * (g["n_beads"] - 1) * S * 1e-3))
                            for i, g in enumerate(groups)], axis=1)
    rates *= np.random.default_rng(1).uniform(0.5, 1.5, rates.shape)
    small = [g for g in range(ng)][: ng if trials < 100 else 12]     # the oracle's share
    groups = [groups[g] for g in small]
    rates = np.ascontiguousarray(rates[:, : sum(g["n_beads"] - 1 for g in groups)])
    rep = ra.Replicas(groups, 13, sample_every=S, max_windows=1)
    o = ora.Oracle(groups, 13, S, 1)
    announce("event sampling, %d groups, %d trials, cap %d" % (len(groups), trials, cap))
    m_ref, f_ref = o.mftu_events(rates, trials, cap)
    m, f = rep.mftu_events(torch.from_numpy(rates).cuda(), trials, cap)
    assert np.array_equal(f.cpu().numpy(), f_ref)
    assert np.allclose(m.cpu().numpy(), m_ref, rtol=1e-13, atol=0)
    rep.close()


def test_mftu_events_of_one_slow_group_take_the_whole_chip():
    # 64 groups of which one holds nearly all the work, against that group alone: 1.6 times
    # its time; with a fixed share of the workgroups per group it was 17
    import time
    import torch
    from paper_2206_05851_amd import ra
    groups = [wl.group(50, 1, 1e-3, stream_id=g) for g in range(64)]
    rates = torch.full((1, 64 * 49), 1.0 / (100 * 49 * 1e-2), dtype=torch.float64)
    rates[:, 20 * 49:21 * 49] = 1.0 / (1e5 * 49 * 1e-2)
    best = []
    for gs, r in ((groups, rates), (groups[20:21], rates[:, 20 * 49:21 * 49].contiguous())):
        rep = ra.Replicas(gs, 3, sample_every=10, max_windows=1)
        r = r.cuda()
        rep.mftu_events(r, 1024, 1 << 17)
        t_best = 1e9
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            rep.mftu_events(r, 1024, 1 << 17)
            torch.cuda.synchronize()
            t_best = min(t_best, time.perf_counter() - t)
        best.append(t_best)
        rep.close()
    announce("event sampling: 64 groups %.2f ms, the slow one alone %.2f ms" % (best[0] * 1e3, best[1] * 1e3))
    assert best[0] < 5 * best[1]


def test_mftu_events_of_one_context_may_overlap():
    # two captured calls on one context, with outputs of their own, replayed at the same
    # time on two streams: the first windows of the calls made one after the other
    import torch
    from paper_2206_05851_amd import ra
    groups = [wl.group(50, 1, 1e-3, stream_id=5), wl.group(20, 1, 1e-3, stream_id=6)]
    T, cap = 1024, 1 << 18
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        rep = ra.Replicas(groups, 9, sample_every=10, max_windows=1)
    rng = np.random.default_rng(3)
    rates = [torch.from_numpy(10.0 ** rng.uniform(-5.5, -4.0, (2, 68))).cuda() for _ in range(2)]
    torch.cuda.synchronize()
    graphs, outs, want = [], [], []
    for r in rates:
        with torch.cuda.stream(s):
            want.append(rep.mftu_events(r, T, cap))
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            outs.append(rep.mftu_events(r, T, cap))
        graphs.append(g)
    other = torch.cuda.Stream()
    announce("event sampling, two calls at once")
    for _ in range(3):
        for o in outs:
            o[0].zero_()
            o[1].zero_()
        torch.cuda.synchronize()
        for g, st in zip(graphs, (s, other)):
            with torch.cuda.stream(st):
                g.replay()
        torch.cuda.synchronize()
        for (m, f), (m_ref, f_ref) in zip(outs, want):
            assert torch.equal(f, f_ref)
            assert torch.equal(m, m_ref)


def test_conformation_after_cycle_matches_oracle():
    gs = [wl.group(40, 16, 1e-4, wl.FENE, 1.0, 100.0, wl.SHEAR, wl.wi_to_rate(50.0, 40), stream_id=1),
          wl.group(7, 9, 1e-3, wl.HOOKEAN, 1.0, 0.0, wl.QUIESCENT, 0.0, stream_id=2)]
    ps = [wl.equilibrium_parent(40, wl.FENE, 1.0, 100.0, seed=3), wl.equilibrium_parent(7, seed=4)]
    (gp, gr, *_), (op, orr, *_) = _run_both(gs, ps, 6, 60, 40, 3)
    dbar, rg2, srg2, db = [t.cpu().numpy() for t in gr.conformation(per_bead=True)]
    odbar, org2, osrg2, odb = orr.conformation(per_bead=True)
    e = [rel_err(dbar, odbar, 1e-2), rel_err(rg2, org2, 1e-2), rel_err(srg2, osrg2, 1e-2),
         np.max(np.abs(db - odb))]
    announce("conformation dbar %.2e rg2 %.2e src %.2e d_bead abs %.2e" % tuple(e))
    assert max(e[:3]) < 1e-4 and e[3] < 1e-4
    assert np.all(dbar > 0)
    # right after a fresh clone every replica is its source (FP32 rounding only)
    from paper_2206_05851_amd import ra
    fresh = ra.Replicas(gs, 6, sample_every=10, max_windows=1)
    fresh.init_chains(ps)
    d0, r0, s0 = [t.cpu().numpy() for t in fresh.conformation()]
    assert np.max(d0) < 1e-5
    assert rel_err(r0, np.repeat(s0, [16, 9], axis=0)) < 1e-5


def test_reclone_and_cycle_errors():
    from paper_2206_05851_amd import ra
    g = wl.group(10, 8, 1e-3)
    p = wl.equilibrium_parent(10, seed=0)
    rep = ra.Replicas([g], 0, sample_every=10, max_windows=4, checkpoint_every=10, max_steps=40)
    par = ra.Replicas([dict(g, n_replicas=1)], 0, sample_every=10, max_windows=4, noise_tag=1)
    with pytest.raises(ra.RAError, match="RA_ESTATE"):
        rep.reclone(par)                          # parent not initialised
    par.init_chains([p])
    other = ra.Replicas([wl.group(11, 1, 1e-3)], 0, sample_every=10, max_windows=4)
    other.init_chains([wl.equilibrium_parent(11, seed=0)])
    with pytest.raises(ra.RAError, match="RA_EINVAL"):
        rep.reclone(other)                        # chain length differs
    f64 = ra.Replicas([dict(g, n_replicas=1)], 0, precision=64, sample_every=10, max_windows=4)
    f64.init_chains([p])
    with pytest.raises(ra.RAError, match="RA_EINVAL"):
        rep.reclone(f64)                          # precision differs
    with pytest.raises(ra.RAError, match="RA_EINVAL"):
        rep.rsf_cycle(par, 2, 7)                  # parent samples every 10, not 7
    with pytest.raises(ra.RAError, match="RA_EINVAL"):
        rep.rsf_cycle(par, 5, 10)                 # window capacity of 4
    rep.rsf_cycle(par, 2, 10)
    rep.step(5)
    with pytest.raises(ra.RAError, match="RA_EINVAL"):
        rep.reclone(par)                          # mid-window
    rep.step(5)
    mean, _ = rep.average_forces()
    import torch
    with pytest.raises(ra.RAError, match="RA_ESTATE"):
        rep.backward(mean, torch.zeros_like(mean))   # no adjoint through a re-clone
    rep.init_chains([p])
    rep.step(10)
    rep.backward(mean[:1].contiguous(), torch.zeros_like(mean[:1]))
    rep.sync_status()


def test_rsf50_full_size_first_window_per_replica():
    # The rsf50 workload in full (FENE N=50 in shear at Wi=50, the parent and
    # 1000 replicas, 20 windows of 750 steps), launched as bench.py runs it
    # (parent on its own stream, graphs on, dual launches); the oracle replays
    # the parent's first two windows and replicas 0..3 of the first window.
    import torch
    from oracle import ora
    from paper_2206_05851_amd import ra
    groups, parents, run = wl.rsf50()
    g = groups[0]
    S, P, W = run["sample_every"], run["parent_steps"], run["n_windows"]
    announce("rsf50 full size")
    pstream = torch.cuda.Stream()
    par = ra.Replicas([dict(g, n_replicas=1)], run["seed"], sample_every=P, max_windows=W, tsf=True, noise_tag=1,
                      stream=pstream, use_graph=True)
    par.init_chains(parents)
    rep = ra.Replicas(groups, run["seed"], sample_every=S, max_windows=W, use_graph=True)
    rep.rsf_cycle(par, W, P)
    smp = rep.samples()[0].cpu().numpy()
    psmp, ptsf = [t[0].cpu().numpy() for t in par.samples(tsf=True)]
    par.sync_status()
    rep.sync_status()
    assert np.all(np.isfinite(smp)) and smp.shape == (W, 1000, 49)
    op = ora.Oracle([dict(g, n_replicas=1)], run["seed"], P, 2, tsf=True)
    op.set_tag(ora.TAG_PARENT)
    op.init_chains(parents)
    orr = ora.Oracle(groups, run["seed"], S, 2)
    orr.set_replicas(0, 0, 4)
    orr.rsf_cycle(op, 2, P)
    osmp, otsf = op.samples(tsf=True)
    e = [rel_err(psmp[:2], osmp[0], 1.0), rel_err(ptsf[:2], otsf[0], 1.0),
         rel_err(smp[:2, :4], orr.samples()[0], 1.0)]
    announce("rsf50 windows 0-1: parent %.2e, parent TSF %.2e, replicas 0-3 %.2e" % tuple(e))
    assert max(e) < 1e-4
