"""GPU adjoint (ra_backward, reverse mode over checkpointed segments) against
the oracle's forward-mode pathwise tangents on the same seeds (up to the
differentiation workload's tile and horizon), and against central finite
differences of the FP64 oracle with common random numbers at the full
differentiation workload (N=100, 4096 replicas, 2000 steps)."""
import numpy as np
import pytest

from gpu_util import announce, cpu_threads, oracle_mean_parallel, require_gpu, run_gpu, run_oracle
from paper_2206_05851_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    require_gpu()


def _grad_pair(groups, parents, seed, steps, S, K, k0=1e-6, xd=0.1, wseed=0, rate_scale=1e5, tile_policy=0,
               noise_map=0):
    import torch
    W = steps // S
    nspr = sum(g["n_beads"] - 1 for g in groups)
    rng = np.random.default_rng(wseed)
    gm = rng.normal(size=(W, nspr))
    gr = rng.normal(size=(W, nspr)) * rate_scale
    rep = run_gpu(groups, parents, seed, steps, S, checkpoint_every=K, max_steps=steps,
                  tile_policy=tile_policy, noise_map=noise_map)
    assert rep.checkpoint_interval() == (1 if K == -1 else K)
    mean, _ = rep.average_forces()
    g_gpu = rep.backward(mean, torch.from_numpy(gm).cuda(), torch.from_numpy(gr).cuda(), k0, xd)
    g_gpu = g_gpu.cpu().numpy()
    rep.sync_status()
    o = run_oracle(groups, parents, seed, steps, S, tangents=True, noise_map=noise_map)
    g_ref = o.backward(gm, gr, k0, xd)
    return g_gpu, g_ref


def _check(g_gpu, g_ref, rtol):
    scale = np.maximum(np.abs(g_ref), 1e-3 * np.max(np.abs(g_ref)))
    err = np.max(np.abs(g_gpu - g_ref) / scale)
    announce("adjoint max rel err %.2e" % err)
    assert err < rtol, (g_gpu, g_ref)


@pytest.mark.parametrize("spring,flow,N,policy", [(wl.FENE, wl.UNIAXIAL, 12, 0), (wl.FENE, wl.SHEAR, 33, 0),
                                                  (wl.FENE, wl.SHEAR, 33, 1002), (wl.HOOKEAN, wl.PLANAR, 10, 1003),
                                                  (wl.FENE, wl.PLANAR, 150, 0), (wl.FENE, wl.UNIAXIAL, 300, 0)])
def test_adjoint_matches_oracle_tangents_200_steps(spring, flow, N, policy):
    # policy 0 is the cost model's tile; 1000 + m forces m beads per lane
    b = 40.0 if spring == wl.FENE else 0.0
    g = wl.group(N, 64, 1e-4, spring, 1.3, b, flow, 30.0 if flow == wl.SHEAR else 0.8)
    parent = wl.equilibrium_parent(N, spring, 1.3, b, seed=N)
    announce("adjoint N=%d spring=%d flow=%d policy=%d" % (N, spring, flow, policy))
    g_gpu, g_ref = _grad_pair([g], [parent], 17, 200, 50, 50, tile_policy=policy)
    _check(g_gpu, g_ref, 1e-4)
    if spring == wl.HOOKEAN:
        assert g_gpu[0, 2] == 0.0


@pytest.mark.parametrize("N,K", [(50, 50), (50, 7), (50, -1), (130, 25)])
def test_adjoint_under_noise_map_one(N, K):
    # noise map 1: the segment recompute rebuilds the fourth-normal carry at
    # each segment start (K = 7 and 25 start segments off the 4-step grid);
    # N = 130 runs 3 beads per lane
    g = wl.group(N, 64, 1e-4, wl.FENE, 1.3, 40.0, wl.UNIAXIAL, 0.8, stream_id=2)
    parent = wl.equilibrium_parent(N, wl.FENE, 1.3, 40.0, seed=N + 1)
    announce("adjoint noise map 1 N=%d K=%d" % (N, K))
    g_gpu, g_ref = _grad_pair([g], [parent], 23, 200, 50, K, noise_map=1)
    _check(g_gpu, g_ref, 1e-4)


def test_adjoint_batch_and_guard():
    N = 6
    guard = np.zeros((N, 3))
    guard[1:, 0] = np.cumsum([0.5, np.sqrt(0.9995) * 10.0, 1.0, np.sqrt(0.95) * 10.0, 0.7])
    gs = [wl.group(N, 32, 1e-4, wl.FENE, 1.0, 100.0, wl.UNIAXIAL, 0.1, stream_id=2),
          wl.group(24, 40, 1e-4, wl.FENE, 1.0, 50.0, wl.SHEAR, 10.0, stream_id=7)]
    ps = [guard, wl.equilibrium_parent(24, wl.FENE, 1.0, 50.0, seed=4)]
    announce("adjoint batch with guard")
    g_gpu, g_ref = _grad_pair(gs, ps, 5, 150, 50, 30)
    _check(g_gpu, g_ref, 1e-4)


@pytest.mark.parametrize("K", [1, 7, -1])
def test_adjoint_checkpoint_interval_keeps_the_gradient(K):
    # K = 1 keeps every state, so the backward reads each reverse step's state
    # from its checkpoint instead of recomputing it; any interval must give the
    # oracle's tangents and, up to FP32 summation order, the gradient of K = 50.
    # K = -1 (automatic) keeps every state when they fit, as here.
    N = 6
    guard = np.zeros((N, 3))
    guard[1:, 0] = np.cumsum([0.5, np.sqrt(0.9995) * 10.0, 1.0, np.sqrt(0.95) * 10.0, 0.7])
    gs = [wl.group(N, 32, 1e-4, wl.FENE, 1.0, 100.0, wl.UNIAXIAL, 0.1, stream_id=2),
          wl.group(24, 40, 1e-4, wl.FENE, 1.0, 50.0, wl.SHEAR, 10.0, stream_id=7)]
    ps = [guard, wl.equilibrium_parent(24, wl.FENE, 1.0, 50.0, seed=4)]
    announce("adjoint checkpoint interval %d" % K)
    g_k, g_ref = _grad_pair(gs, ps, 5, 150, 50, K)
    _check(g_k, g_ref, 1e-4)
    g_50, _ = _grad_pair(gs, ps, 5, 150, 50, 50)
    assert np.max(np.abs(g_k - g_50) / np.maximum(np.abs(g_50), 1e-3 * np.max(np.abs(g_50)))) < 1e-5


def test_adjoint_every_state_kept_multi_bead_lanes():
    # the no-recompute backward (automatic interval = 1) with 3 beads per lane
    N = 150
    g = wl.group(N, 64, 1e-4, wl.FENE, 1.3, 40.0, wl.PLANAR, 0.8)
    parent = wl.equilibrium_parent(N, wl.FENE, 1.3, 40.0, seed=N)
    announce("adjoint N=150, every state kept")
    g_gpu, g_ref = _grad_pair([g], [parent], 17, 200, 50, -1)
    _check(g_gpu, g_ref, 1e-4)


def test_adjoint_long_horizon():
    N = 20
    g = wl.group(N, 128, 1e-4, wl.FENE, 1.0, 100.0, wl.UNIAXIAL, wl.wi_to_rate(4.0, N))
    parent = wl.equilibrium_parent(N, wl.FENE, 1.0, 100.0, seed=6)
    announce("adjoint 2000 steps")
    g_gpu, g_ref = _grad_pair([g], [parent], 9, 2000, 100, 100)
    _check(g_gpu, g_ref, 1e-3)


def test_autograd_function_uses_adjoint():
    import torch
    from paper_2206_05851_amd import ra
    N = 16
    g = wl.group(N, 64, 1e-4, wl.FENE, 1.0, 60.0, wl.UNIAXIAL, 0.5)
    parent = wl.equilibrium_parent(N, wl.FENE, 1.0, 60.0, seed=1)
    params = torch.tensor([[0.5, 1.0, 60.0]], dtype=torch.float64, requires_grad=True)
    mean, rates = ra.ReplicaAverage.apply(params, [g], [parent], 200, 3, 50, 1e-6, 0.1, 50)
    rng = np.random.default_rng(2)
    wm = torch.from_numpy(rng.normal(size=tuple(mean.shape))).cuda()
    wr = torch.from_numpy(rng.normal(size=tuple(rates.shape)) * 1e5).cuda()
    J = (wm * mean).sum() + (wr * rates).sum()
    J.backward()
    o = run_oracle([g], [parent], 3, 200, 50, tangents=True)
    ref = o.backward(wm.cpu().numpy(), wr.cpu().numpy(), 1e-6, 0.1)
    _check(params.grad.numpy(), ref, 1e-4)


@pytest.mark.parametrize("noise_map", [0, 1])
def test_adjoint_c4_tile_matches_oracle_tangents(noise_map):
    # The differentiation workload's shape (N = 100, b = 100, uniaxial Wi = 4,
    # dt = 1e-4, 2000 steps, checkpoints every 100 steps, 2 beads per lane) on
    # its first 64 replicas: the counters carry the global replica index, so
    # these are replicas 0..63 of the full run. Objective with both terms
    # (replica-averaged tension profile and Bell rates).
    groups, parents, run = wl.adjoint100(n_replicas=64)
    steps, S, K = run["steps"], run["sample_every"], run["checkpoint_every"]
    announce("C4 tile adjoint vs oracle tangents: N=100 R=64 2000 steps K=100 noise map %d" % noise_map)
    g_gpu, g_ref = _grad_pair(groups, parents, run["seed"], steps, S, K, run["k0"], run["x_dagger"], wseed=4,
                              noise_map=noise_map)
    rep = run_gpu(groups, parents, run["seed"], 0, S, max_windows=steps // S, checkpoint_every=K,
                  max_steps=steps, noise_map=noise_map)
    assert rep.tile_info()[0][0] == 2
    rep.close()
    _check(g_gpu, g_ref, 1e-3)


@pytest.mark.timeout(600)
def test_adjoint_full_size_against_oracle_fd_with_crn():
    # Full differentiation workload (4096 replicas, noise map 1 as in the
    # benchmark): the FP32 reverse-mode gradient of J = sum gm * mean against
    # central finite differences of the FP64 oracle with the same counters
    # (common random numbers), relative step 1e-4. The oracle runs its
    # replicas on host threads.
    import torch
    groups, parents, run = wl.adjoint100()
    steps, S, K = run["steps"], run["sample_every"], run["checkpoint_every"]
    W = steps // S
    rng = np.random.default_rng(3)
    gm = rng.normal(size=(W, 99))
    announce("C4 full size adjoint: N=100 R=4096 2000 steps, noise map 1")
    rep = run_gpu(groups, parents, run["seed"], steps, S, checkpoint_every=K, max_steps=steps, noise_map=1)
    mean, _ = rep.average_forces()
    grad = rep.backward(mean, torch.from_numpy(gm).cuda(), None).cpu().numpy()[0]
    rep.sync_status()
    rep.close()

    def J(over):
        g = dict(groups[0], **over)
        m = oracle_mean_parallel([g], parents, run["seed"], steps, S, noise_map=1)
        return float((m * gm).sum())

    h = 1e-4
    for p, key in enumerate(("rate", "H", "b")):
        th = groups[0][key]
        announce("oracle FD d/d%s on %d host threads" % (key, cpu_threads()))
        fd = (J({key: th * (1 + h)}) - J({key: th * (1 - h)})) / (2 * h * th)
        announce("d/d%s adjoint %.6e oracle fd %.6e" % (key, grad[p], fd))
        assert abs(grad[p] - fd) <= 1e-3 * max(abs(fd), 1e-3 * np.max(np.abs(grad))), key


@pytest.mark.parametrize("R,noise_map,K,S,steps", [(5, 0, 1, 7, 35), (5, 1, 1, 7, 30), (5, 1, 3, 9, 29), (5, 0, 5, 4, 23),
                                                   (5, 0, 1, 1, 3), (520, 0, 1, 13, 26), (520, 1, 4, 13, 26),
                                                   (1100, 1, 1, 10, 20), (1100, 0, 6, 10, 20)])
def test_adjoint_of_mixed_widths_equals_each_group_alone(R, noise_map, K, S, steps):
    # 1-4 beads per lane in one batch: one launch over all items up to 2048 of them
    # (R = 5, 520), one per kernel above (R = 1100), states kept at every step
    # or recomputed, segments shorter and longer than the sweep's read-ahead and
    # ending off the windows; against contexts of one group. The sums differ by
    # FP32 order at most (tiles may differ): as between checkpoint intervals.
    import torch
    Ns = (20, 100, 180, 230)
    groups = [wl.group(N, R, 1e-4, wl.FENE if i % 2 else wl.HOOKEAN, 1.2, 70.0 if i % 2 else 0.0, wl.SHEAR, 3.0,
                       stream_id=i) for i, N in enumerate(Ns)]
    parents = [wl.equilibrium_parent(g["n_beads"], g["spring"], 1.2, g["b"], seed=40 + i)
               for i, g in enumerate(groups)]
    W = steps // S
    gm = torch.from_numpy(np.random.default_rng(4).normal(size=(W, sum(Ns) - 4))).cuda()

    def grad(gs, ps, cot):
        rep = run_gpu(gs, ps, 31, steps, S, checkpoint_every=K, max_steps=steps, noise_map=noise_map)
        mean, _ = rep.average_forces()
        g = rep.backward(mean, cot.contiguous()).cpu().numpy()
        smp = [x.cpu().numpy() for x in rep.samples()]
        rep.sync_status()
        return g, smp

    announce("adjoint mixed widths R=%d map=%d K=%d" % (R, noise_map, K))
    g_all, smp_all = grad(groups, parents, gm)
    o = 0
    for i, N in enumerate(Ns):
        g_one, smp_one = grad([groups[i]], [parents[i]], gm[:, o:o + N - 1])
        assert np.array_equal(smp_all[i], smp_one[0])
        assert np.max(np.abs(g_all[i] - g_one[0]) / np.maximum(np.abs(g_one[0]), 1e-3 * np.max(np.abs(g_one)))) < 1e-5
        o += N - 1


@pytest.mark.parametrize("N,R,K,S,steps,noise_map", [(50, 6, 1, 128, 260, 0), (50, 6, 300, 129, 258, 1), (50, 6, 131, 1, 133, 0),
                                                     (64, 2100, 5, 8, 24, 1), (64, 2100, 1, 3, 9, 0), (150, 2100, 7, 10, 20, 0),
                                                     (300, 4, 1, 127, 254, 0), (600, 3, 140, 64, 192, 2), (1000, 2, 1, 1, 130, 0),
                                                     (1000, 2, 9, 20, 40, 2)])
def test_adjoint_sweep_cut_at_windows_and_partial_sums(N, R, K, S, steps, noise_map):
    # sampled states and the 128-step partial sums at, before and after each other,
    # with one bead per lane in short lists and with wide lanes (cut sweeps), and in lists
    # of more than 2048 items (packed rows): the oracle's tangents within the
    # bound of the other lengths here
    g = wl.group(N, R, 1e-4, wl.FENE, 1.3, 40.0, wl.UNIAXIAL, 0.8, stream_id=1)
    parent = wl.equilibrium_parent(N, wl.FENE, 1.3, 40.0, seed=N + 3)
    announce("adjoint sweep N=%d R=%d K=%d S=%d steps=%d map=%d" % (N, R, K, S, steps, noise_map))
    g_gpu, g_ref = _grad_pair([g], [parent], 29, steps, S, K, noise_map=noise_map)
    _check(g_gpu, g_ref, 1e-4)


def test_adjoint_of_kept_states_is_faster_than_recomputing_wide_lanes():
    # 1000 beads: the sweep over kept states against the sweep with its recompute,
    # which is a forward more. Measured ratio 0.46; with the sweep's steps unrolled
    # past the instruction cache it was 0.66.
    import time
    import torch
    g = wl.group(1000, 4, 1e-4, wl.FENE, 1.3, 40.0, wl.UNIAXIAL, 0.8)
    parent = wl.equilibrium_parent(1000, wl.FENE, 1.3, 40.0, seed=8)
    best = {}
    for K in (1, 20):
        rep = run_gpu([g], [parent], 3, 200, 50, checkpoint_every=K, max_steps=200)
        mean, _ = rep.average_forces()
        one = torch.ones_like(mean)
        for _ in range(3):
            rep.backward(mean, one)
        best[K] = 1e9
        for _ in range(5):
            torch.cuda.synchronize()
            t = time.perf_counter()
            for _ in range(10):
                rep.backward(mean, one)
            torch.cuda.synchronize()
            best[K] = min(best[K], time.perf_counter() - t)
        rep.sync_status()
    announce("adjoint of 1000 beads, kept states %.0f us, recomputed %.0f us" % (best[1] * 1e5, best[20] * 1e5))
    assert best[1] < 0.56 * best[20]
