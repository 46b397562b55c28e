"""GPU tests of the variants around the plain FP64 path: FP32 pair terms,
nonlinear EOS, the surrogate network, batched replicas, graph replay, SEM,
failure codes, and the full 1M-particle size."""
import math

import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dp():
    import torch
    assert torch.cuda.is_available()
    import paper_1507_06643_amd as m
    return m


def _gpu_state(s):
    q, p, e, st = s.get_state()
    return q.cpu().numpy(), p.cpu().numpy(), e.cpu().numpy(), st


def _one_step_vs_oracle(dp, n, box, periodic=(1, 1, 1), prime=3, **kw):
    """Advance `prime` steps on the GPU, then compare one more GPU step with
    the oracle's step from the same state; returns the max errors (q/L, p,
    eps/mean eps) and the energy records."""
    okw = {k: v for k, v in kw.items() if k not in ("precision", "theta_mode")}
    eps0 = kw.pop("eps0", 100.0)
    okw.pop("eps0", None)
    q, p, e = W.equilibrium_state(n, box, seed=n + 7, eps0=eps0)
    s = dp.System(dp.Config(n=n, box=list(box), periodic=periodic, **kw), q, p, e)
    s.step(prime)
    qs, ps, es, st = _gpu_state(s)
    S = O.State(O.make_params(n, box, periodic=periodic, step=st, **okw), qs, ps, es)
    rc, _ = S.step(1)
    assert rc == 0
    s.step(1)
    qg, pg, eg, _ = _gpu_state(s)
    dq = qg - S.q
    for k in range(3):
        if periodic[k]:
            dq[:, k] -= box[k] * np.rint(dq[:, k] / box[k])
    errs = (np.abs(dq).max() / max(box), np.abs(pg - S.p).max(),
            np.abs(eg - S.eps).max() / np.abs(S.eps).mean())
    en, eo = s.energies(), S.energies()
    s.close()
    return errs, en, eo


# ---------------------------------------------------------------------------
# FP32 pair terms: per-step error against the FP64 oracle is stated here.
# FP32 carries ~6e-8 relative rounding per pair term; a momentum change of
# ~N_nb * |dp_ij| ~ 1 gives ~1e-6 absolute per step.
# ---------------------------------------------------------------------------
FP32_TOL = {"q": 1e-9, "p": 2e-5, "eps": 2e-7}


def test_fp32_step_error_vs_fp64_oracle(dp):
    n = 20000
    L = W.cubic_side(n)
    (eq, ep, ee), en, eo = _one_step_vs_oracle(dp, n, [L] * 3, precision=dp.FP32, dt=0.005)
    assert eq < FP32_TOL["q"] and ep < FP32_TOL["p"] and ee < FP32_TOL["eps"], (eq, ep, ee)
    # the conserved sums stay FP64-exact in structure: energy/momentum agree closely
    assert abs(en[3] - eo[3]) < 1e-9 * abs(eo[3])


def test_fp32_conserves_energy_without_conservative_force(dp):
    n = 4000
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=51)
    s = dp.System(dp.Config(n=n, box=[L] * 3, a=0.0, precision=dp.FP32), q, p, e)
    E0 = s.energies()[3]
    s.step(300)
    h = s.history()
    assert np.abs(h[:, 3] - E0).max() < 1e-12 * E0
    assert np.abs(h[:, 4:7]).max() < 1e-10
    s.close()


# ---------------------------------------------------------------------------
# Nonlinear (Einstein) EOS with Newton inversion.
# ---------------------------------------------------------------------------
def test_theta_newton_matches_oracle(dp):
    n = 200
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=3, eps0=25.0)
    s = dp.System(dp.Config(n=n, box=[L] * 3, eos=dp.EOS_EINSTEIN), q, p, e)
    P = O.make_params(n, [L] * 3, eos=1)
    th = np.exp(np.linspace(np.log(0.05), np.log(100.0), 3001))
    eps = O.eos_energy(P, th)
    got_eps = s.eos_energy(th).cpu().numpy()
    assert np.abs(got_eps / eps - 1).max() < 4e-15
    got, its = s.theta(eps, mode=dp.THETA_NEWTON)
    want, oits = O.theta_newton(P, eps)
    assert np.abs(got.cpu().numpy() / want - 1).max() < 1e-13
    assert its.cpu().numpy().max() < 60
    s.close()


def test_step_parity_einstein_eos(dp):
    n = 3000
    L = W.cubic_side(n)
    P = O.make_params(10, [5, 5, 5], eos=1)
    eps1 = float(O.eos_energy(P, 1.0)[0])
    (eq, ep, ee), en, eo = _one_step_vs_oracle(dp, n, [L] * 3, eos=dp.EOS_EINSTEIN, dt=0.005,
                                               eps0=eps1)
    assert max(eq, ep, ee) < 1e-12, (eq, ep, ee)
    assert abs(en[8] - eo[8]) < 1e-12 * eo[8]


# ---------------------------------------------------------------------------
# Surrogate network: GPU gradients vs the oracle's FP64 backprop, BF16
# inference vs the oracle forward on the BF16-rounded weights, training, and
# the error of the surrogate temperature against Newton's.
# ---------------------------------------------------------------------------
def _bf16_round(w):
    w = np.asarray(w, dtype=np.float32)
    u = w.view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) >> 16
    return (u.astype(np.uint32) << 16).view(np.float32).astype(np.float64)


@pytest.fixture(scope="module")
def eos_system(dp):
    n = 200
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=4, eps0=25.0)
    s = dp.System(dp.Config(n=n, box=[L] * 3, eos=dp.EOS_EINSTEIN, theta_mode=dp.THETA_MLP), q, p, e)
    yield s
    s.close()


def test_mlp_gradients_match_oracle(dp, eos_system):
    rng = np.random.default_rng(8)
    w = rng.normal(0, 0.5, 1153).astype(np.float32)
    eos_system.mlp_set(w, np.array([3.0, 3.0, 0.0, 2.3]))
    x = rng.uniform(-1, 1, 3000).astype(np.float32)
    t = rng.uniform(-1, 1, 3000).astype(np.float32)
    loss, g = eos_system.mlp_grad(x, t)
    lo, go = O.mlp_loss_grad(w.astype(np.float64), x.astype(np.float64), t.astype(np.float64))
    assert loss == pytest.approx(lo, rel=1e-5)
    scale = np.abs(go).max()
    assert np.abs(g - go).max() < 2e-5 * scale


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65, 4095, 4096, 4097, 20001])
def test_mlp_gradients_at_the_edges_of_the_sample_tiles(dp, eos_system, n):
    """Batches around 16 samples (a wave's), 64 (a block's) and 4096 (one
    pass of every block).  FP32 sums in at most a few hundred roundings each:
    2e-5 of the largest entry, as for the whole gradient above."""
    rng = np.random.default_rng(100 + n)
    w = rng.normal(0, 0.5, 1153).astype(np.float32)
    eos_system.mlp_set(w, np.array([3.0, 3.0, 0.0, 2.3]))
    x = rng.uniform(-1, 1, n).astype(np.float32)
    t = rng.uniform(-1, 1, n).astype(np.float32)
    loss, g = eos_system.mlp_grad(x, t)
    lo, go = O.mlp_loss_grad(w.astype(np.float64), x.astype(np.float64), t.astype(np.float64))
    assert loss == pytest.approx(lo, rel=1e-5)
    assert np.abs(g - go).max() < 2e-5 * np.abs(go).max()


def test_mlp_training_batch_wraps_around_the_samples(dp, eos_system):
    """A batch of 103 out of 50 samples takes each twice and the first three
    once more: from the same start, its mean loss is that of those samples."""
    kw = dict(nsamples=50, iters=1, lr=3e-3, seed=5)
    one = eos_system.mlp_train(batch=50, **kw)[0].astype(np.float64)
    three = eos_system.mlp_train(batch=3, **kw)[0].astype(np.float64)
    both = eos_system.mlp_train(batch=103, **kw)[0].astype(np.float64)
    assert both == pytest.approx((2 * 50 * one + 3 * three) / 103, rel=1e-6)


def _as_inferred(w):
    """The weights as inference uses them: W2 (the matrix-core layer) rounded
    to BF16, the input and output layers FP32."""
    out = np.asarray(w, dtype=np.float32).astype(np.float64)
    out[64:64 + 1024] = _bf16_round(np.asarray(w, dtype=np.float32)[64:64 + 1024])
    return out


def test_mlp_bf16_inference_matches_oracle_forward(dp, eos_system):
    rng = np.random.default_rng(9)
    w = rng.normal(0, 0.5, 1153).astype(np.float32)
    eos_system.mlp_set(w, np.array([3.0, 3.0, 0.0, 2.3]))
    x = np.concatenate([rng.uniform(-1, 1, 1000), [-1.0, 1.0, 0.0]]).astype(np.float32)
    y = eos_system.mlp_eval(x).cpu().numpy()
    # oracle forward on the weights as inference uses them, activations FP64:
    # the BF16 rounding of the first hidden layer on the GPU (relative 2^-9
    # per unit) bounds the difference
    yo = O.mlp_forward(_as_inferred(w), x.astype(np.float64))
    err = np.abs(y - yo).max() / max(1.0, np.abs(yo).max())
    print(f"BF16 inference vs FP64 forward: max |dy| / max |y| = {err:.2e}")
    assert err < 0.01
    # operand-layout check: the same weights with W2 transposed (a swapped
    # A/B operand) or with the hidden units permuted give a much larger error
    wt = _as_inferred(w)
    w2 = wt[64:64 + 1024].reshape(32, 32)
    wt_T = wt.copy()
    wt_T[64:64 + 1024] = w2.T.reshape(-1)
    err = np.abs(y - yo).mean()
    assert err < 0.2 * np.abs(y - O.mlp_forward(wt_T, x.astype(np.float64))).mean()


def test_mlp_training_and_surrogate_accuracy(dp, eos_system):
    curve = eos_system.mlp_train(nsamples=10**6, iters=20000, batch=4096, lr=3e-3, seed=5)
    assert curve[-1] < 1e-3 * curve[0]
    assert curve[-1] < 1e-5
    P = O.make_params(10, [5, 5, 5], eos=1)
    th = np.exp(np.linspace(np.log(0.2), np.log(20.0), 20001))
    eps = O.eos_energy(P, th)
    net, _ = eos_system.theta(eps, mode=dp.THETA_MLP)
    rel = np.abs(net.cpu().numpy() / th - 1)
    print(f"surrogate theta over [0.2, 20]: max rel error {rel.max():.2e}, "
          f"rms {np.sqrt((rel ** 2).mean()):.2e}")
    assert rel.max() < 0.01, rel.max()
    polished, its = eos_system.theta(eps, mode=dp.THETA_MLP_NEWTON)
    assert np.abs(polished.cpu().numpy() / th - 1).max() < 1e-13
    newton, its0 = eos_system.theta(eps, mode=dp.THETA_NEWTON)
    # the network start saves Newton iterations
    assert its.cpu().numpy().mean() < its0.cpu().numpy().mean()
    # outside the training range the surrogate mode falls back to Newton
    out = np.array([0.5, 5000.0])
    got, it_out = eos_system.theta(out, mode=dp.THETA_MLP)
    want, _ = O.theta_newton(P, out)
    assert np.abs(got.cpu().numpy() / want - 1).max() < 1e-13
    assert it_out.cpu().numpy().min() > 0


def test_surrogate_inside_sweep2_matches_theta_kernel(dp, eos_system):
    """In the learned-EOS modes sweep 2 evaluates the network for its own
    particles.  Per particle, the 1/T_i it leaves equal 1/theta of the
    stand-alone theta kernel for the same internal energies bit for bit; in
    the surrogate mode theta agrees with the oracle's FP64 forward of the same
    network within the BF16 rounding of the matrix-core layer, and in the
    Newton-polished mode with the oracle's Newton inversion to rounding."""
    eos_system.mlp_train(nsamples=10**6, iters=4000, batch=4096, lr=3e-3, seed=6)
    n = 4000
    L = W.cubic_side(n)
    P = O.make_params(10, [5, 5, 5], eos=1)
    eps1 = float(O.eos_energy(P, 1.0)[0])
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=95, eps0=eps1)
    w, norm = eos_system.mlp_get()
    for mode in (dp.THETA_MLP, dp.THETA_MLP_NEWTON):
        s = dp.System(dp.Config(n=n, box=[L] * 3, eos=dp.EOS_EINSTEIN, theta_mode=mode,
                                dt=0.005), q, p, e)
        s.mlp_set(w, norm)
        s.step(3)
        _, _, eg, _ = s.get_state()
        eg = eg.cpu().numpy()
        inv_t = s.debug_inv_temperature().cpu().numpy()
        th, _ = s.theta(eg, mode=mode)
        th = th.cpu().numpy()
        assert np.array_equal(inv_t, 1.0 / th)
        tint = n / inv_t.sum()
        assert abs(s.energies()[8] / tint - 1) < 1e-13
        if mode == dp.THETA_MLP:
            lo, hi = math.exp(norm[0] - norm[1]), math.exp(norm[0] + norm[1])
            inr = (eg >= lo) & (eg <= hi)
            assert inr.sum() > 0.99 * n
            x = np.clip((np.log(eg) - norm[0]) / norm[1], -1.0, 1.0).astype(np.float32)
            yo = O.mlp_forward(_as_inferred(w), x.astype(np.float64))
            th_o = np.exp(norm[2] + norm[3] * yo)
            rel = np.abs(th[inr] / th_o[inr] - 1)
            print(f"sweep-2 surrogate theta vs oracle forward: max rel {rel.max():.2e}")
            assert rel.max() < 1e-2
        else:
            th_n, _ = O.theta_newton(P, eg)
            assert np.abs(th / th_n - 1).max() < 1e-13
        s.close()


def test_full_size_one_step_parity_learned_eos(dp):
    """N = 1,048,576, the Einstein EOS with the surrogate as Newton's
    starting point (Newton polishes theta to a few ulp, as the oracle's
    Newton does): one step matches the oracle to 1e-12."""
    n = 1_048_576
    L = W.cubic_side(n)
    P = O.make_params(10, [5, 5, 5], eos=1)
    eps1 = float(O.eos_energy(P, 1.0)[0])
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=n + 11, eps0=eps1)
    s = dp.System(dp.Config(n=n, box=[L] * 3, eos=dp.EOS_EINSTEIN,
                            theta_mode=dp.THETA_MLP_NEWTON, dt=0.005), q, p, e)
    s.mlp_train(nsamples=10**6, iters=2000, batch=4096, lr=3e-3, seed=11)
    s.step(2)
    qs, ps, es, st = _gpu_state(s)
    S = O.State(O.make_params(n, [L] * 3, eos=1, dt=0.005, step=st), qs, ps, es)
    rc, _ = S.step(1)
    assert rc == 0
    s.step(1)
    qg, pg, eg, _ = _gpu_state(s)
    dq = qg - S.q
    dq -= L * np.rint(dq / L)
    errs = (np.abs(dq).max() / L, np.abs(pg - S.p).max(), np.abs(eg - S.eps).max() / S.eps.mean())
    assert max(errs) < 1e-12, errs
    en, eo = s.energies(), S.energies()
    assert abs(en[3] - eo[3]) < 1e-12 * abs(eo[3])
    assert abs(en[8] - eo[8]) < 1e-12 * abs(eo[8])
    s.close()


# ---------------------------------------------------------------------------
# Batched replicas: each replica equals the single system built from its own
# parameters, bit for bit; graph replay equals eager stepping bit for bit.
# ---------------------------------------------------------------------------
def test_batched_replicas_match_single_systems(dp):
    sizes, seeds = W.replica_sizes(6, 500, 3000, seed=77)
    cfgs, qs, ps, es = [], [], [], []
    for r, (nr, sd) in enumerate(zip(sizes, seeds)):
        L = W.cubic_side(int(nr))
        q, p, e = W.equilibrium_state(int(nr), [L] * 3, seed=1000 + r)
        cfgs.append(dp.Config(n=int(nr), box=[L] * 3, seed=int(sd), replica=r))
        qs.append(q); ps.append(p); es.append(e)
    b = dp.System(cfgs, np.concatenate(qs), np.concatenate(ps), np.concatenate(es))
    b.step(15)
    qb, pb, eb, st = _gpu_state(b)
    enb = b.energies()
    for r in range(len(cfgs)):
        s = dp.System(cfgs[r], qs[r], ps[r], es[r])
        s.step(15)
        q1, p1, e1, _ = _gpu_state(s)
        lo, hi = b.offsets[r], b.offsets[r + 1]
        assert np.array_equal(qb[lo:hi], q1)
        assert np.array_equal(pb[lo:hi], p1)
        assert np.array_equal(eb[lo:hi], e1)
        assert np.array_equal(enb[r], s.energies())
        s.close()
    b.close()


def test_batched_replicas_smaller_than_a_wave_match_single_systems(dp):
    """Replicas of fewer particles than a force-pass wave serves (16), so that
    one wave meets up to five replicas, next to larger ones: each replica
    still equals its own single system bit for bit."""
    sizes = [600, 7, 3, 12, 2, 20, 5, 9, 300]
    cfgs, qs, ps, es = [], [], [], []
    for r, nr in enumerate(sizes):
        L = W.cubic_side(nr) if nr >= 300 else 3.95
        q, p, e = W.equilibrium_state(nr, [L] * 3, seed=1500 + r)
        cfgs.append(dp.Config(n=nr, box=[L] * 3, seed=40 + r, replica=r))
        qs.append(q); ps.append(p); es.append(e)
    b = dp.System(cfgs, np.concatenate(qs), np.concatenate(ps), np.concatenate(es))
    b.step(12)
    qb, pb, eb, _ = _gpu_state(b)
    enb = b.energies()
    for r in range(len(cfgs)):
        s = dp.System(cfgs[r], qs[r], ps[r], es[r])
        s.step(12)
        q1, p1, e1, _ = _gpu_state(s)
        lo, hi = b.offsets[r], b.offsets[r + 1]
        assert np.array_equal(qb[lo:hi], q1), r
        assert np.array_equal(pb[lo:hi], p1), r
        assert np.array_equal(eb[lo:hi], e1), r
        assert np.array_equal(enb[r], s.energies(), equal_nan=True), r
        s.close()
    b.close()


@pytest.mark.parametrize("nrep", [14, 42])
@pytest.mark.parametrize("kw", [dict(), dict(precision=1), dict(model=1),
                                dict(eos=1, theta_mode=1), dict(project=True)])
def test_tile_shapes_give_the_same_bits(dp, nrep, kw):
    """Batches of about 28,000 and 85,000 particles run tiles of 64 and of 128;
    their replicas alone, tiles of 32.  States, observables and records agree
    bit for bit (replicas that end inside a tile, one open along x)."""
    sizes, seeds = W.replica_sizes(nrep, 500, 3500, seed=9)
    cfgs, qs, ps, es = [], [], [], []
    for r, (nr, sd) in enumerate(zip(sizes, seeds)):
        L = W.cubic_side(int(nr))
        box, per = ([1.6 * L, L / 1.25, L / 1.28], [0, 1, 1]) if r == 1 else ([L] * 3, [1, 1, 1])
        q, p, e = W.equilibrium_state(int(nr), box, seed=900 + r)
        cfgs.append(dp.Config(n=int(nr), box=box, periodic=per, seed=int(sd), replica=r, dt=0.01,
                              **kw))
        qs.append(q); ps.append(p); es.append(e)
    net = np.random.default_rng(3).normal(0, 0.3, 1153).astype(np.float32)

    def system(*args):
        s = dp.System(*args)
        if kw.get("theta_mode"):
            s.mlp_set(net, np.array([5.0, 3.0, 0.0, 2.3]))
        return s

    b = system(cfgs, np.vstack(qs), np.vstack(ps), np.concatenate(es))
    b.step(5)
    qb, pb, eb, _ = [x.cpu().numpy() if hasattr(x, "cpu") else x for x in b.get_state()]
    hb = b.history(8)
    for r in sorted({0, 1, nrep // 2, nrep - 1}):
        s = system(cfgs[r], qs[r], ps[r], es[r])
        s.step(5)
        lo, hi = b.offsets[r], b.offsets[r + 1]
        q1, p1, e1, _ = [x.cpu().numpy() if hasattr(x, "cpu") else x for x in s.get_state()]
        assert np.array_equal(qb[lo:hi], q1), r
        assert np.array_equal(pb[lo:hi], p1), r
        assert np.array_equal(eb[lo:hi], e1), r
        assert np.array_equal(hb[:, r], s.history(8)), r
        s.close()
    b.close()


def test_batched_256_replicas_one_step_vs_oracle(dp):
    """The batched workload itself (256 replicas, sizes uniform in
    [500, 8000] at density 3, one seed per replica, dt = 0.01): after 3 steps
    of the whole batch, one more batched step matches the oracle's step of the
    smallest, the largest and the median-size replica from the same state at
    1e-12 (Sec. 3.2.1: every replica is an independent system)."""
    sizes, seeds = W.replica_sizes(256, 500, 8000, seed=20260103)
    cfgs, qs, ps, es = [], [], [], []
    for r, (nr, sd) in enumerate(zip(sizes, seeds)):
        L = W.cubic_side(int(nr))
        q, p, e = W.equilibrium_state(int(nr), [L] * 3, seed=30000 + r)
        cfgs.append(dp.Config(n=int(nr), box=[L] * 3, dt=0.01, seed=int(sd), replica=r))
        qs.append(q); ps.append(p); es.append(e)
    b = dp.System(cfgs, np.concatenate(qs), np.concatenate(ps), np.concatenate(es))
    b.step(3)
    qb, pb, eb, st = _gpu_state(b)
    b.step(1)
    q1, p1, e1, _ = _gpu_state(b)
    b.close()
    order = np.argsort(sizes, kind="stable")
    for r in (int(order[0]), int(order[-1]), int(order[len(order) // 2])):
        lo, hi = b.offsets[r], b.offsets[r + 1]
        n, L = int(sizes[r]), W.cubic_side(int(sizes[r]))
        S = O.State(O.make_params(n, [L] * 3, dt=0.01, seed=int(seeds[r]), replica=r, step=st),
                    qb[lo:hi], pb[lo:hi], eb[lo:hi])
        rc, _ = S.step(1)
        assert rc == 0
        dq = q1[lo:hi] - S.q
        dq -= L * np.rint(dq / L)
        assert np.abs(dq).max() / L < 1e-12, (r, n)
        assert np.abs(p1[lo:hi] - S.p).max() < 1e-12, (r, n)
        assert np.abs(e1[lo:hi] - S.eps).max() / np.abs(S.eps).mean() < 1e-12, (r, n)


def test_graph_replay_equals_eager(dp):
    n = 5000
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=61)
    a = dp.System(dp.Config(n=n, box=[L] * 3), q, p, e)
    g = dp.System(dp.Config(n=n, box=[L] * 3), q, p, e)
    a.step(12)
    g.step_graph(4, 3)
    sa, sg = _gpu_state(a), _gpu_state(g)
    for x, y in zip(sa[:3], sg[:3]):
        assert np.array_equal(x, y)
    assert sa[3] == sg[3] == 12
    # eager work between replays, then more replays
    g.step(2)
    g.step_graph(4, 2)
    a.step(10)
    sa, sg = _gpu_state(a), _gpu_state(g)
    for x, y in zip(sa[:3], sg[:3]):
        assert np.array_equal(x, y)
    ha = a.history()
    hg = g.history()
    assert np.array_equal(ha[-10:], hg[-10:])
    a.close()
    g.close()


def test_batched_graph_replay(dp):
    sizes, seeds = W.replica_sizes(16, 500, 8000, seed=78)
    cfgs, qs, ps, es = [], [], [], []
    for r, (nr, sd) in enumerate(zip(sizes, seeds)):
        L = W.cubic_side(int(nr))
        q, p, e = W.equilibrium_state(int(nr), [L] * 3, seed=2000 + r)
        cfgs.append(dp.Config(n=int(nr), box=[L] * 3, seed=int(sd), replica=r))
        qs.append(q); ps.append(p); es.append(e)
    Q, Pm, E = np.concatenate(qs), np.concatenate(ps), np.concatenate(es)
    a = dp.System(cfgs, Q, Pm, E)
    g = dp.System(cfgs, Q, Pm, E)
    a.step(8)
    g.step_graph(2, 4)
    assert np.array_equal(a.energies(), g.energies())
    h = g.history()
    assert h.shape == (8, 16, 12)
    a.close()
    g.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_batched_learned_eos_replicas_match_single_systems(dp, eos_system, precision):
    """Replicas stepped with the learned EOS (the surrogate evaluated inside
    sweep 2) and FP64 or FP32 pair terms equal their single runs bit for
    bit, with one set of network weights."""
    eos_system.mlp_train(nsamples=200000, iters=300, batch=4096, lr=3e-3, seed=9)
    w, norm = eos_system.mlp_get()
    sizes, seeds = W.replica_sizes(4, 500, 3000, seed=80)
    cfgs, qs, ps, es = [], [], [], []
    for r, (nr, sd) in enumerate(zip(sizes, seeds)):
        L = W.cubic_side(int(nr))
        q, p, e = W.equilibrium_state(int(nr), [L] * 3, seed=4000 + r, eps0=25.0)
        cfgs.append(dp.Config(n=int(nr), box=[L] * 3, seed=int(sd), replica=r, dt=0.005,
                              eos=dp.EOS_EINSTEIN, theta_mode=dp.THETA_MLP,
                              precision=precision))
        qs.append(q); ps.append(p); es.append(e)
    b = dp.System(cfgs, np.concatenate(qs), np.concatenate(ps), np.concatenate(es))
    b.mlp_set(w, norm)
    b.step(6)
    qb, pb, eb, _ = _gpu_state(b)
    enb = b.energies()
    for r in range(len(cfgs)):
        s = dp.System(cfgs[r], qs[r], ps[r], es[r])
        s.mlp_set(w, norm)
        s.step(6)
        q1, p1, e1, _ = _gpu_state(s)
        lo, hi = b.offsets[r], b.offsets[r + 1]
        assert np.array_equal(qb[lo:hi], q1)
        assert np.array_equal(pb[lo:hi], p1)
        assert np.array_equal(eb[lo:hi], e1)
        assert np.array_equal(enb[r], s.energies())
        s.close()
    b.close()


@pytest.mark.parametrize("precision", [0, 1])
def test_step_end_in_sweep_two_with_the_surrogate(dp, eos_system, precision):
    """With the learned EOS the network runs inside sweep 2, before the
    step's end that a call of several steps also does there: eight one-step
    calls (separate kick and observables passes) and one eight-step call
    give the same states and records bit for bit, in FP64 and FP32."""
    eos_system.mlp_train(nsamples=200000, iters=300, batch=4096, lr=3e-3, seed=9)
    w, norm = eos_system.mlp_get()
    n = 3001
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=4100, eps0=25.0)
    cfg = dp.Config(n=n, box=[L] * 3, dt=0.005, eos=dp.EOS_EINSTEIN, theta_mode=dp.THETA_MLP,
                    precision=precision, seed=17)
    a = dp.System(cfg, q, p, e)
    b = dp.System(cfg, q, p, e)
    for s_ in (a, b):
        s_.mlp_set(w, norm)
        s_.history()
    a.step(8)
    for _ in range(8):
        b.step(1)
    sa, sb = _gpu_state(a), _gpu_state(b)
    for x, y in zip(sa[:3], sb[:3]):
        assert np.array_equal(x, y)
    assert np.array_equal(a.history(), b.history())
    a.close()
    b.close()


def test_graph_follows_new_surrogate_weights(dp, eos_system):
    """A captured step graph holds the surrogate's mode and normalisation as
    kernel arguments: a graph captured before the network had weights (the
    inversion by Newton) is dropped when weights are set, and the replays
    that follow (captured again) step like eager steps with the network,
    bit for bit."""
    eos_system.mlp_train(nsamples=200000, iters=300, batch=4096, lr=3e-3, seed=10)
    w, norm = eos_system.mlp_get()
    n = 3001
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=4200, eps0=25.0)
    cfg = dp.Config(n=n, box=[L] * 3, dt=0.005, eos=dp.EOS_EINSTEIN, theta_mode=dp.THETA_MLP,
                    seed=23)
    g = dp.System(cfg, q, p, e)
    g.step_graph(2, 1)  # captured without weights
    g.mlp_set(w, norm)
    g.step_graph(2, 2)
    a = dp.System(cfg, q, p, e)
    a.step(2)
    a.mlp_set(w, norm)
    a.step(2)
    a.step(2)
    sg, sa = _gpu_state(g), _gpu_state(a)
    for x, y in zip(sg[:3], sa[:3]):
        assert np.array_equal(x, y)
    assert sg[3] == sa[3] == 6
    g.close()
    a.close()


# ---------------------------------------------------------------------------
# SEM (Sec. 3.1.1): one step against the oracle's SEM.
# ---------------------------------------------------------------------------
def test_sem_step_parity(dp):
    n = 3000
    L = W.cubic_side(n)
    (eq, ep, ee), en, eo = _one_step_vs_oracle(dp, n, [L] * 3, scheme=dp.SCHEME_SEM, dt=0.005)
    assert max(eq, ep, ee) < 1e-12, (eq, ep, ee)


# ---------------------------------------------------------------------------
# Failure paths: codes, state kept at the failing step.
# ---------------------------------------------------------------------------
def test_negative_internal_energy_reported(dp):
    """Tiny heat capacity and a large noise: the reinjection drives some eps
    below zero (Sec. 4.4.2); the step returns DPDE_ENEG_EINT."""
    n = 2000
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=71, eps0=0.05)
    s = dp.System(dp.Config(n=n, box=[L] * 3, cv=0.05, gamma=40.0, dt=0.02), q, p, e)
    rc = s.step_raw(50)
    assert rc == dp._lib.DPDE_ENEG_EINT
    q1, p1, e1, st = s.get_state()
    assert st < 50
    # the state is readable and finite
    assert np.isfinite(q1.cpu().numpy()).all()
    s.close()


def test_handle_steps_on_after_a_failed_step(dp):
    """A call that fails mid-way (an internal energy driven below zero, the
    next kick possibly already done at the end of sweep 2) leaves nothing
    behind: after set_state the handle steps in one call exactly like a fresh
    handle from the same state, up to the step before the failure."""
    # a heat capacity of 20 with strong friction: the CPU oracle completes
    # four steps from this state before an internal energy turns negative
    n = 2000
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=71, eps0=20.0)
    cfg = dp.Config(n=n, box=[L] * 3, cv=20.0, gamma=20.0, dt=0.02)
    s = dp.System(cfg, q, p, e)
    assert s.step_raw(30) == dp._lib.DPDE_ENEG_EINT
    failed_at = s.get_state()[3]
    print("steps completed before the failure:", failed_at)
    assert failed_at >= 3
    k = failed_at - 1
    s.set_state(q, p, e, 0)
    s.history()
    s.step(k)
    f = dp.System(cfg, q, p, e)
    f.history()
    f.step(k)
    a, b = _gpu_state(s), _gpu_state(f)
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y)
    assert a[3] == b[3] == k
    assert np.array_equal(s.history(), f.history())
    s.close()
    f.close()


def test_invalid_inputs_rejected(dp):
    n = 300
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=72)
    bad = q.copy()
    bad[5, 1] = np.nan
    with pytest.raises(dp.DpdeError) as ex:
        dp.System(dp.Config(n=n, box=[L] * 3), bad, p, e)
    assert ex.value.code == dp._lib.DPDE_EINVAL
    e2 = e.copy()
    e2[3] = -1.0
    with pytest.raises(dp.DpdeError) as ex:
        dp.System(dp.Config(n=n, box=[L] * 3), q, p, e2)
    assert ex.value.code == dp._lib.DPDE_ENEG_EINT
    with pytest.raises(dp.DpdeError) as ex:
        dp.System(dp.Config(n=n, box=[2.9, L, L]), q, p, e)
    assert ex.value.code == dp._lib.DPDE_EBOX


def test_neighbour_overflow_reported(dp):
    n = 3000
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=73)
    with pytest.raises(dp.DpdeError) as ex:
        dp.System(dp.Config(n=n, box=[L] * 3, neighbor_cap=4), q, p, e)
    assert ex.value.code == dp._lib.DPDE_EOVERFLOW


# ---------------------------------------------------------------------------
# Full size: N = 1,048,576 in the launch configuration the benchmark times.
# The oracle replays one step from the GPU state (a few seconds on one core).
# ---------------------------------------------------------------------------
def test_full_size_one_step_parity(dp):
    n = 1_048_576
    L = W.cubic_side(n)
    (eq, ep, ee), en, eo = _one_step_vs_oracle(dp, n, [L] * 3, prime=2, dt=0.005)
    assert max(eq, ep, ee) < 1e-12, (eq, ep, ee)
    assert abs(en[3] - eo[3]) < 1e-12 * abs(eo[3])
    assert abs(en[8] - eo[8]) < 1e-12 * abs(eo[8])


# ---------------------------------------------------------------------------
# Autotuner: candidates are timed on the live system and the state restored;
# block sizes do not enter the arithmetic, so the trajectory is unchanged.
# ---------------------------------------------------------------------------
def test_autotune_leaves_trajectory_unchanged(dp):
    n = 6000
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=91)
    a = dp.System(dp.Config(n=n, box=[L] * 3), q, p, e)
    b = dp.System(dp.Config(n=n, box=[L] * 3), q, p, e)
    a.step(5)
    b.step(5)
    ha = a.history()
    hb = b.history()
    builds = b.list_builds()
    pb, ab, ms = b.autotune(3)
    assert pb in (64, 128, 256) and ab in (128, 256, 512) and ms > 0
    assert b.list_builds() == builds
    assert b.history().shape[0] == 0  # trial records were rolled back
    # the tuned handle continues as an untuned one given the same shape (the
    # block sizes and the cell order change no bit; the pair forms agree to
    # rounding, so the reference takes the winner's form)
    a.set_shape(**b.get_shape())
    a.step(25)
    b.step(25)
    sa, sb = a.get_state(), b.get_state()
    for x, y in zip(sa[:3], sb[:3]):
        assert torch_equal(x, y)
    assert sa[3] == sb[3] == 30
    assert np.array_equal(a.history(), b.history())
    a.close()
    b.close()
    dp.tuning_clear()  # later handles of this size class start from the defaults


def test_autotune_records_the_shape_of_the_size_class(dp, tmp_path):
    """The winner goes into the library's tuning table under (size class,
    replica class, precision); a new handle of that class starts with it, and
    the table survives a save / clear / load round trip."""
    n = 5000
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=92)
    dp.tuning_clear()
    try:
        s = dp.System(dp.Config(n=n, box=[L] * 3, precision=dp.FP32), q, p, e)
        s.autotune(2)
        sh = s.get_shape()
        s.close()
        got = dp.tuning_lookup(n, 1, dp.FP32)
        assert got is not None and got[0] == sh and got[1] > 0
        assert dp.tuning_lookup(n, 1, dp.FP64) is None
        assert dp.tuning_lookup(2 * 4096, 1, dp.FP32) is None  # the next size class
        s2 = dp.System(dp.Config(n=n + 100, box=[W.cubic_side(n + 100)] * 3,
                                 precision=dp.FP32), *W.equilibrium_state(
                                     n + 100, [W.cubic_side(n + 100)] * 3, seed=93))
        assert s2.get_shape() == sh
        s2.close()
        path = str(tmp_path / "tuning.txt")
        dp.tuning_save(path)
        dp.tuning_clear()
        assert dp.tuning_lookup(n, 1, dp.FP32) is None
        dp.tuning_load(path)
        assert dp.tuning_lookup(n, 1, dp.FP32)[0] == sh
    finally:
        dp.tuning_clear()


def test_autotune_table_keys_batches_by_replica_count(dp):
    """A batch is its own replica class: its tuned shape is recorded under
    (size class, 1 + floor(log2 nrep), precision) and does not leak to a
    single system of the same total size, and the next batch of that class
    starts with it."""
    def batch(nrep, seed):
        sizes, seeds = W.replica_sizes(nrep, 500, 1500, seed=seed)
        cfgs, qs, ps, es = [], [], [], []
        for r, (nr, sd) in enumerate(zip(sizes, seeds)):
            L = W.cubic_side(int(nr))
            q, p, e = W.equilibrium_state(int(nr), [L] * 3, seed=4000 + r)
            cfgs.append(dp.Config(n=int(nr), box=[L] * 3, seed=int(sd), replica=r))
            qs.append(q); ps.append(p); es.append(e)
        return dp.System(cfgs, np.concatenate(qs), np.concatenate(ps), np.concatenate(es))
    dp.tuning_clear()
    try:
        b = batch(8, 31)
        b.autotune(2)
        sh, n = b.get_shape(), b.n
        b.close()
        got = dp.tuning_lookup(n, 8, dp.FP64)
        assert got is not None and got[0] == sh
        assert dp.tuning_lookup(n, 1, dp.FP64) is None
        b2 = batch(8, 31)
        assert b2.get_shape() == sh
        b2.close()
    finally:
        dp.tuning_clear()


def torch_equal(x, y):
    return bool((x == y).all().item())
