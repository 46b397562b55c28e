"""Limits and rare paths of the GPU library: list capacities, failing calls,
crowded and sparse boxes, every tile shape."""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.fixture(scope="module")
def dp():
    import torch
    assert torch.cuda.is_available()
    import paper_1507_06643_amd as m
    return m


def _state(s):
    q, p, e, step = s.get_state()
    return q.cpu().numpy(), p.cpu().numpy(), e.cpu().numpy(), step


def _same(a, b):
    return all(np.array_equal(x, y) for x, y in zip(a, b))


def _longest_tile_list(s, q, box, reach, tile):
    """The longest list when pairs inside a tile of `tile` particles of the
    memory order are listed once (by the lower index if the two differ in
    parity, else by the higher one) and all others on both sides."""
    from scipy.spatial import cKDTree
    slot = np.empty(s.n, dtype=np.int64)
    slot[s.debug_order().cpu().numpy()] = np.arange(s.n)
    pr = cKDTree(q, boxsize=box).query_pairs(reach, output_type="ndarray")
    i, j = np.sort(slot[pr], axis=1).T
    once = (i ^ j) < tile
    lower = ((i ^ j) & 1) == 1
    count = np.bincount(i[~once | lower], minlength=s.n)
    return (count + np.bincount(j[~once | ~lower], minlength=s.n)).max()


@pytest.mark.parametrize("n", [1000, 20000])
def test_list_capacity_is_that_of_tiles_of_128(dp, n):
    """Small systems run tiles of 32 or 64 particles, whose lists are longer
    than those of tiles of 128: a capacity that holds the latter is accepted
    and changes no bit, one entry less is refused."""
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=n)
    kw = dict(n=n, box=[L] * 3, dt=0.01)
    ref = dp.System(dp.Config(**kw), q, p, e)
    cap = int(_longest_tile_list(ref, q, [L] * 3, 1.3, 128))
    assert _longest_tile_list(ref, q, [L] * 3, 1.3, 32 if n <= 16384 else 64) > cap
    s = dp.System(dp.Config(neighbor_cap=cap, **kw), q, p, e)
    assert np.array_equal(s.debug_pairs(), ref.debug_pairs())
    for x in (ref, s):
        x.step(2)
    assert _same(_state(ref), _state(s))
    with pytest.raises(dp.DpdeError) as ex:
        dp.System(dp.Config(neighbor_cap=cap - 1, **kw), q, p, e)
    assert ex.value.code == dp._lib.DPDE_EOVERFLOW
    s.close()
    ref.close()


@pytest.mark.parametrize("n", [400, 26000])
def test_capacity_below_the_staged_rows(dp, n):
    """Lists of fewer entries than pass A stages in LDS (28 and more): a
    dilute system with room for six neighbours steps like one with room for
    ninety-six, and like the oracle."""
    box = [(n / 0.2) ** (1 / 3)] * 3
    q, p, e = W.equilibrium_state(n, box, seed=n)
    runs = []
    for cap in (96, 16):
        s = dp.System(dp.Config(n=n, box=box, dt=0.01, neighbor_cap=cap), q, p, e)
        s.step(1)
        runs.append(_state(s))
        s.close()
    assert _same(*runs)
    S = O.State(O.make_params(n, box, dt=0.01), q, p, e)
    assert S.step(1)[0] == 0
    assert np.abs(runs[1][1] - S.p).max() < TOL
    assert np.abs(runs[1][2] - S.eps).max() < TOL * np.abs(S.eps).mean()


def _failing(dp, form):
    """A system whose strong friction drives an internal energy below zero
    after one to four steps (as the CPU oracle finds for these heat capacities)."""
    n = 2000
    L = W.cubic_side(n)
    cv = {"sem": 4.6, "sem_projected": 7.0, "hybrid": 8.0}.get(form, 20.0)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=71, eps0=cv)
    kw = dict(n=n, box=[L] * 3, cv=cv, gamma=20.0, dt=0.02)
    kw.update({"tile": {}, "both_sides": {}, "sem": dict(scheme=dp.SCHEME_SEM),
               "sem_projected": dict(scheme=dp.SCHEME_SEM, project=True),
               "hybrid": dict(scheme=dp.SCHEME_HYBRID, ndom=(2, 2, 2)),
               "projected": dict(project=True)}[form])
    s = dp.System(dp.Config(**kw), q, p, e)
    if form == "both_sides":
        s.set_shape(pairs=dp.PAIRS_BOTH_SIDES)
    return s, kw


@pytest.mark.parametrize("form", ["tile", "both_sides", "sem", "sem_projected", "hybrid",
                                  "projected"])
@pytest.mark.parametrize("how", ["even", "odd", "graph"])
def test_failed_call_leaves_the_failing_step(dp, form, how):
    """After a call that fails in step k, positions are those of step k (the
    kick and drift from the state after k steps) whether an even or odd number
    of steps were still to come, and the record and the counter belong to that
    state."""
    s, kw = _failing(dp, form)
    for k in range(20):  # single steps up to the failure
        before, F = _state(s), s.forces()[0].cpu().numpy()
        if s.step_raw(1):
            break
    assert 1 <= k < 19
    s.close()
    s, _ = _failing(dp, form)
    if how == "graph":
        with pytest.raises(dp.DpdeError) as ex:
            s.step_graph(k + 2 + k % 2, 2)
        assert ex.value.code == dp._lib.DPDE_ENEG_EINT
    else:
        assert s.step_raw(k + (3 if how == "even" else 2)) == dp._lib.DPDE_ENEG_EINT
    q, p, e, step = _state(s)
    assert step == k and len(s.history()) == k
    L = kw["box"][0]
    want = before[0] + kw["dt"] * (before[1] + 0.5 * kw["dt"] * F)
    d = q - want
    assert np.abs(d - L * np.rint(d / L)).max() < TOL * L
    rec = s.energies()
    assert rec[1] == pytest.approx(0.5 * (p ** 2).sum(), rel=1e-12)
    assert rec[2] == pytest.approx(e.sum(), rel=1e-12)
    s.close()


@pytest.mark.parametrize("form", ["tile", "both_sides", "sem", "hybrid"])
def test_a_kick_that_overflows_fails_its_own_step(dp, form):
    """A particle flying off at 1e308 per step leaves the range of FP64 in the
    kick of the second step: one call of five steps completes the first one,
    records it and fails in the second, as single steps do."""
    n, box = 40, [20.0] * 3
    q, p, e = W.equilibrium_state(n, box, seed=5)
    p[7, 0] = 1e308
    kw = dict(n=n, box=box, periodic=[0, 0, 0], a=0.0, gamma=0.0, dt=1.0)
    kw.update({"sem": dict(scheme=dp.SCHEME_SEM),
               "hybrid": dict(scheme=dp.SCHEME_HYBRID, ndom=(2, 2, 2))}.get(form, {}))
    runs = []
    for calls in ([1, 1], [5]):
        s = dp.System(dp.Config(**kw), q, p, e)
        if form == "both_sides":
            s.set_shape(pairs=dp.PAIRS_BOTH_SIDES)
        for c in calls[:-1]:
            s.step(c)
        assert s.step_raw(calls[-1]) == dp._lib.DPDE_ENONFINITE
        runs.append((_state(s)[3], s.history()))
        s.close()
    assert runs[0][0] == runs[1][0] == 1
    assert runs[0][1].shape == runs[1][1].shape == (1, 12)
    assert np.array_equal(runs[0][1], runs[1][1], equal_nan=True)


def _kernel_us(s, steps):
    """Mean time of every kernel over some single steps."""
    s.step(2)
    s.profile(True)
    s.profile_read()
    for _ in range(steps):
        s.step(1)
    out = {k: 1e3 * ms / count for k, (ms, count) in s.profile_read().items()}
    s.profile(False)
    return out


def test_list_build_of_a_sparse_box_depends_on_its_particles(dp):
    """7 million cells, a build on every step: a hundred particles are listed
    no slower than twenty thousand (both take a few microseconds; clearing the
    cells by the few blocks of the hundred took 560), and the pairs stay those
    of the oracle."""
    us = {}
    box = [200.0] * 3
    for n in (100, 20000):
        q, p, e = W.equilibrium_state(n, box, seed=n)
        if n == 100:
            q = np.mod(q * 0.02 + 199.0, 200.0)  # close together, across the corner
        s = dp.System(dp.Config(n=n, box=box, dt=0.01, skin=0.05), q, p, e)
        us[n] = _kernel_us(s, 5)["build_skin"]
        s.step(5)
        assert s.list_builds() > 5
        s.set_state(*s.get_state())
        qs = _state(s)[0]
        assert np.array_equal(s.debug_pairs(), O.pairs(O.make_params(n, box), qs, "cells"))
        s.close()
    assert us[100] < 2.0 * us[20000], us


@pytest.mark.parametrize("n", [1500, 9000, 40000])
def test_an_overflow_leaves_the_binning_clear(dp, n):
    """A state whose lists overflow is refused; the next one is binned as on a
    fresh handle (n in one block, with the scan in the last block, and with a
    scan of its own)."""
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=n)
    s = dp.System(dp.Config(n=n, box=[L] * 3, dt=0.01), q, p, e)
    for crowd in (q * 0.3, q * 0.15 + 0.7 * L):
        with pytest.raises(dp.DpdeError) as ex:
            s.set_state(crowd, p, e, 0)
        assert ex.value.code == dp._lib.DPDE_EOVERFLOW
    s.set_state(q, p, e, 0)
    ref = dp.System(dp.Config(n=n, box=[L] * 3, dt=0.01), q, p, e)
    for x in (s, ref):
        x.step(6)
    assert _same(_state(s), _state(ref))
    assert np.array_equal(s.debug_order().cpu().numpy(), ref.debug_order().cpu().numpy())
    s.close()
    ref.close()


@pytest.mark.parametrize("pairs", [0, 1])
@pytest.mark.parametrize("n,density", [(61, 0.5), (700, 0.6), (700, 0.8), (16384, 0.65),
                                       (16385, 0.75), (40000, 1.5), (40000, 1.7), (80001, 0.3)])
def test_pairs_on_both_sides_of_the_few_per_cell_rule(dp, n, density, pairs):
    """Where cells hold few particles the lists are built by four lanes per
    particle, elsewhere by a wave per piece of a cell: pairs of the oracle at
    densities around the rule (1.5 and 3.5 per cell), in blocked order, with a
    free boundary and a crowd, for tiles of 32, 64 and 128 and both-sides lists."""
    side = max((n / density) ** (1 / 3), 3.95)
    box, per = [1.3 * side, side, side / 1.3 if n > 100 else side], [0, 1, 1]
    q, p, e = W.equilibrium_state(n, box, seed=n)
    rng = np.random.default_rng(n)
    q[::7, 0] += 0.4 * box[0]           # some beyond the open face
    q[:40] = np.array([1.0, 0.1, 0.1]) + 0.9 * rng.random((40, 3))
    s = dp.System(dp.Config(n=n, box=box, periodic=per, dt=0.005, neighbor_cap=192), q, p, e)
    P = O.make_params(n, box, periodic=per)
    s.set_shape(pairs=pairs, order_block=1 + n % 2)
    assert np.array_equal(s.debug_pairs(), O.pairs(P, q, "cells"))
    s.step(8)
    s.set_state(*s.get_state())
    assert np.array_equal(s.debug_pairs(), O.pairs(P, _state(s)[0], "cells"))
    s.close()


def test_batched_lists_of_few_per_cell(dp):
    """Replicas of one particle per cell and fewer (tiles across replicas)."""
    cfgs, qs, ps, es = [], [], [], []
    for r, n in enumerate([300, 41, 129, 500, 10]):
        box = [max((n / 0.4) ** (1 / 3), 3.95)] * 3
        q, p, e = W.equilibrium_state(n, box, seed=50 + r)
        cfgs.append(dp.Config(n=n, box=box, dt=0.01, seed=r, replica=r))
        qs.append(q); ps.append(p); es.append(e)
    for pairs in (0, 1):
        b = dp.System(cfgs, np.vstack(qs), np.vstack(ps), np.concatenate(es))
        b.set_shape(pairs=pairs)
        b.step(12)
        got = _state(b)
        for r, c in enumerate(cfgs):
            s = dp.System(c, qs[r], ps[r], es[r])
            s.set_shape(pairs=pairs)
            s.step(12)
            rows = slice(b.offsets[r], b.offsets[r + 1])
            assert _same(_state(s)[:3], [x[rows] for x in got[:3]]), (r, pairs)
            s.close()
        b.close()


def test_list_build_is_no_dearer_where_cells_hold_few(dp):
    """N = 262,144 at density 0.3 (0.7 particles to a cell) against density 3:
    46 against 82 us per build (117 by the pieces of cells)."""
    n, us = 262144, {}
    for density in (0.3, 3.0):
        box = [(n / density) ** (1 / 3)] * 3
        q, p, e = W.equilibrium_state(n, box, seed=1)
        s = dp.System(dp.Config(n=n, box=box, dt=0.005), q, p, e)
        s.profile(True)
        for _ in range(6):
            s.set_state(q, p, e, 0)
        ms, count = s.profile_read()["build_skin"]
        us[density] = 1e3 * ms / count
        s.close()
    assert us[0.3] < us[3.0], us


def test_list_build_of_a_crowded_cell(dp):
    """Particles that left through an open face stay in the border cells, all
    of a long column here in one.  Four times as many take sixteen times the
    tests; with two lanes listing a crowded cell's candidates and a quarter of
    the waves at work a build took 7.4 times as long (326 to 2420 us), without
    3.8 times.  The pairs stay the oracle's."""
    n, us = 40000, {}
    box = [W.cubic_side(n)] * 3
    for out in (3000, 12000):
        q, p, e = W.equilibrium_state(n, box, seed=5)
        rng = np.random.default_rng(6)
        k = rng.permutation(n)[:out]
        q[k, 0] = box[0] + 5.0 + 1e4 * rng.random(out)
        q[k, 1:] = rng.random((out, 2))
        p[k] = 0.0
        s = dp.System(dp.Config(n=n, box=box, periodic=[0, 1, 1], dt=0.005), q, p, e)
        s.profile(True)
        for _ in range(6):
            s.set_state(q, p, e, 0)
        ms, count = s.profile_read()["build_skin"]
        us[out] = 1e3 * ms / count
        if out == 3000:
            P = O.make_params(n, box, periodic=[0, 1, 1])
            assert np.array_equal(s.debug_pairs(), O.pairs(P, q, "cells"))
        s.close()
    assert us[12000] < 5.5 * us[3000], us


def _binning_us(s, state, builds=6):
    """Mean times of the binning's kernels over forced builds of a state."""
    s.profile(True)
    s.profile_read()
    for _ in range(builds):
        s.set_state(*state, 0)
    out = {k: 1e3 * ms / count for k, (ms, count) in s.profile_read().items()}
    s.profile(False)
    return out


def test_scan_of_many_cells(dp):
    """300,000 cells against 10,000 (N = 65,536 at density 0.1 and 3): 16
    against 12 us (33 where every block added up all counts before its own)."""
    n, us = 65536, {}
    for density in (0.1, 3.0):
        box = [(n / density) ** (1 / 3)] * 3
        q, p, e = W.equilibrium_state(n, box, seed=1)
        s = dp.System(dp.Config(n=n, box=box), q, p, e)
        t = _binning_us(s, (q, p, e))
        us[density] = sum(v for k, v in t.items() if k.startswith("scan"))
        s.close()
    assert us[0.1] < 2.0 * us[3.0], us


def test_ranking_of_a_large_set_state(dp):
    """A set state lies in identifier order.  N = 600,000 of which 30,000 share a
    border cell: ranked within twice the time that steps take from the sorted
    state; the order is that of identifiers inside each cell, the pairs and the
    next steps those of the state's own resumption."""
    n, out = 600000, 30000
    box = [W.cubic_side(n)] * 3
    q, p, e = W.equilibrium_state(n, box, seed=5)
    rng = np.random.default_rng(6)
    k = rng.permutation(n)[:out]
    q[k, 0] = box[0] + 5.0 + 1e4 * rng.random(out)
    q[k, 1:] = rng.random((out, 2))
    p[k] = 0.0
    s = dp.System(dp.Config(n=n, box=box, periodic=[0, 1, 1], dt=0.005, skin=0.02), q, p, e)
    forced = _binning_us(s, (q, p, e))["rank_gather"]
    rows, cells = s.debug_order().cpu().numpy(), s.debug_cells().cpu().numpy()
    assert np.array_equal(np.lexsort((np.arange(n), cells)), rows)
    s.step(1)
    steps = _kernel_us(s, 4)["rank_gather"]
    assert forced < 2.0 * steps, (forced, steps)
    a = _state(s)
    s.step(2)
    b = _state(s)
    s.set_state(*a)
    s.step(2)
    assert _same(_state(s), b)
    s.close()


def test_records_of_many_replicas(dp):
    """3000 replicas of ten particles: the final pass over their sums, a block
    per replica, takes as long as the pass that makes them (79 and 74 us; 89
    where every block read the next step's maxima and ended on a barrier)."""
    rng = np.random.default_rng(1)
    cfgs = [dp.Config(n=10, box=[3.95] * 3, dt=0.01, seed=r, replica=r) for r in range(3000)]
    s = dp.System(cfgs, rng.random((30000, 3)) * 3.95, rng.normal(size=(30000, 3)),
                  np.full(30000, 100.0))
    us = _kernel_us(s, 30)
    assert us["stats_final"] < 1.14 * us["stats_tiles"], us
    h = s.history()
    assert h.shape[1:] == (3000, 12) and np.array_equal(h[:, :, 9], np.arange(1, 33)[:, None] * np.ones(3000))
    s.close()


@pytest.mark.parametrize("n,density", [(1000, 0.5), (4000, 0.6), (30000, 0.6), (40000, 1.4)])
def test_list_capacity_where_cells_hold_few(dp, n, density):
    """As test_list_capacity_is_that_of_tiles_of_128, for the lists built by
    four lanes per particle."""
    box = [(n / density) ** (1 / 3)] * 3
    q, p, e = W.equilibrium_state(n, box, seed=n)
    kw = dict(n=n, box=box, dt=0.01)
    ref = dp.System(dp.Config(**kw), q, p, e)
    cap = int(_longest_tile_list(ref, q, box, 1.3, 128))
    assert _longest_tile_list(ref, q, box, 1.3, 32 if n <= 16384 else 64) > cap
    s = dp.System(dp.Config(neighbor_cap=cap, **kw), q, p, e)
    assert np.array_equal(s.debug_pairs(), ref.debug_pairs())
    s.step(1)
    ref.step(1)
    assert _same(_state(ref), _state(s))
    with pytest.raises(dp.DpdeError) as ex:
        dp.System(dp.Config(neighbor_cap=cap - 1, **kw), q, p, e)
    assert ex.value.code == dp._lib.DPDE_EOVERFLOW
    s.close()
    ref.close()


def test_memory_of_a_hybrid_handle(dp):
    """Hybrid needs a third list and the intra-domain pairs beside what SER
    holds; the pairs share the memory of the increments, so that it stays below
    the 20 bytes an entry that the pairs alone took."""
    import torch
    n, cap, used = 200000, 96, {}
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=3)
    q, p, e = (torch.as_tensor(x).cuda() for x in (q, p, e))
    for scheme in (dp.SCHEME_SER, dp.SCHEME_SER, dp.SCHEME_HYBRID):  # (the first loads the code)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        s = dp.System(dp.Config(n=n, box=[L] * 3, dt=0.005, scheme=scheme, ndom=(16, 16, 16)),
                      q, p, e)
        used[scheme] = free - torch.cuda.mem_get_info()[0]
        s.close()
    more = used[dp.SCHEME_HYBRID] - used[dp.SCHEME_SER]
    assert more <= 20 * n * cap, used


@pytest.mark.parametrize("density,shapes", [(3.0, 12 + 36), (0.3, 36 + 36)])
def test_autotune_times_each_shape_once(dp, density, shapes):
    """The tile form's passes have blocks of their own, so that only where the
    list build has blocks of pair_block threads (few particles to a cell) do
    its shapes differ by them.  Each shape takes a forced build, a warm-up and
    the timed steps; one more build restores the state."""
    n = 3000
    box = [(n / density) ** (1 / 3)] * 3
    s = dp.System(dp.Config(n=n, box=box), *W.equilibrium_state(n, box, seed=91))
    s.profile(True)
    s.profile_read()
    try:
        s.autotune(1)
    finally:
        dp.tuning_clear()
    assert s.profile_read()["pass_a_forces"][1] == 3 * shapes + 1
    s.close()


TILE_CASES = ["plain", "fp32", "projected_model", "projected_model_fp32", "regenerated",
              "regenerated_fp32", "regenerated_projected_model", "free_x", "projection", "newton",
              "surrogate", "surrogate_regenerated", "blocked", "dense"]


def _tile_case(dp, case):
    n, kw, box, per = 1517, dict(dt=0.01), None, [1, 1, 1]
    if "fp32" in case:
        kw["precision"] = dp.FP32
    if "projected_model" in case:
        kw["model"] = dp.MODEL_PROJECTED
    if case == "projection":
        kw["project"] = True
    if case in ("newton", "surrogate", "surrogate_regenerated"):
        kw["eos"] = dp.EOS_EINSTEIN
    if "surrogate" in case:
        kw["theta_mode"] = dp.THETA_MLP
    box = [W.cubic_side(n)] * 3
    if case == "free_x":
        box, per = [1.7 * box[0], box[0] / 1.25, box[0] / 1.35], [0, 1, 1]
    if case == "dense":
        kw.update(dt=0.002, neighbor_cap=512)
    q, p, e = W.equilibrium_state(n, box, seed=77)
    if case == "dense":  # lists beyond the rows of pass A and of its work lists
        q[:500] = np.random.default_rng(4).random((500, 3)) * 1.5 + 2.0
    ckw = dict(n=n, box=box, periodic=per, **kw)

    class Config(dp.Config):
        def to_c(self):
            P = super().to_c()
            if "regenerated" in case:
                P.flags |= dp._lib.DPDE_FLAG_REGENERATE_NOISE
            return P

    return Config, ckw, (q, p, e)


@pytest.mark.parametrize("case", TILE_CASES)
def test_every_tile_gives_the_same_bits(dp, case):
    """Tiles of 32, 64 and 128 (the ones that large systems run) on one small
    system, ragged in all of them: the same states, records and pairs bit for
    bit, over steps with list builds; and one step of the oracle."""
    Config, ckw, state = _tile_case(dp, case)
    runs = []
    for tile in (32, 64, 128):
        s = dp.System(Config(**ckw), *state)
        if "surrogate" in case:
            net = np.random.default_rng(3).normal(0, 0.3, 1153).astype(np.float32)
            s.mlp_set(net, np.array([5.0, 3.0, 0.0, 2.3]))
        if case == "blocked":
            s.set_shape(order_block=3)
        s.debug_tile(tile)
        s.step(12)
        runs.append((_state(s), s.history(), s.debug_pairs(), s.list_builds()))
        if tile == 128 and case not in ("surrogate", "surrogate_regenerated"):
            q, p, e, st = runs[-1][0]
            ok = {k: v for k, v in ckw.items()
                  if k not in ("n", "box", "precision", "neighbor_cap", "theta_mode", "project")}
            P = O.make_params(ckw["n"], ckw["box"], step=st, **ok)
            if case == "projection":
                P.project = 1
            S = O.State(P, q, p, e)
            if case == "projection":
                P.E0 = runs[-1][1][0, 3]
            assert S.step(1)[0] == 0
            s.step(1)
            q, p, e, _ = _state(s)
            tol = 5e-6 if "fp32" in case else TOL
            assert np.abs(p - S.p).max() < tol
            assert np.abs(e - S.eps).max() < tol * np.abs(S.eps).mean()
        s.close()
    for other in runs[1:]:
        assert _same(runs[0][0], other[0])
        for a, b in zip(runs[0][1:], other[1:]):
            assert np.array_equal(a, b)
    assert runs[0][3] > 2 or case == "dense"


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("tile", [64, 128])
def test_small_replicas_in_every_tile(dp, tile, prec):
    """Replicas below the particles of a wave of pass A in the larger tiles."""
    cfgs, qs, ps, es = [], [], [], []
    for r, n in enumerate([7, 300, 5, 13, 12, 200, 3, 2, 64]):
        box = [max(W.cubic_side(n), 3.95)] * 3
        q, p, e = W.equilibrium_state(n, box, seed=50 + r)
        cfgs.append(dp.Config(n=n, box=box, dt=0.01, seed=r, replica=r, precision=prec))
        qs.append(q); ps.append(p); es.append(e)
    runs = []
    for t in (32, tile):
        b = dp.System(cfgs, np.vstack(qs), np.vstack(ps), np.concatenate(es))
        b.debug_tile(t)
        b.step(12)
        runs.append((_state(b), b.history()))
        b.close()
    assert _same(runs[0][0], runs[1][0])
    assert np.array_equal(runs[0][1], runs[1][1])


@pytest.mark.parametrize("n", [16384, 16385, 73728, 73729])
def test_at_the_sizes_where_the_tile_changes(dp, n):
    """The largest systems of the smaller tiles and the smallest of the larger
    ones: the bits of tiles of 128, one step of the oracle."""
    L = W.cubic_side(n)
    q, p, e = W.equilibrium_state(n, [L] * 3, seed=n)
    runs = []
    for tile in (None, 128):
        s = dp.System(dp.Config(n=n, box=[L] * 3, dt=0.01), q, p, e)
        if tile:
            s.debug_tile(tile)
        s.step(6)
        runs.append((_state(s), s.history()))
        if not tile:
            S = O.State(O.make_params(n, [L] * 3, dt=0.01, step=6), *runs[0][0][:3])
            assert S.step(1)[0] == 0
            s.step(1)
            got = _state(s)
            assert np.abs(got[1] - S.p).max() < TOL
            assert np.abs(got[2] - S.eps).max() < TOL * np.abs(S.eps).mean()
        s.close()
    assert _same(runs[0][0], runs[1][0])
    assert np.array_equal(runs[0][1], runs[1][1])


def test_tile_hook_refuses_other_tiles(dp):
    n = 17000
    L = W.cubic_side(n)
    s = dp.System(dp.Config(n=n, box=[L] * 3), *W.equilibrium_state(n, [L] * 3, seed=1))
    for tile in (0, 16, 32, 96, 256):
        with pytest.raises(dp.DpdeError) as ex:
            s.debug_tile(tile)
        assert ex.value.code == dp._lib.DPDE_EINVAL
    s.close()


@pytest.mark.parametrize("n,density,tile", [(60000, 3.0, 64), (60000, 6.0, 64),
                                            (60000, 10.0, 128), (24000, 20.0, 128),
                                            (16384, 20.0, 32), (73729, 0.5, 128)])
def test_tile_of_dense_systems(dp, n, density, tile):
    """Dense systems fill the chip at fewer particles: they take tiles of 128
    where tiles of 64 are slower (the hook accepts a system's own tile and
    larger ones)."""
    box = [(n / density) ** (1 / 3)] * 3
    s = dp.System(dp.Config(n=n, box=box, neighbor_cap=512), *W.equilibrium_state(n, box, seed=1))
    for t in (32, 64, 128):
        if t >= tile:
            s.debug_tile(t)
        else:
            with pytest.raises(dp.DpdeError):
                s.debug_tile(t)
    s.close()


def test_ranking_of_a_crowded_cell_by_one_block(dp):
    """A thousand particles in one border cell, set in identifier order: up to
    2048 particles one block bins and ranks them, in about the time that the
    separate launches take at N = 8000 (159 and 140 us; 218 along the chain)."""
    us = {}
    for n in (1800, 8000):
        box = [W.cubic_side(n)] * 3
        q, p, e = W.equilibrium_state(n, box, seed=5)
        rng = np.random.default_rng(6)
        k = rng.permutation(n)[:1000]
        q[k, 0] = box[0] + 5.0 + 1e4 * rng.random(1000)
        q[k, 1:] = rng.random((1000, 2))
        p[k] = 0.0
        s = dp.System(dp.Config(n=n, box=box, periodic=[0, 1, 1], dt=0.005), q, p, e)
        t = _binning_us(s, (q, p, e))
        us[n] = t["bin"] + t.get("rank_gather", 0.0)
        rows, cells = s.debug_order().cpu().numpy(), s.debug_cells().cpu().numpy()
        assert np.array_equal(np.lexsort((np.arange(n), cells)), rows)
        s.close()
    assert us[1800] < 1.35 * us[8000], us
