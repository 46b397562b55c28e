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
