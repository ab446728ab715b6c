"""A batch's bits do not depend on the route that its size gives it: workgroups of eight, four and one
waves per tower, shared packs of several sizes, two and three waves per SIMD.  And an island whose
bodies' arrays do not fit LDS, whose colour masks stay in device memory, against the oracle."""
import os

import numpy as np
import pytest

from paper_2606_28394_amd import workloads as W
from test_gpu_mega import _compare

pytestmark = pytest.mark.gpu
NET = os.path.join(os.path.dirname(W.__file__), "data", "warmstart_mlp.npy")


@pytest.fixture(scope="module")
def J():
    from paper_2606_28394_amd import jenga
    jenga.load_library()
    return jenga


def _after(J, sc, steps, **kw):
    if kw.get("warm_start") == 2:
        kw.update(mlp=np.load(NET), mlp_iters=4)
    w = J.World(sc, **kw)
    w.step(steps)
    w.step(1)
    st = w.stats()
    assert st.error_word == 0
    out = [np.asarray(x) for x in w.state()] + [np.asarray([st.candidates, st.manifolds, st.points, st.colours])]
    w.close()
    return out


@pytest.mark.parametrize("towers,levels,start,one,other", [
    (3, (30, 40), 0, {}, {"small_batch": -1}),                        # eight waves; more manifolds than its lane pairs own
    (260, (8, 9), 1, {}, {"small_batch": -1}),                        # four waves
    (2100, (8, 8), 0, {"pack_bodies": 24}, {"pack_bodies": 120}),     # three waves per SIMD, and two
    (2100, (8, 8), 1, {}, {"pack_bodies": 250}),                      # the library's packs; more than a wave's lanes in a colour
    (1100, (8, 10), 2, {}, {"pack_bodies": 30}),                      # the network's packs, one and several towers each
])
def test_routes_give_the_same_bits(J, towers, levels, start, one, other):
    sc = W.tilted_towers(5, towers, levels_range=levels, n_steps=8)
    for x, y in zip(_after(J, sc, 3, warm_start=start, **one), _after(J, sc, 3, warm_start=start, **other)):
        np.testing.assert_array_equal(x, y)


def test_island_beyond_lds_matches_oracle(J, oracle):
    sc = W.masonry_wall(46, 100, seed=3, n_steps=2)
    ow = oracle.OracleWorld(sc)
    _compare(J, oracle, sc, [(ow.x.copy(), ow.q.copy(), ow.v.copy(), ow.w.copy())], "wall 46x100")
