"""Which route a batch takes and the LDS that it is launched with: what fits a workgroup is stepped, to the
same bits on every route, whatever the manifold capacity and however many pushes a tower has."""
import os

import numpy as np
import pytest

from paper_2606_28394_amd import workloads as W

pytestmark = pytest.mark.gpu
NET = os.path.join(os.path.dirname(W.__file__), "data", "warmstart_mlp.npy")


@pytest.fixture(scope="module")
def J():
    from paper_2606_28394_amd import jenga
    jenga.load_library()
    return jenga


def _towers(levels, pushes=None, seed=90):
    """Upright towers; pushes[t] rows of no force on tower t's bodies in turn (they only take room)."""
    sb = W.SceneBuilder(W.default_params(), 4)
    for t, n in enumerate(levels):
        he, m, pos, quat, _, _ = W.jenga_tower(n, W.rng_for(seed, t))
        b0 = sum(3 * k for k in levels[:t])
        sb.add_tower(he, m, pos, quat, 0.4)
        for r in range((pushes or [0] * len(levels))[t]):
            sb.add_push(b0 + r % (3 * n), [0.0, 0.0, 0.0], 0, 4)
    return sb.build()


def _after(J, sc, steps=3, **kw):
    w = J.World(sc, **kw)
    w.step(steps)
    st = w.stats()
    assert st.error_word == 0
    out = [np.asarray(x) for x in w.state()] + [np.asarray([st.candidates, st.manifolds, st.points, st.colours])]
    w.close()
    return out


# (previous-step starts: the widest layout of a small batch)
@pytest.mark.parametrize("levels,pushes,kw", [
    ([70], None, {"manifolds_per_body": 8.0}),        # fits LDS without the small batch's shared words only
    ([58, 8], None, {"manifolds_per_body": 10.0}),
    ([85], [40], {}),                                 # the same at the default capacity
    ([85], [1060], {"manifolds_per_body": 4.0}),      # on chip, but not with the shared words: one wave
])
def test_towers_at_the_lds_limit_are_stepped(J, levels, pushes, kw):
    a = _after(J, _towers(levels, pushes), warm_start=1, **kw)
    b = _after(J, _towers(levels), warm_start=1, small_batch=-1)
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("levels,pushes,kw", [
    ([84, 8], [0, 100], {}),      # one's bodies and the other's pushes are more than a workgroup's LDS
    ([83, 60, 8, 8, 8, 8, 8], [0, 40, 0, 300, 700, 1100, 2100], {}),
])
def test_towers_that_fit_alone_are_stepped_together(J, levels, pushes, kw):
    a = _after(J, _towers(levels, pushes), warm_start=1, **kw)
    b = _after(J, _towers(levels), warm_start=1, pack_bodies=-1)
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


def test_shared_packs_hold_their_pushes(J):
    """Ten towers would share a pack of 250 bodies, but not with 450 pushes each."""
    a = _after(J, _towers([8] * 10, [450] * 10), pack_bodies=250)
    for x, y in zip(a, _after(J, _towers([8] * 10))):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("pushes,start", [(4050, 0), (4062, 1), (4062, 2)])
def test_islands_hold_as_many_pushes_as_lds(J, pushes, start):
    """An island's push rows leave LDS for some of its waves' words only: it runs fewer of them."""
    kw = dict(warm_start=start)
    if start == 2:
        kw.update(mlp=np.load(NET), mlp_iters=4)
    for x, y in zip(_after(J, _towers([100], [pushes]), **kw), _after(J, _towers([100]), **kw)):
        np.testing.assert_array_equal(x, y)


def _heaps(n, dense):
    """Towers of 54 cubes: three by three by six of them pressed together (365 pairs) or apart (none)."""
    k = np.stack(np.meshgrid(range(3), range(3), range(6), indexing="ij"), -1).reshape(-1, 3)
    sb = W.SceneBuilder(W.default_params(), 1)
    for t in range(n):
        pos = k * (0.0199 if dense(t) else 0.1) + [0.0, 0.0, 0.5]
        sb.add_tower(np.full((54, 3), 0.01), np.full(54, 0.01), pos, np.tile([1.0, 0, 0, 0], (54, 1)), 0.4)
    return sb.build()


def test_a_batch_in_shared_packs_has_room_for_a_heap(J):
    """2,100 towers, just more than get a workgroup each: a heap beside a tower without contacts has 365 pairs."""
    w = J.World(_heaps(2100, lambda t: t < 40 and t % 2 == 0))
    w.step(1)
    assert w.stats().error_word == 0
    assert [w.stats(t).manifolds for t in range(0, 40, 2)] == [365] * 20
    state = [x[:54] for x in w.state()]
    w.close()
    alone = J.World(_heaps(1, lambda t: True), manifolds_per_body=8.0)
    alone.step(1)
    for x, y in zip(state, alone.state()):
        np.testing.assert_array_equal(x, y)
    alone.close()


@pytest.mark.parametrize("what,start", [("episodes", 0), ("episodes", 1), ("friction_cone", 0), ("restitution_bias", 1),
                                        ("manifold_mode", 0), ("manifold_mode", 1)])
def test_shared_packs_of_both_builds_give_the_same_bits(J, what, start):
    """2,100 packs of one tower (with the criteria, three waves to a SIMD) and 420 of five (two)."""
    sc = W.tilted_towers(5, 2100, levels_range=(8, 8), n_steps=8)
    if what != "episodes":
        sc = dict(sc, params=dict(sc["params"], **{what: 1}))
    out = []
    for bodies in (24, 120):
        w = J.World(sc, warm_start=start, pack_bodies=bodies, manifolds_per_body=6.0)
        if what == "episodes":
            w.begin_episodes()
        w.step(2)
        w.step(2)
        st = w.stats()
        assert st.error_word == 0
        out.append([*w.state(), np.asarray([st.candidates, st.manifolds, st.points, st.colours])] +
                   ([np.frombuffer(bytes(w.episode(t)), np.uint8) for t in range(0, 2100, 50)] if what == "episodes" else []))
        w.close()
    for x, y in zip(*out):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("start", [0, 1])
def test_pair_words_on_chip_give_the_same_bits(J, start):
    """600 towers, one to a pack with its pairs' words in LDS, and in shared packs with them in device memory."""
    sc = W.tilted_towers(5, 600, levels_range=(8, 20), n_steps=8)
    for x, y in zip(_after(J, sc, warm_start=start), _after(J, sc, warm_start=start, pack_bodies=128)):
        np.testing.assert_array_equal(x, y)
