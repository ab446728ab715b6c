"""Disc friction where a point has no normal impulse and a tangential one whose square is denormal."""
import numpy as np
import pytest

from paper_2606_28394_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("route", [dict(), dict(small_batch=-1), dict(pack_bodies=-1), dict(mega=1)],
                         ids=["small_batch", "one_wave", "island", "grid"])
@pytest.mark.parametrize("speed", [1e-19, 1e-17])
def test_tiny_slip_without_load_stays_finite(route, speed):
    """A box that presses into the ground at rest, without gravity: its points carry no load, so the ground
    holds nothing back, and its slip keeps every bit."""
    from paper_2606_28394_amd import jenga as J
    kw = dict(route)
    sb = W.SceneBuilder(W.default_params(friction_cone=1, gravity=(0.0, 0.0, 0.0), mega_bodies=kw.pop("mega", 0)), 2)
    he, m = W.BLOCK_HALF, W.BLOCK_MASS
    sb.add_tower([he], [m], [[0, 0, he[2] - 1e-4]], [[1, 0, 0, 0]], 0.4, [[speed, -0.5 * speed, 0.0]], None)
    w = J.World(sb.build(), **kw)
    w.step(2)
    x, q, v, om = w.state()
    st = w.stats()
    w.close()
    assert st.error_word == 0 and st.manifolds > 0
    np.testing.assert_array_equal(v, np.asarray([[speed, -0.5 * speed, 0.0]], np.float32))
    assert np.isfinite(x).all() and np.isfinite(q).all() and not om.any()
