"""Islands stepped by the whole GPU (towers of at least mega_bodies bodies): the cooperative
grid-wide kernel against the oracle, which colours such towers with the same partitioned rule.

- a 1,152-stone wall forced onto the path (mega_bodies 256, partitions of 128 stones): one step
  from the initial state and from the state 20 steps on (pair sets, colours, points exactly,
  impulses on the first step, velocities at the walls' 1e-3 after it);
- one partition: the colouring is the canonical greedy one, so the grid-wide kernel must give
  what the island path (one workgroup, device memory) gives, to a few FP32 roundings;
- a site-scale wall of 100,000 stones (100 courses x 1,000): one step against the oracle;
- small scenes for the kernel's other branches: one step against the oracle.
"""
import os
import sys
import time

import numpy as np
import pytest

from paper_2606_28394_amd import workloads as W
from parity_util import compare_contacts, compare_state, fmt, gpu_manifolds, impulses_feasible, oracle_manifolds

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def J():
    from paper_2606_28394_amd import jenga
    jenga.load_library()
    return jenga


def _say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _wall(courses, per_course, n_steps=40, **params):
    sc = W.masonry_wall(courses, per_course, seed=7, n_steps=n_steps)
    sc["params"] = dict(sc["params"], **params)
    return sc


def _compare(J, oracle, sc, states, label):
    """One step from each state on both sides.  Both start from the state rounded to FP32 (what
    the GPU holds): 300 m from the origin an FP32 position resolves 30 um, so pairs that overlap
    by less than that would otherwise differ by the input rounding rather than by the arithmetic."""
    ow = oracle.OracleWorld(sc)
    gw = J.World(sc)
    for si, S in enumerate(states):
        S = tuple(np.asarray(z, np.float32).astype(np.float64) for z in S)
        ow.set_state(*S)
        gw.set_state(*S)
        t0 = time.time()
        ow.step(1)
        t1 = time.time()
        gw.step(1)
        st = gw.stats()
        assert st.error_word == 0, f"{label}: device error word {st.error_word}"
        gc = gw.contacts(0)
        rep = compare_contacts(oracle_manifolds(ow, 0), gpu_manifolds(gc, 0), sc["mass"], impulses=(si == 0))
        _say(label, si, "oracle step", round(t1 - t0, 1), "s;", fmt(rep)[:260])
        assert rep["ok"], f"{label} state {si}: {fmt(rep)}"
        assert impulses_feasible(gc, float(sc["mu"][0]))
        cs = compare_state(ow, *gw.state(), vtol=1e-4 if si == 0 else 1e-3)
        _say(label, si, "state", cs)
        assert cs["ok"], f"{label} state {si}: {cs}"
        if si == 0:
            assert abs(st.residual_rms - ow.tower_stats(0).res_rms) <= 1e-2 * ow.tower_stats(0).res_rms + 1e-7
    gw.close()


def test_grid_wide_wall_matches_oracle(J, oracle):
    sc = _wall(24, 48, mega_bodies=256, colour_partition=128)
    ow = oracle.OracleWorld(sc)
    states = [(ow.x.copy(), ow.q.copy(), ow.v.copy(), ow.w.copy())]
    ow.step(20)
    states.append((ow.x.copy(), ow.q.copy(), ow.v.copy(), ow.w.copy()))
    _compare(J, oracle, sc, states, "wall 24x48, partitions of 128")


def test_one_partition_matches_island_path(J):
    """With one partition the grid-wide kernel computes what one workgroup computes: same pairs,
    colours and slots every step, states within a few FP32 roundings over 10 steps."""
    base = _wall(16, 32, n_steps=12)
    mega = dict(base, params=dict(base["params"], mega_bodies=256, colour_partition=1 << 20))
    gi = J.World(base, pack_bodies=-1)
    gm = J.World(mega)
    for k in range(10):
        gi.step(1)
        gm.step(1)
        ci, cm = gpu_manifolds(gi.contacts(0), 0), gpu_manifolds(gm.contacts(0), 0)
        assert set(ci) == set(cm), k
        assert all(ci[p]["colour"] == cm[p]["colour"] and list(ci[p]["slot"]) == list(cm[p]["slot"]) for p in ci), k
    (xi, qi, vi, wi), (xm, qm, vm, wm) = gi.state(), gm.state()
    ex = float(np.abs(xi - xm).max())
    ev = float(np.abs(vi - vm).max())
    _say("one partition vs island path after 10 steps: x", ex, "v", ev)
    assert ex <= 1e-6 and float(np.abs(qi - qm).max()) <= 1e-5 and ev <= 1e-4
    si, sm = gi.stats(), gm.stats()
    assert si.candidates == sm.candidates and si.manifolds == sm.manifolds and si.points == sm.points
    gi.close()
    gm.close()


def test_site_scale_wall_matches_oracle(J, oracle):
    """100,000 stones in one island (the default path for islands of 16,384 bodies or more)."""
    sc = _wall(100, 1000, n_steps=2)
    assert int(sc["tower_ptr"][-1]) == 100_000
    ow = oracle.OracleWorld(sc)
    _compare(J, oracle, sc, [(ow.x.copy(), ow.q.copy(), ow.v.copy(), ow.w.copy())], "wall 100x1000")


def _crowded_slab(**params):
    """A slab with 49 boxes on it: 50 colours, a body with 49 near boxes, and a lane pair with more
    visits in a sweep than it has records in LDS."""
    n = 7
    he = [[2.0, 2.0, 0.1]] + [[0.1, 0.1, 0.1]] * (n * n)
    mass = [900.0] + [4.0] * (n * n)
    pos = [[0.0, 0.0, 0.1 - 1e-4]]
    pos += [[0.5 * (i - 3), 0.5 * (j - 3), 0.3 - 2e-4] for i in range(n) for j in range(n)]
    vel = np.zeros((n * n + 1, 3))
    vel[0, 0] = 0.2
    sb = W.SceneBuilder(dict(W.default_params(), **params), n_steps=4)
    sb.add_tower(np.array(he), np.array(mass), np.array(pos), np.tile([1.0, 0.0, 0.0, 0.0], (n * n + 1, 1)), 0.5, vel,
                 np.zeros((n * n + 1, 3)))
    return sb.build()


@pytest.mark.parametrize("label,courses,per_course,params", [
    ("crowded slab", 0, 0, {}),
    ("two stones", 1, 2, {}),
    ("pairs between partitions far apart", 10, 48, dict(colour_partition=16)),
    ("partitions too large for LDS", 48, 48, dict(colour_partition=2100)),
    ("more near boxes than a walk keeps", 8, 16, dict(margin=0.5, mega_cand_per_body=120.0)),
    ("disc friction", 8, 16, dict(friction_cone=1, colour_partition=32)),
    ("restitution targets", 8, 16, dict(restitution=0.3, restitution_bias=1, colour_partition=32)),
])
def test_grid_wide_edges_match_oracle(J, oracle, label, courses, per_course, params):
    """The kernel's branches at small sizes, one step against the oracle (the bounds of the walls)."""
    sc = _wall(courses, per_course, mega_bodies=1, **params) if courses else _crowded_slab(mega_bodies=1)
    ow = oracle.OracleWorld(sc)
    _compare(J, oracle, sc, [(ow.x.copy(), ow.q.copy(), ow.v.copy(), ow.w.copy())], label)
