"""Grid-wide sweeps in which a body has more visits than the byte that counts them holds, against the oracle."""
import pytest

from paper_2606_28394_amd import workloads as W
from test_gpu_mega import _compare

pytestmark = pytest.mark.gpu


def test_more_visits_than_a_byte_counts(oracle):
    from paper_2606_28394_amd import jenga as J
    # (a stone touches four to six others: 70 sweeps are 280 visits and more)
    sc = W.masonry_wall(24, 12, seed=5, n_steps=2, params=W.default_params(iters=70, mega_bodies=1, colour_partition=64))
    ow = oracle.OracleWorld(sc)
    _compare(J, oracle, sc, [(ow.x.copy(), ow.q.copy(), ow.v.copy(), ow.w.copy())], "wall 24x12, 70 sweeps")
