"""ad_mobility_apply under every stage form a launch can select: the product
uses the pair kernel's own work list, whatever list the stage form needs."""
import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params, make_single

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tensor", ["oseen", "rpy"])
@pytest.mark.parametrize("sizes", [[1], [8], [32], [3, 20, 1, 32]])
def test_fp64_mobility_with_the_resident_form(oracle, sizes, tensor):
    """launch="tuned" selects the resident form for small FP64 systems: the
    velocities stay bitwise the sequential sum's."""
    X = np.concatenate([make_single(S, 60.0, 3 + b).X for b, S in enumerate(sizes)])
    F = np.random.default_rng(5).standard_normal(X.shape)
    sim = P.Simulator(Params(), sizes, precision="fp64", launch="tuned", tensor=tensor)
    assert sim.launch["fused"] == 4
    u = sim.mobility(X, F).cpu().numpy()
    off = np.concatenate([[0], np.cumsum(2 * np.asarray(sizes))])
    for b in range(len(sizes)):
        sl = slice(off[b], off[b + 1])
        want = oracle.mobility(Params(), X[sl], F[sl], int(tensor == "rpy"))
        assert np.array_equal(u[sl], want), b
