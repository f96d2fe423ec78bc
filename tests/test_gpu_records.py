"""Records (dumbbell centres, per-system mean positions) at the sizes where
the record kernel's tiles and batches begin and end. The mean is the plain sum
in ascending sphere index divided by the count, so the comparison is exact."""
import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params

pytestmark = pytest.mark.gpu


def _ascending_mean(X):
    s = np.zeros(3)
    for x in X:
        s = s + x
    return s / len(X)


@pytest.mark.parametrize("sizes", [[1], [8], [9], [255], [256], [257], [264], [520], [1, 300, 8, 512, 7]])
def test_record_is_the_ascending_mean(sizes):
    rng = np.random.default_rng(sum(sizes))
    n = 2 * sum(sizes)
    # far apart, so that only the record is of interest
    X = 50.0 * np.arange(n)[:, None] * np.array([1.0, 0.5, 0.25]) + rng.uniform(-3, 3, (n, 3))
    sim = P.Simulator(Params(), sizes, precision="fp64")
    sim.set_state(X, rng.uniform(0, 6, sum(sizes)))
    centres, com, code = sim.run(2, 1)
    assert code == 0
    Xg = sim.get_state()[0].cpu().numpy()
    assert np.array_equal(centres[1].cpu().numpy(), 0.5 * (Xg[0::2] + Xg[1::2]))
    off = np.concatenate([[0], np.cumsum(2 * np.asarray(sizes))])
    want = np.array([_ascending_mean(Xg[off[b]:off[b + 1]]) for b in range(len(sizes))])
    assert np.array_equal(com[1].cpu().numpy(), want)
