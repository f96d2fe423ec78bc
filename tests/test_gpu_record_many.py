"""Records of ensembles either side of the number of systems from which a thread
takes a system's mean: the plain ascending sum divided by the count, exactly."""
import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[1] * 127, [1] * 128, [1] * 300 + [2], [1] * 255 + [2], [4] * 511, [4] * 513,
                                   [3, 1, 2] * 400, [16] * 2048])
def test_means_are_the_ascending_sums(sizes):
    rng = np.random.default_rng(len(sizes))
    n = 2 * sum(sizes)
    X = 5.0 * np.arange(n)[:, None] * np.array([1.0, 0.5, 0.25]) % 977.0 + rng.uniform(-2, 2, (n, 3))
    sim = P.Simulator(Params(), sizes, precision="fp64")
    sim.set_state(X, rng.uniform(0, 6, sum(sizes)))
    centres, com, code = sim.run(1, 1)
    assert code == 0
    Xg = sim.get_state()[0].cpu().numpy()
    assert np.array_equal(centres[0].cpu().numpy(), 0.5 * (Xg[0::2] + Xg[1::2]))
    off = np.concatenate([[0], np.cumsum(2 * np.asarray(sizes))])
    want = np.zeros((len(sizes), 3))
    for b in range(len(sizes)):
        for x in Xg[off[b]:off[b + 1]]:
            want[b] = want[b] + x
    assert np.array_equal(com[0].cpu().numpy(), want / np.diff(off)[:, None])
