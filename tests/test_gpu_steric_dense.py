"""Full steric sums with many spheres in reach of each other, whose terms are
added by rows, beside few, added one by one: bit for bit the oracle's sums in
ascending j."""
from dataclasses import replace

import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params

pytestmark = pytest.mark.gpu


def _check(oracle, p, sizes, X, phi):
    s = P.Simulator(p, sizes, precision="fp64")
    s.set_state(X, phi)
    got = s.forces(X, 0.3).cpu().numpy()
    off = 2 * np.concatenate([[0], np.cumsum(sizes)])
    for b in range(len(sizes)):
        x = slice(off[b], off[b + 1])
        want = oracle.forces(p, X[x], phi[off[b] // 2:off[b + 1] // 2], 0.3, allow_nonfinite=True)
        assert np.array_equal(got[x], want, equal_nan=True), b


@pytest.mark.parametrize("reach", [3.0, 8.0, 12.0, 1e4])
@pytest.mark.parametrize("sizes", [[1], [8], [9], [16], [31], [33], [65], [200], [8195], [1, 7, 33, 2, 90, 64], [5] * 700])
def test_forces_bitwise(oracle, sizes, reach):
    p = replace(Params(), steric_k=100.0, steric_r=reach)
    rng = np.random.default_rng(len(sizes) + sizes[0])
    n = sum(sizes)
    X = rng.uniform(0, 5.0 * max(sizes) ** (1 / 3), (2 * n, 3))
    _check(oracle, p, sizes, X, rng.uniform(0, 6.0, n))


@pytest.mark.parametrize("what", ["coincident", "nan", "infinite"])
def test_special_distances_among_many_in_reach(oracle, what):
    p = replace(Params(), steric_k=100.0, steric_r=50.0)
    rng = np.random.default_rng(3)
    X = rng.uniform(0, 40, (400, 3))
    X[130] = {"coincident": X[7], "nan": np.nan, "infinite": np.inf}[what]
    _check(oracle, p, [200], X, rng.uniform(0, 6.0, 200))
    if what == "coincident":
        s = P.Simulator(p, [200], precision="fp64")
        s.set_state(X, np.zeros(200))
        s.forces(X, 0.3)
        assert s.check() == P.binding.AD_ENONFINITE
