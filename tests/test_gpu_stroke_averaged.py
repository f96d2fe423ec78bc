"""The stroke-averaged equations on the GPU against the oracle, at the edges of
their forms: one wave per dumbbell above 1024 (four dumbbells a work-group),
operands outside the short sine and reciprocal square root, and a dumbbell's
own masked term."""
from dataclasses import replace

import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params

pytestmark = pytest.mark.gpu


def _config(S, seed, spacing=40.0):
    """A jittered lattice, unit axes, phases."""
    rng = np.random.default_rng(seed)
    x = int(np.ceil(round(S ** (1 / 3), 9)))
    idx = np.stack(np.meshgrid(*[np.arange(x)] * 3, indexing="ij"), -1).reshape(-1, 3)[:S]
    N = rng.standard_normal((S, 3))
    return (spacing * (idx + rng.uniform(-0.3, 0.3, (S, 3))), N / np.linalg.norm(N, axis=1)[:, None],
            rng.uniform(0.0, 6.0, S))


def _rates_match(oracle, p, R, N, phi):
    """1e-13: sums of n terms of mixed sign, each within a few ulp."""
    got = P.StrokeAveraged(p, R, N, phi).rhs()
    for g, o in zip(got, oracle.sa_rhs(p, R, N, phi)):
        g = g.cpu().numpy()
        assert np.isfinite(g).all()
        # scaled: the norms of very large or small rates would overflow
        u = np.abs(o).max()
        assert np.linalg.norm(g / u - o / u) <= 1e-13 * np.linalg.norm(o / u)


@pytest.mark.parametrize("S", [2, 129, 1030])
def test_own_term_of_large_lengths(oracle, S):
    """A dumbbell's own term is left out whatever ell is: ell^4 overflows here,
    (ell / D)^4 does not."""
    R, N, phi = _config(S, S)
    p = replace(Params(), a=1e79, ell=4e80, lam=1e80)
    _rates_match(oracle, p, R * 1e80, N, phi)
    one = P.StrokeAveraged(p, R[:1], N[:1], phi[:1]).rhs()
    assert all((v == 0.0).all() for v in one)
