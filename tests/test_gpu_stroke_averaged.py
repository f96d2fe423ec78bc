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


@pytest.mark.parametrize("S", [1023, 1024, 1025, 1026, 1027, 1028, 2501])
def test_rates_around_the_change_of_waves_per_dumbbell(oracle, S):
    """Four waves a dumbbell up to 1024, one above: every remainder of the last
    work-group's four dumbbells."""
    _rates_match(oracle, Params(), *_config(S, S))


@pytest.mark.parametrize("S", [1024, 1027])
def test_run_around_the_change_of_waves_per_dumbbell(oracle, S):
    p = Params()
    R, N, phi = _config(S, S)
    sa = P.StrokeAveraged(p, R, N, phi)
    assert sa.run(5.0, 7) == 0
    Ro, No = oracle.sa_run(p, R, N, phi, 5.0, 7)
    Rg, Ng = sa.R.cpu().numpy(), sa.N.cpu().numpy()
    # the displacement against positions up to 440: 7 steps' roundings of them
    assert np.abs((Rg - R) - (Ro - R)).max() <= 8 * np.spacing(np.abs(R).max()) + 1e-12 * np.abs(Ro - R).max()
    assert np.abs(Ng - No).max() <= 1e-13


@pytest.mark.parametrize("S", [5, 1030])
def test_coincident_centres_are_flagged_and_left_out(oracle, S):
    R, N, phi = _config(S, S)
    R[S - 1] = R[1]
    assert P.StrokeAveraged(Params(), R, N, phi).run(1.0, 1) == P.binding.AD_ENONFINITE
    keep = np.arange(S) != 1  # the others' rates do not depend on the flag
    got = P.StrokeAveraged(Params(), R, N, phi).rhs()[0].cpu().numpy()
    assert np.isfinite(got[keep]).all()


@pytest.mark.parametrize("S", [40, 1030])
@pytest.mark.parametrize("case", ["phases", "some phases", "close", "far", "one far"])
def test_operands_the_short_forms_do_not_take(oracle, case, S):
    """Phase differences from 2^19 on, D^2 outside 2^+-900, in every lane and
    in some."""
    p = Params()
    R, N, phi = _config(S, S)
    if case == "phases":
        phi = phi + 2.0 ** 19 * 1.5 * np.arange(S)
    elif case == "some phases":
        phi[::7] += 3e6
    elif case in ("close", "far"):
        f = 1e-138 if case == "close" else 1e137
        R, p = R * f, replace(p, a=f, ell=4 * f, lam=f)
    else:
        R[S // 2] = [1e140, 0.0, 0.0]
    _rates_match(oracle, p, R, N, phi)
