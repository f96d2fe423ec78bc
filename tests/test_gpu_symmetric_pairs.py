"""The FP32C pair sum that forms every unordered pair once (one large system,
fused = 0): part-filled blocks and chunks, both block sizes, hi/lo and single
positions, RPY, and the steric candidates it records."""
from dataclasses import replace

import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params, make_single

pytestmark = pytest.mark.gpu

# the bar of the launch-shape gate: relative error of a one-step displacement
GATE = 5e-7


def _displacements(params, X, phi, n, **kw):
    s = P.Simulator(params, [len(phi)], **kw)
    s.set_state(X, phi)
    s.step(n)
    out = s.get_state()[0].cpu().numpy() - X
    assert s.check() == 0
    return out


@pytest.mark.parametrize("tensor", ["oseen", "rpy"])
@pytest.mark.parametrize("N,posmode", [(8704, 1), (9728, 1), (9730, 1), (9792, 1), (10238, 1), (10242, 1), (32770, 1),
                                       (13312, 2), (16384, 2), (16898, 2), (33794, 2)])
def test_one_step_against_fp64(N, posmode, tensor):
    sus = make_single(N // 2, 240.0 * (N / 4096) ** (1 / 3), 1)
    got = _displacements(sus.params, sus.X, sus.phi, 1, precision="fp32c", tensor=tensor,
                         launch=dict(fused=0, posmode=posmode))
    want = _displacements(sus.params, sus.X, sus.phi, 1, precision="fp64_tiled", tensor=tensor)
    assert np.linalg.norm(got - want) <= GATE * np.linalg.norm(want)
    # no sphere is left out or counted twice: each one's error is small too
    assert np.linalg.norm(got - want, axis=1).max() <= 1e-5 * np.linalg.norm(want, axis=1).mean()


@pytest.mark.parametrize("integrator", ["rk4", "heun"])
def test_replayed_and_split_steps_give_the_same_bits(integrator):
    sus = make_single(4900, 320.0, 2)
    kw = dict(precision="fp32c", integrator=integrator, launch=dict(fused=0, posmode=1))
    a = _displacements(sus.params, sus.X, sus.phi, 19, graph=True, **kw)
    b = _displacements(sus.params, sus.X, sus.phi, 19, **kw)
    s = P.Simulator(sus.params, [sus.S], graph=True, **kw)
    s.set_state(sus.X, sus.phi)
    for n in (1, 4, 14):
        s.step(n)
        s.mobility(sus.X, np.ones_like(sus.X))  # shares the partial sums' memory
    assert np.array_equal(a, b) and np.array_equal(a, s.get_state()[0].cpu().numpy() - sus.X)


@pytest.mark.parametrize("N,posmode,side,rmin", [(4096, 1, 120.0, 1.6), (4098, 2, 120.0, 1.6), (8192, 1, 170.0, 1.6), (8194, 1, 90.0, 1.8), (8702, 2, 100.0, 1.6),
                                               (8704, 1, 170.0, 1.6), (8706, 1, 90.0, 1.8), (9214, 2, 100.0, 1.6)])
def test_steric_contacts_against_fp64(N, posmode, side, rmin):
    """Contacts across chunks and blocks, dense enough that several lie in one
    group of steps; the FP64 form sums every pair."""
    p = replace(Params(), steric_k=100.0)
    sus = make_single(N // 2, side, 3, params=p, rmin=rmin)
    got = _displacements(p, sus.X, sus.phi, 2, precision="fp32c", launch=dict(fused=0, posmode=posmode))
    want = _displacements(p, sus.X, sus.phi, 2, precision="fp64_tiled")
    # single-float positions lose most where contacts leave net forces
    assert np.linalg.norm(got - want) <= (1e-6 if posmode == 1 else 2e-5) * np.linalg.norm(want)
