"""The streamed stage kernel either side of the sizes where its targets per
work-group change, and the noise formed inside the stage kernels."""
import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params, make_single

pytestmark = pytest.mark.gpu


def _run(sus, n, **kw):
    s = P.Simulator(sus.params, [sus.S], **kw)
    s.set_state(sus.X, sus.phi)
    s.step(n)
    assert s.check() == 0
    return s.get_state()[0].cpu().numpy() - sus.X


# the bar of the launch-shape gate: relative error of a displacement
GATE = 5e-7


@pytest.mark.parametrize("integrator,kT", [("rk4", 0.0), ("heun", 0.0), ("heun", 0.02)])
@pytest.mark.parametrize("posmode", [1, 2])
@pytest.mark.parametrize("N", [2, 1022, 1024, 1026, 2046, 2048, 4094, 4096, 4098, 8194])
def test_streamed_stage_against_fp64(N, posmode, integrator, kT):
    sus = make_single(N // 2, 240.0 * (N / 4096) ** (1 / 3) + 10.0, 4)
    kw = dict(integrator=integrator, kT=kT, seed=11)
    got = _run(sus, 3, precision="fp32c", launch=dict(fused=3, posmode=posmode), **kw)
    want = _run(sus, 3, precision="fp64", **kw)
    assert np.linalg.norm(got - want) <= GATE * np.linalg.norm(want)
    # the noise is the same FP64 numbers on both sides; what the FP32 sums add
    # is small for every sphere
    assert np.linalg.norm(got - want, axis=1).max() <= 1e-5 * np.linalg.norm(want, axis=1).mean()


@pytest.mark.parametrize("seed", [0, 7, 2 ** 40 + 3])
def test_noise_normals_against_the_oracle(oracle, seed):
    """A force-free, far-apart pair of spheres moves by the noise alone, whose
    normals are the oracle's to a few ulp of log, sin and cos (1e-14: the
    displacement's own rounding at positions near 1)."""
    p = Params(k=0.0, lam=0.0)
    n = 400
    X = np.zeros((2, 3))
    X[1] = [1.0, 0.0, 0.0]
    s = P.Simulator(p, [1], precision="fp64", integrator="heun", kT=0.5, seed=seed)
    s.set_state(X, np.zeros(1))
    g = np.sqrt(2.0 * 0.5 / (6.0 * np.pi) * p.dt)
    prev = X
    for step in range(n):
        s.step(1)
        now = s.get_state()[0].cpu().numpy()
        z = np.array([oracle.gauss3(seed, i, step) for i in range(2)])
        assert np.abs((now - prev) - g * z).max() <= 1e-14 * (1.0 + np.abs(now).max())
        prev = now
