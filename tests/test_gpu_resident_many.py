"""The resident FP64 form either side of the numbers of systems up to which
all of them are resident at once with the form of up to 16 spheres, beyond which
the kernel without it takes them: bit for bit the form with a launch per stage."""
import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params, make_single

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tensor", ["oseen", "rpy"])
@pytest.mark.parametrize("integrator,kT", [("rk4", 0.0), ("heun", 0.0), ("heun", 0.02)])
@pytest.mark.parametrize("W,S", [(768, 5), (769, 5), (1024, 5), (1025, 8), (1281, 3), (1300, 7), (2100, 2)])
def test_same_bits_as_two_kernels(W, S, integrator, kT, tensor):
    ens = [make_single(S, 15.0 * (2 * S) ** (1 / 3), 60 + b) for b in range(7)]
    sizes = [S] * W
    X = np.concatenate([ens[b % 7].X for b in range(W)])
    phi = np.random.default_rng(W).uniform(0.0, 6.0, W * S)
    out = []
    for fused in (4, 0):
        s = P.Simulator(Params(), sizes, precision="fp64", launch=dict(fused=fused), integrator=integrator, kT=kT,
                        seed=3, tensor=tensor)
        s.set_state(X, phi)
        s.step(5)
        assert s.check() == 0
        out.append(s.get_state()[0].cpu().numpy())
    assert np.array_equal(*out)


def test_systems_of_few_and_of_many_spheres_together():
    sizes = [1, 8, 9, 3] * 300
    ens = {S: make_single(S, 15.0 * (2 * S) ** (1 / 3), S) for S in (1, 8, 9, 3)}
    X, phi = np.concatenate([ens[S].X for S in sizes]), np.concatenate([ens[S].phi for S in sizes])
    out = []
    for fused in (4, 0):
        s = P.Simulator(Params(), sizes, precision="fp64", launch=dict(fused=fused))
        s.set_state(X, phi)
        s.step(5)
        out.append(s.get_state()[0].cpu().numpy())
    assert np.array_equal(*out)
