"""The resident FP64 form either side of 16 spheres, up to which a thread forms
its pair's separation and spring force side by side by the short quotients:
bit for bit the two-kernel FP64 form, also where the short quotients do not
hold (operands out of their range, zero forces)."""
from dataclasses import replace

import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import make_single

pytestmark = pytest.mark.gpu


def _run(params, X, phi, n, fused, **kw):
    s = P.Simulator(params, [len(phi)], precision="fp64", launch=dict(fused=fused), **kw)
    s.set_state(X, phi)
    s.step(n)
    return s.get_state()[0].cpu().numpy(), s.check()


@pytest.mark.parametrize("tensor", ["oseen", "rpy"])
@pytest.mark.parametrize("integrator,kT", [("rk4", 0.0), ("heun", 0.0), ("heun", 0.02)])
@pytest.mark.parametrize("N", [2, 4, 8, 10, 14, 16, 18, 24, 128])
def test_same_bits_as_two_kernels(N, integrator, kT, tensor):
    sus = make_single(N // 2, 15.0 * N ** (1 / 3), 5)
    kw = dict(integrator=integrator, kT=kT, seed=3, tensor=tensor)
    a, b = (_run(sus.params, sus.X, sus.phi, 37, f, **kw) for f in (4, 0))
    assert np.array_equal(a[0], b[0]) and a[1] == b[1] == 0


@pytest.mark.parametrize("scale,k", [(1e-65, 1.0), (1e62, 1.0), (1.0, 0.0), (1.0, 1e-160), (1.0, 1e155)])
@pytest.mark.parametrize("N", [6, 16])
def test_operands_the_short_forms_do_not_take(N, scale, k):
    sus = make_single(N // 2, 20.0, 6)
    p = replace(sus.params, k=k)
    a, b = (_run(p, sus.X * scale, sus.phi, 1, f) for f in (4, 0))
    assert np.array_equal(a[0], b[0], equal_nan=True) and a[1] == b[1]


def test_coincident_spheres_are_flagged():
    sus = make_single(8, 20.0, 7)
    X = sus.X.copy()
    X[9] = X[2]
    a, b = (_run(sus.params, X, sus.phi, 1, f) for f in (4, 0))
    assert np.array_equal(a[0], b[0], equal_nan=True) and a[1] == b[1] != 0
