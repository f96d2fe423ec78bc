"""The full steric sums (forces of a state, first stage, FP64 stages): bit for
bit the plain sum in ascending j, for the sizes where the spheres per wave and
the last tile of sources change."""
from dataclasses import replace

import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params

pytestmark = pytest.mark.gpu


def _plain(p, X, off, F):
    """F plus the steric sums, each in ascending j, as the kernel's operations."""
    F = F.copy()
    rc2 = p.steric_r * p.steric_r
    for j0, j1 in zip(off[:-1], off[1:]):
        Y = X[j0:j1]
        for i in range(len(Y)):
            r = Y[i] - Y
            r2 = (r[:, 0] * r[:, 0] + r[:, 1] * r[:, 1]) + r[:, 2] * r[:, 2]
            near = np.nonzero(~(r2 >= rc2) & (r2 != 0.0))[0]
            acc = np.zeros(3)
            for j in near:
                if j != i:
                    d = np.sqrt(r2[j])
                    acc = acc + p.steric_k * (p.steric_r - d) / d * r[j]
            if len(near):
                F[j0 + i] = F[j0 + i] + acc
    return F


def _forces(params, sizes, X, phi):
    s = P.Simulator(params, sizes, precision="fp64")
    s.set_state(X, phi)
    return np.asarray(s.forces(X, 0.3).cpu())


@pytest.mark.parametrize("sizes", [[1], [2], [31], [32], [33], [65], [500], [8191], [8193], [8195], [1, 7, 33, 2, 90], [2] * 1023, [2] * 1024])
def test_forces_bitwise(sizes):
    p = replace(Params(), steric_k=100.0)
    rng = np.random.default_rng(len(sizes) + sizes[0])
    n = sum(sizes)
    X = rng.uniform(0, 3.0 * max(sizes) ** (1 / 3), (2 * n, 3))
    phi = rng.uniform(0, 6.0, n)
    off = 2 * np.concatenate([[0], np.cumsum(sizes)])
    springs = _forces(replace(p, steric_k=0.0), sizes, X, phi)
    got = _forces(p, sizes, X, phi)
    want = _plain(p, X, off, springs)
    assert n == 1 or not np.array_equal(want, springs)
    assert np.array_equal(got, want)


def test_coincident_spheres_and_nan():
    p = replace(Params(), steric_k=100.0)
    X = np.random.default_rng(0).uniform(0, 40, (200, 3))
    phi = np.zeros(100)
    X[150] = X[31]
    s = P.Simulator(p, [100], precision="fp64")
    s.set_state(X, phi)
    s.step(1)
    assert s.check() != 0
    X[150] = np.nan
    F = np.asarray(s.forces(X, 0.0).cpu())
    assert np.isnan(F).all()  # the plain sum adds a NaN distance to every sphere
