"""AD_FP64's short quotients at the operands where a quotient lies nearest to a
rounding boundary: r.F / r2 with r2's significand 2 - (2k + 1) 2^-52, whose
reciprocal itself lies next to one. Products bit for bit the oracle's."""
import math

import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params

pytestmark = pytest.mark.gpu


def hard_numerators(X, offsets=range(-9, 10, 2)):
    """53-bit a with a / X = m + tiny, m odd of 54 bits (a midpoint): a 2^54 = m X - c."""
    inv = pow(X, -1, 1 << 54)
    out = []
    for c in offsets:
        m = inv * c % (1 << 54)
        if m < 1 << 53 or not m & 1:
            continue
        a, rest = divmod(m * X - c, 1 << 54)
        if rest == 0 and 0 < a < 1 << 53:
            out.append(a)
    return out


def separation(r2):
    """(rx, ry) with fl(fl(rx rx) + fl(ry ry)) = r2."""
    rx = math.sqrt(r2)
    for _ in range(40):
        d = r2 - rx * rx
        if d >= 0:
            ry = math.sqrt(d)
            for _ in range(8):
                if rx * rx + ry * ry == r2 and ry > 0:
                    return rx, ry
                ry = np.nextafter(ry, 1.0)
        rx = float(np.nextafter(rx, 0.0))
    return None


def force(rx, a):
    """F with fl(rx F) = a."""
    f = a / rx
    for g in (f, np.nextafter(f, 0.0), np.nextafter(f, np.inf)):
        if rx * float(g) == a:
            return float(g)
    return None


def _cases():
    for k in range(260):
        X = (1 << 53) - (2 * k + 1)
        for e in (-52, -51):
            at = separation(math.ldexp(X, e))
            if at is None:
                continue
            for a in hard_numerators(X):
                f = force(at[0], math.ldexp(a, -49))
                if f is not None:
                    yield at, f


def test_products_bitwise(oracle):
    cases = list(_cases())
    assert len(cases) > 200
    p, wrong = Params(), []
    # one system per case: two spheres, the force on the second
    X = np.array([[[0, 0, 0], [-x, -y, 0]] for (x, y), _ in cases], dtype=float).reshape(-1, 3)
    F = np.array([[[0, 0, 0], [f, 0, 0]] for _, f in cases], dtype=float).reshape(-1, 3)
    for tensor in ("oseen", "rpy"):
        u = P.Simulator(p, [1] * len(cases), precision="fp64", tensor=tensor).mobility(X, F).cpu().numpy()
        for b in range(len(cases)):
            s = slice(2 * b, 2 * b + 2)
            if not np.array_equal(u[s], oracle.mobility(p, X[s], F[s], int(tensor == "rpy"))):
                wrong.append((tensor, cases[b]))
    assert not wrong, (len(wrong), wrong[:3])
