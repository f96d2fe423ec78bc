"""The FP32C pair kernels' steric candidate lists hold spheres of the system
only, also where lengths are so large that the far-away entries that pad a
tile or a block come into reach."""
from dataclasses import replace

import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params, make_single

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("posmode", [1, 2])
@pytest.mark.parametrize("N", [62, 8706, 33794])
def test_reach_beyond_the_padding(N, posmode):
    """Every sphere is in reach of every other and of the padding: the lists
    overflow, which is reported, and nothing else is written: the phases, which
    follow the lists in the workspace, still give the same forces."""
    p = replace(Params(), steric_k=1e-3, steric_r=1e16)
    sus = make_single(N // 2, 20.0 * N ** (1 / 3), 1)
    X = sus.X
    s = P.Simulator(p, [N // 2], precision="fp32c", launch=dict(fused=0, posmode=posmode))
    s.set_state(X, sus.phi)
    before = s.forces(X + 0.25, 0.3).cpu().numpy()
    _, _, code = s.run(1, 0)
    assert code != 0
    after = s.forces(X + 0.25, 0.3).cpu().numpy()
    assert np.array_equal(before, after)


@pytest.mark.parametrize("S", [35, 67])
def test_contacts_near_the_padding_point(S):
    """A suspension at the padding's own coordinates, chunks that end in
    part-filled groups: each sphere has its true contacts only."""
    scale = 1e13
    p = replace(Params(), a=scale, ell=4 * scale, lam=scale, k=1.0, steric_k=100.0, steric_r=2 * scale,
                eta=1.0 / scale)
    sus = make_single(S, 16.0, 3, params=replace(Params(), steric_k=100.0), rmin=1.8)
    X = sus.X * scale + 1e15
    out = []
    for kw in (dict(precision="fp32c", launch=dict(fused=0, jchunk=64, wg=64, ipl=1, posmode=1)),
               dict(precision="fp64_tiled")):
        s = P.Simulator(p, [S], **kw)
        s.set_state(X, sus.phi)
        s.step(2)
        assert s.check() == 0
        out.append(s.get_state()[0].cpu().numpy() - X)
    assert np.linalg.norm(out[0] - out[1]) <= 1e-6 * np.linalg.norm(out[1])
