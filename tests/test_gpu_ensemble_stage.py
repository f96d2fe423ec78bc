"""The ensemble forms of the fused stage (sources in LDS, 16 or 64 targets per
work-group) at system sizes where a wave's share of the sources, the chunks
that hold the work-group's own spheres and the groups of four begin and end."""
import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params, make_single

pytestmark = pytest.mark.gpu

# the bar of the launch-shape gate: relative error of a displacement
GATE = 5e-7


@pytest.mark.parametrize("integrator,kT,tensor", [("rk4", 0.0, "oseen"), ("heun", 0.02, "rpy")])
@pytest.mark.parametrize("posmode", [1, 2])
@pytest.mark.parametrize("fused", [1, 2])
def test_every_size_of_a_systems_share_against_fp64(fused, posmode, integrator, kT, tensor):
    sizes = [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 34, 35, 47, 61, 63, 64, 65, 66, 67, 68, 69, 70, 97, 130, 201]
    ens = [make_single(S, 18.0 * S ** (1 / 3) + 10.0, 20 + S) for S in sizes]
    X, phi = np.concatenate([e.X for e in ens]), np.concatenate([e.phi for e in ens])
    out = []
    for kw in (dict(precision="fp32c", launch=dict(fused=fused, posmode=posmode)), dict(precision="fp64")):
        s = P.Simulator(Params(), sizes, integrator=integrator, kT=kT, seed=5, tensor=tensor, **kw)
        s.set_state(X, phi)
        s.step(3)
        assert s.check() == 0
        out.append(s.get_state()[0].cpu().numpy() - X)
    off = np.concatenate([[0], np.cumsum(2 * np.asarray(sizes))])
    for b, S in enumerate(sizes):
        g, w = (o[off[b]:off[b + 1]] for o in out)
        assert np.linalg.norm(g - w) <= GATE * np.linalg.norm(w), S
        # a term left out or counted twice shows at one sphere
        assert np.linalg.norm(g - w, axis=1).max() <= 1e-5 * np.linalg.norm(w, axis=1).mean(), S
