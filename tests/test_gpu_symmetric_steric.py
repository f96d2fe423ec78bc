"""The symmetric FP32C pair sum with steric forces: with the Rotne-Prager
correction, single-float positions and both block sizes. The spheres in contact
are compared on their own, since a candidate that is missed would hardly show in
a norm over all."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import paper_1004_1932_amd as P
from paper_1004_1932_amd import autotune
from workload import Params, make_single

pytestmark = pytest.mark.gpu


def _in_contact(X, reach):
    """Spheres with another dumbbell's sphere nearer than reach."""
    x = torch.as_tensor(X).cuda()
    out = torch.zeros(len(X), dtype=torch.bool, device=x.device)
    own = torch.arange(len(X), device=x.device) // 2
    for i in range(0, len(X), 2048):
        d = torch.cdist(x[i:i + 2048], x, compute_mode="donot_use_mm_for_euclid_dist")
        out[i:i + 2048] = ((d < reach) & (own[i:i + 2048, None] != own)).any(1)
    return out.cpu().numpy()


@pytest.mark.parametrize("tensor", ["oseen", "rpy"])
@pytest.mark.parametrize("N,posmode,side,rmin", [(8702, 1, 100.0, 1.7), (8704, 1, 100.0, 1.7), (8704, 2, 100.0, 1.7),
                                                 (9730, 2, 120.0, 1.6), (12802, 1, 110.0, 1.8), (32770, 2, 190.0, 1.7),
                                                 (33794, 1, 190.0, 1.7)])
def test_contacts_against_fp64(N, posmode, side, rmin, tensor):
    p = replace(Params(), steric_k=100.0)
    launch = dict(fused=0, posmode=posmode)
    assert autotune.step_ignores_shape(p, [N // 2], launch) == (N >= 8704)  # which kernel this is
    sus = make_single(N // 2, side, 3, params=p, rmin=rmin)
    out = []
    for kw in (dict(precision="fp32c", launch=launch), dict(precision="fp64_tiled")):
        s = P.Simulator(p, [N // 2], tensor=tensor, **kw)
        s.set_state(sus.X, sus.phi)
        s.step(2)
        assert s.check() == 0
        out.append(s.get_state()[0].cpu().numpy() - sus.X)
    # single-float positions lose most where contacts leave net forces
    bar = 1e-6 if posmode == 1 else 2e-5
    assert np.linalg.norm(out[0] - out[1]) <= bar * np.linalg.norm(out[1])
    touch = _in_contact(sus.X, 2.0)
    assert touch.sum() > 50
    # a contact force that is missed moves its spheres by a good part of their own displacement
    each = np.linalg.norm(out[0] - out[1], axis=1)[touch]
    assert each.max() <= 100 * bar * np.linalg.norm(out[1], axis=1)[touch].mean()
