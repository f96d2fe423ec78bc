"""A launch shape whose steps would take the symmetric pair sum, on a workspace
bound for another shape that does not hold its partial sums: the state is kept
and the ordered pair sum steps it."""
import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params, make_single

pytestmark = pytest.mark.gpu


def test_set_launch_keeps_the_state():
    N = 9000
    sus = make_single(N // 2, 300.0, 1)
    want = P.Simulator(sus.params, [sus.S], precision="fp64_tiled")
    want.set_state(sus.X, sus.phi)
    want.step(3)
    shape = dict(ipl=1, jchunk=512, wg=256, wj=4, posmode=1)
    s = P.Simulator(sus.params, [sus.S], precision="fp32c", launch=dict(shape, fused=3), graph=True)
    s.set_state(sus.X, sus.phi)
    s.step(1)
    ws = s.ws.data_ptr()
    s.set_launch(**shape, fused=0)
    s.step(1)               # the state is still there
    s.set_launch(**shape, fused=3)
    s.set_launch(**shape, fused=0)
    s.step(1)
    assert s.ws.data_ptr() == ws and s.check() == 0
    d, w = (x.get_state()[0].cpu().numpy() - sus.X for x in (s, want))
    assert np.linalg.norm(d - w) <= 5e-7 * np.linalg.norm(w)


def test_a_larger_workspace_takes_it_again():
    N = 9000
    sus = make_single(N // 2, 300.0, 1)
    shape = dict(ipl=1, jchunk=512, wg=256, wj=4, posmode=1)
    full = P.Simulator(sus.params, [sus.S], precision="fp32c", launch=dict(shape, fused=0))
    s = P.Simulator(sus.params, [sus.S], precision="fp32c", launch=dict(shape, fused=3))
    s.set_launch(**shape, fused=0)
    small = P.binding.ad_workspace_size(s.ctx)
    assert small < P.binding.ad_workspace_size(full.ctx)
    s.ws = full.ws.new_empty(full.ws.numel())
    P.binding.ad_bind_workspace(s.ctx, s.ws)
    assert P.binding.ad_workspace_size(s.ctx) == P.binding.ad_workspace_size(full.ctx)
    out = []
    for x in (s, full):
        x.set_state(sus.X, sus.phi)
        x.step(2)
        out.append(x.get_state()[0].cpu().numpy())
    assert np.array_equal(*out)
