"""AD_FP64 ensembles of thousands of small systems and a larger one, whose size
decides between a thread per target and blocks of targets: bit for bit the
oracle's run of the systems on their own."""
import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params, make_single

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tensor", ["oseen", "rpy"])
@pytest.mark.parametrize("small,large", [(1, 8), (1, 9), (3, 17), (3, 40), (8, 32), (8, 33), (2, 500)])
def test_one_larger_system_bitwise(oracle, small, large, tensor):
    W = 4095
    sizes = [small] * 2000 + [large] + [small] * (W - 2000)
    a = [make_single(small, 12.0 * small ** (1 / 3) + 20.0, 70 + b) for b in range(5)]
    big = make_single(large, 12.0 * large ** (1 / 3) + 20.0, 80)
    ens = [a[b % 5] for b in range(2000)] + [big] + [a[b % 5] for b in range(W - 2000)]
    X, phi = np.concatenate([e.X for e in ens]), np.concatenate([e.phi for e in ens])
    s = P.Simulator(Params(), sizes, precision="fp64", tensor=tensor)
    s.set_state(X, phi)
    s.step(2)
    got = s.get_state()[0].cpu().numpy()
    assert s.check() == 0
    off = np.concatenate([[0], np.cumsum(2 * np.asarray(sizes))])
    for b in (0, 1999, 2000, 2001, W):
        want = oracle.run(Params(), ens[b].X, ens[b].phi, 2, tensor=int(tensor == "rpy"))[0]
        assert np.array_equal(got[off[b]:off[b + 1]], want), b
