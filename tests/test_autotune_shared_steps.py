"""The autotuner where a step does not depend on the pair kernel's shape: such
shapes share one step time and are ranked by their products (no GPU needed)."""
from dataclasses import replace

import numpy as np
import torch

from paper_1004_1932_amd import autotune as A
from paper_1004_1932_amd import binding as B
from workload import Params

HILO, SINGLE = B.AD_POS_HILO, B.AD_POS_SINGLE


def test_which_steps_ignore_the_shape():
    p, st = Params(), replace(Params(), steric_k=100.0)
    f = A.step_ignores_shape
    assert f(p, [4352], dict(posmode=HILO)) and f(p, [6656], dict(posmode=SINGLE, fused=0))
    assert not f(p, [4351], dict(posmode=HILO)) and not f(p, [6655], dict(posmode=SINGLE))
    assert f(st, [4352], dict(posmode=SINGLE)) and not f(st, [4351], dict(posmode=HILO))
    assert not f(p, [20000], dict(posmode=HILO, fused=3)) and not f(p, [20000, 3], dict(posmode=HILO))
    assert not f(p, [1 << 19], dict(posmode=HILO))


class Fake:
    """A simulator whose steps and products are exact."""
    device = "cpu"

    def __init__(self, params, S, precision="fp32c", graph=False):
        self.n, self.launch = 2 * int(np.sum(S)), dict(posmode=HILO, fused=0)

    def set_launch(self, **kw):
        self.launch = dict(kw, fused=kw.get("fused", 0))

    def set_state(self, X, phi):
        self.X = torch.as_tensor(np.asarray(X))

    def get_state(self):
        return self.X + 1.0, 0.0, 0

    def forces(self, X, t):
        return torch.ones_like(X)

    def mobility(self, X, F):
        return torch.ones_like(X)

    def step(self, n):
        pass

    def close(self):
        pass


def test_products_decide_between_shapes_of_one_step(monkeypatch):
    """The step timings of equal kernels differ by noise (here: fall with every
    measurement); the pick must not."""
    steps = []

    def step_time(sim, n):
        steps.append(dict(sim.launch))
        return 2.0 / (1 + len(steps))

    monkeypatch.setattr(A.B, "Simulator", Fake)
    monkeypatch.setattr(A, "_step_time", step_time)
    monkeypatch.setattr(A, "_product_time", lambda sim, X, F, n: {1: 3.0, 2: 1.0, 4: 2.0}[sim.launch["ipl"]])
    cands = [dict(ipl=i, wg=256, wj=4, jchunk=512, posmode=HILO) for i in (1, 2, 4)]
    S = 5000
    X = np.random.default_rng(0).uniform(0, 9, (2 * S, 3))
    r = A.tune(Params(), [S], X, np.zeros(S), cands=cands, steps=3)
    assert r["launch"]["ipl"] == 2 and len(steps) == 1
    # below the kernel's sizes the step times decide
    steps.clear()
    r = A.tune(Params(), [1000], X[:2000], np.zeros(1000), cands=cands, steps=3)
    assert r["launch"]["ipl"] == 4 and len(steps) == 3
