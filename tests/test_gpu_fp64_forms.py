"""The FP64 pair sums at the edges of their forms: the short correctly rounded
quotients and the plain expressions they give way to, the work-group shapes of
AD_FP64, and AD_FP64_TILED's groups of targets and sources."""
import numpy as np
import pytest

import paper_1004_1932_amd as P
from workload import Params, make_single

pytestmark = pytest.mark.gpu


def _system(S, seed=0):
    return make_single(S, 12.0 * S ** (1 / 3) + 20.0, seed).X


@pytest.mark.parametrize("tensor", ["oseen", "rpy"])
@pytest.mark.parametrize("S", [33, 64, 65, 768, 769, 1280, 1281, 1536, 1537])
def test_fp64_product_block_shapes_bitwise(oracle, S, tensor):
    """One dumbbell either side of the sizes where targets, producers and
    chunk length change."""
    X = _system(S)
    F = np.random.default_rng(S).standard_normal(X.shape)
    u = P.Simulator(Params(), [S], precision="fp64", tensor=tensor).mobility(X, F).cpu().numpy()
    assert np.array_equal(u, oracle.mobility(Params(), X, F, int(tensor == "rpy")))


@pytest.mark.parametrize("tensor", ["oseen", "rpy"])
@pytest.mark.parametrize("case", ["zero forces", "one force", "tiny forces", "large forces", "all-ones", "scaled down",
                                  "scaled up", "mixed"])
def test_fp64_product_operand_ranges_bitwise(oracle, case, tensor):
    """Operands in and out of the short forms' range: r2 beyond 2^+-400, r.F
    beyond 2^+-500 and zero, distances whose square (or its root) has an
    all-ones significand."""
    S = 70
    X = _system(S, 2)
    F = np.random.default_rng(1).standard_normal(X.shape)
    if case == "zero forces":
        F[:] = 0.0
    elif case == "one force":
        F[:], F[3] = 0.0, [0.0, 1.0, 0.0]
    elif case == "tiny forces":
        F *= 1e-200
    elif case == "large forces":
        F *= 1e200
    elif case == "all-ones":
        one = np.nextafter(2.0, 0.0)                     # significand of ones
        root = np.sqrt(np.nextafter(4.0, 0.0))           # its square rounds to all ones
        X[:] = 0.0
        X[:, 0] = 64.0 * np.arange(2 * S)
        X[1::2, 0] = X[0::2, 0] + one
        X[0], X[1], X[2] = [0, 0, 0], [one, 0, 0], [0, root, 0]
    elif case == "scaled down":
        X *= 2.0 ** -230
    elif case == "scaled up":
        X *= 2.0 ** 230
    else:
        F[::3] *= 1e-170
        X[5] = X[4] + 2.0 ** -230
    u = P.Simulator(Params(), [S], precision="fp64", tensor=tensor).mobility(X, F).cpu().numpy()
    o = oracle.mobility(Params(), X, F, int(tensor == "rpy"), allow_nonfinite=True)
    assert np.array_equal(u, o, equal_nan=True)


@pytest.mark.parametrize("integrator", ["rk4", "heun"])
@pytest.mark.parametrize("sizes", [[33], [800], [1300], [40, 1, 700, 65]])
def test_fp64_stage_closed_by_the_pair_kernel_bitwise(oracle, sizes, integrator):
    """The stage update, next forces and pack in the pair kernel's consumer
    wave, replayed from graphs and launched directly."""
    ens = [make_single(S, 12.0 * S ** (1 / 3) + 20.0, 7 + b) for b, S in enumerate(sizes)]
    X, phi = np.concatenate([e.X for e in ens]), np.concatenate([e.phi for e in ens])
    out = []
    for graph in (False, True):
        s = P.Simulator(Params(), sizes, precision="fp64", integrator=integrator, graph=graph)
        s.set_state(X, phi)
        for n in (1, 5, 17):
            s.step(n)
        out.append(s.get_state()[0].cpu().numpy())
        assert s.check() == 0
    Xo = oracle.run(Params(), X, phi, 23, S_per_sys=sizes, integrator=int(integrator == "heun"))[0]
    assert np.array_equal(out[0], Xo) and np.array_equal(out[1], Xo)


@pytest.mark.parametrize("tensor", ["oseen", "rpy"])
@pytest.mark.parametrize("launch", [None, dict(ipl=1, wg=64, jchunk=64), dict(ipl=2, wg=64, jchunk=100),
                                    dict(ipl=2, wg=256, jchunk=300)])
@pytest.mark.parametrize("sizes", [[1], [31], [32], [33], [127], [130], [257], [5, 66, 1, 129]])
def test_fp64_tiled_groups_of_targets_and_sources(oracle, sizes, launch, tensor):
    """Part-filled target groups, tiles and waves. 1e-13: sums of n terms,
    each within a few ulp, in another order (n <= 514)."""
    X = np.concatenate([_system(S, 3 + b) for b, S in enumerate(sizes)])
    F = np.random.default_rng(9).standard_normal(X.shape)
    s = P.Simulator(Params(), sizes, precision="fp64_tiled", launch=launch, tensor=tensor)
    u = s.mobility(X, F).cpu().numpy()
    off = np.concatenate([[0], np.cumsum(2 * np.asarray(sizes))])
    for b in range(len(sizes)):
        sl = slice(off[b], off[b + 1])
        o = oracle.mobility(Params(), X[sl], F[sl], int(tensor == "rpy"))
        assert np.linalg.norm(u[sl] - o) <= 1e-13 * np.linalg.norm(o), b


@pytest.mark.parametrize("scale", [2.0 ** -230, 1.0, 2.0 ** 230])
def test_fp64_tiled_operand_ranges(oracle, scale):
    X = _system(70, 2) * scale
    F = np.random.default_rng(1).standard_normal(X.shape)
    F[7] = 0.0
    u = P.Simulator(Params(), [70], precision="fp64_tiled").mobility(X, F).cpu().numpy()
    o = oracle.mobility(Params(), X, F)
    assert np.linalg.norm(u - o) <= 1e-13 * np.linalg.norm(o)


@pytest.mark.parametrize("precision", ["fp64", "fp64_tiled"])
def test_fp64_coincident_spheres_flagged_and_skipped(oracle, precision):
    X = _system(90, 4)
    X[101] = X[12]
    F = np.random.default_rng(1).standard_normal(X.shape)
    s = P.Simulator(Params(), [90], precision=precision)
    s.set_state(X, np.zeros(90))
    u = s.mobility(X, F).cpu().numpy()
    assert s.check() == P.binding.AD_ENONFINITE
    o = oracle.mobility(Params(), X, F, allow_nonfinite=True)
    assert np.linalg.norm(u - o) <= 1e-13 * np.linalg.norm(o)


@pytest.mark.parametrize("tensor", ["oseen", "rpy"])
@pytest.mark.parametrize("precision", ["fp64", "fp64_tiled"])
@pytest.mark.parametrize("W,S", [(1300, 1), (160, 9), (21, 127), (21, 129), (10, 300), (4095, 1), (4096, 1), (4100, 2)])
def test_ensembles_of_small_systems(oracle, W, S, precision, tensor):
    """The block shape of small systems, and a thread per target from 4096
    systems on: two steps, some systems against the oracle's run."""
    rng = np.random.default_rng(W)
    ens = [make_single(S, 12.0 * S ** (1 / 3) + 20.0, 40 + b) for b in range(min(W, 7))]
    X = np.concatenate([ens[b % len(ens)].X for b in range(W)])
    phi = rng.uniform(0.0, 6.0, W * S)
    s = P.Simulator(Params(), [S] * W, precision=precision, tensor=tensor)
    s.set_state(X, phi)
    s.step(2)
    got = s.get_state()[0].cpu().numpy()
    assert s.check() == 0
    for b in {0, 1, W // 2, W - 1}:
        x, p = slice(2 * S * b, 2 * S * (b + 1)), slice(S * b, S * (b + 1))
        want = oracle.run(Params(), X[x], phi[p], 2, tensor=int(tensor == "rpy"))[0]
        if precision == "fp64":
            assert np.array_equal(got[x], want)
        else:
            # sums of at most 600 terms in another order, of a displacement
            assert np.abs(got[x] - want).max() <= 1e-12 * np.abs(want - X[x]).max() + 1e-14 * np.abs(X[x]).max()
