"""Species of very different size on the FFT axes, each species held to the
repository's bounds of its own: forward FP64 1e-10 and FP32 2e-5, state
gradients FP64 1e-10 and FP32 1e-4, kappa and alpha gradients FP64 1e-10 and
FP32 1e-3. (Real lines are transformed in pairs, as the two parts of a complex
line, and the rounding errors of each are of the size of the larger.)

Odd line counts leave a line without a partner, on x axes and on strided ones;
the reaction couples two species or (linear) none."""
import numpy as np
import pytest

from oracle import problem
from tests.gpu_util import run
from tests.test_gpu_adjoint import M, _gpu_grads, _rel
from tests.test_gpu_parity import _wl

pytestmark = pytest.mark.gpu

SMALL = {"f64": 1e-8, "f32": 1e-6}
SHAPES = [(41, 256), (256, 41), (6, 512), (512, 7), (3, 1024), (1024, 5), (5, 256, 7), (9, 6, 512),
          (256, 3, 5)]


def _fhn(shape, eps):
    # v starts at eps and is fed by eps beta u: it stays there
    return _wl("fhn-small-" + "x".join(map(str, shape)), "periodic", shape, "fhn",
               (0.1, 0.1 * eps, 0.5, 1.0, 0.0), (1.5, 1.7), (1e-3, 1e-4), 0.1, "fhn_noise", (0.0, 2.5))


def _lin(shape, S):
    return _wl("lin%d-small-%s" % (S, "x".join(map(str, shape))), "periodic", shape, "linear",
               (0.25, -0.5, -1.0)[:S], (1.6, 1.8, 1.2)[:S], (1e-3, 2e-3, 5e-4)[:S], 0.5, "normal",
               (0.0, 1.0))


def _fields(wl, eps, seed):
    u = np.random.default_rng(seed).standard_normal((len(wl.alpha),) + wl.shape)
    u[1] *= eps
    return u


def _ids(v):
    return v.name if hasattr(v, "name") else None


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_small_coupled_species_matches_oracle(shape, dtype):
    eps = SMALL[dtype]
    wl = _fhn(shape, eps)
    u0 = 0.1 * _fields(wl, eps, 5) + np.array([0.5, eps]).reshape((2,) + (1,) * len(shape))
    ref = problem.run(wl, u0, 3, periodic_basis="hartley")
    assert problem.rel_err(run(wl, u0, 3, dtype), ref) <= {"f64": 1e-10, "f32": 2e-5}[dtype]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("S", [2, 3])
@pytest.mark.parametrize("shape", SHAPES[:4] + SHAPES[6:7], ids=str)
def test_small_uncoupled_species_and_its_adjoint_match_oracle(shape, S, dtype):
    eps = SMALL[dtype]
    wl = _lin(shape, S)
    u0, wbar = _fields(wl, eps, 6), _fields(wl, eps, 7)
    got = _gpu_grads(wl, u0, wbar, dtype)
    ref = problem.gradients(wl, u0, M, wbar, periodic_basis="hartley")
    assert problem.rel_err(got["uT"], ref["uT"]) <= {"f64": 1e-10, "f32": 2e-5}[dtype]
    state, par = (1e-10, 1e-10) if dtype == "f64" else (1e-4, 1e-3)
    for s in range(S):
        assert _rel(got["u0"][s], ref["u0"][s]) <= state, s
        for key in ("kappa", "alpha", "params"):
            assert _rel(got[key][s], ref[key][s]) <= par, (key, s, got[key], ref[key])
