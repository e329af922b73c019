"""1D plans: their second axis has one point and no transform. Steps and
gradients against the oracle, and what has to pass the second axis unchanged in
FP32."""
import numpy as np
import pytest

from oracle import problem
from tests.gpu_util import run
from tests.test_gpu_adjoint import M, _gpu_grads, _rel
from tests.test_gpu_parity import FHN, GS, _wl

pytestmark = pytest.mark.gpu

CASES = [
    _wl("fhn1d-neu", "neumann", (65,), "fhn", FHN, (1.5, 1.7), (1e-2, 1e-3), 0.1, "fhn_noise",
        (0.0, 2.5)),
    _wl("gs1d-per", "periodic", (512,), "gray_scott", GS, (1.7, 1.7), (2e-4, 1e-4), 0.5,
        "gs_square", (-1.0, 1.0)),
    _wl("lin1d-dir", "dirichlet", (2,), "linear", (0.25, -0.5, -1.0), (1.6, 1.8, 1.2),
        (1e-3, 2e-3, 5e-4), 0.5, "normal", (0.0, 1.0)),
    _wl("lin1d-neu", "neumann", (700,), "linear", (0.25,), (1.6,), (1e-3,), 0.5, "normal",
        (0.0, 1.0)),
]


def _field(wl, seed):
    return 0.5 + 0.1 * np.random.default_rng(seed).standard_normal((len(wl.alpha),) + wl.shape)


@pytest.mark.parametrize("scheme", ["p13", "exp"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("wl", CASES, ids=[c.name for c in CASES])
def test_1d_step_and_adjoint_match_oracle(wl, dtype, scheme):
    wl = wl.replace(scheme=scheme)
    u0, wbar = _field(wl, 3), _field(wl, 4)
    got = _gpu_grads(wl, u0, wbar, dtype)
    ref = problem.gradients(wl, u0, M, wbar, periodic_basis="hartley")
    assert problem.rel_err(got["uT"], ref["uT"]) <= {"f64": 1e-10, "f32": 2e-5}[dtype]
    state, par = (1e-10, 1e-10) if dtype == "f64" else (1e-4, 1e-3)
    assert _rel(got["u0"], ref["u0"]) <= state
    for key in ("kappa", "alpha", "params"):
        assert _rel(got[key], ref[key]) <= par, (key, got[key], ref[key])


@pytest.mark.parametrize("n", [256, 512, 1024])
@pytest.mark.parametrize("value", [0.7, 1.0 / 3.0, -1.9999999, 3.1415927])
def test_the_one_point_axis_keeps_every_bit_in_fp32(value, n):
    """A constant field on a periodic axis of a power of two points: the x transform
    only adds equal values and multiplies by powers of two, so with kappa = 0 and
    f = 0 the field comes back bit for bit if the second axis changes nothing."""
    wl = _wl("const1d", "periodic", (n,), "linear", (0.0,), (1.5,), (0.0,), 0.5, "normal",
             (0.0, 1.0))
    u0 = np.full((1, n), float(np.float32(value)))
    assert np.array_equal(run(wl, u0, 3, "f32"), u0)
