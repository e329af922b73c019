"""Plans that share kernels: a plan computes the same after another one of the
same axis length and another size was made (the kernels' launch limits hold
for both)."""
import numpy as np
import pytest

import workloads as W
from tests.gpu_util import plan_for, run
from tests.test_gpu_parity import GS, _wl

pytestmark = pytest.mark.gpu


def _gs(shape):
    return _wl("gs-" + "x".join(map(str, shape)), "periodic", shape, "gray_scott", GS, (1.7, 1.7),
               (2e-5, 1e-5), 1.0, "gs_square", (-1.0, 1.0))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n", [256, 512, 1024])
def test_large_fft_plan_runs_after_a_small_one_was_made(n, dtype):
    big, small = _gs((n, 1024)), _gs((4, n))
    u0 = W.initial_fields(big)
    with_plan = plan_for(big, dtype)  # blocks of four wavefronts
    want = run(big, u0, 1, dtype, plan=with_plan)
    other = plan_for(small, dtype)  # of one or two
    got = run(big, u0, 1, dtype, plan=with_plan)
    assert np.array_equal(got, want)
    other.close()
    with_plan.close()
