"""The allocation-free backward close to its limit: the fields fit, by less than
the gradients' block partials (one FP64 value per parameter and block of the x
launch) take."""
import numpy as np
import pytest
import torch

from paper_2003_13569_amd import sfrde as C
from tests.gpu_util import plan_for
from tests.test_gpu_parity import FHN, _wl

pytestmark = pytest.mark.gpu


def test_partials_do_not_count_against_the_fields():
    # 5 + 9 K fields, FP64 accumulator (two fields) and derivative tables (six) of
    # 2 x 70 x 95 x 63 FP32 values: 134.05 of the 134.22 MB
    K = 3
    wl = _wl("fhn-limit", "neumann", (70, 95, 63), "fhn", FHN, (1.5, 1.5), (1e-2, 1e-3), 0.1,
             "fhn_noise", (0.0, 2.5))
    p = plan_for(wl, "f32")
    u0 = 0.5 + 0.05 * np.random.default_rng(8).standard_normal((2,) + wl.shape)
    u = torch.tensor(u0, dtype=torch.float32, device="cuda")
    ckpt = p.integrate(u, K, 0.0, ckpt_every=K)
    g = torch.tensor(np.random.default_rng(9).standard_normal(u0.shape), dtype=torch.float32,
                     device="cuda")
    out = []
    for fn in (C.sfrde_backward_noalloc, C.sfrde_backward):
        gu0 = torch.full_like(g, float("nan"))
        res = fn(p.handle, ckpt.data_ptr(), K, K, 0.0, g.data_ptr(), gu0.data_ptr(), p.S,
                 p.nparams, True, True, True, 1)
        torch.cuda.synchronize()
        out.append([gu0.cpu().numpy()] + [np.array(r) for r in res])
    for a, b in zip(*out):
        assert np.all(np.isfinite(a)) and np.array_equal(a, b)
    p.close()
