"""FP32 fields past 96 MB go through their tiles in another order (the sweep) with
the waves of a block in step: grids of odd and even extents whose tile counts
fill no round, against the same plan in FP64, which keeps the usual order. FP32
to 2e-5 of FP64 after one step (and its adjoint's state gradient to 1e-4), the
repository's bounds."""
import pytest
import torch

from paper_2003_13569_amd.torch_api import Plan

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc,shape", [("neumann", (231, 233, 235)), ("dirichlet", (230, 233, 236)),
                                      ("periodic", (226, 241, 234)), ("neumann", (250, 197, 256))],
                         ids=str)
def test_swept_fp32_fields_match_fp64(bc, shape):
    h = [1.0 / (n + {"periodic": 0, "dirichlet": 1, "neumann": -1}[bc]) for n in shape]
    gen = torch.Generator(device="cuda").manual_seed(4)
    u0 = 0.9 + 0.01 * torch.randn((2,) + shape, generator=gen, device="cuda", dtype=torch.float64)
    g = torch.randn((2,) + shape, generator=gen, device="cuda", dtype=torch.float64)
    assert u0.numel() * 4 > 96 << 20
    out = {}
    for dtype, td in (("f64", torch.float64), ("f32", torch.float32)):
        p = Plan(shape, bc, h, (1.8, 1.6), (0.05, 1.0), 0.005, "schnakenberg",
                 (1.0, 0.1305, 0.7695), dtype)
        u, gu = u0.to(td, copy=True), g.to(td)
        g0 = torch.empty_like(u)
        ckpt = p.integrate(u, 1, 0.0, ckpt_every=1)
        p.backward(ckpt, 1, 1, gu, 0.0, g0)
        torch.cuda.synchronize()
        out[dtype] = (u.double(), g0.double())
        p.close()
    for (a, b, tol) in zip(out["f32"], out["f64"], (2e-5, 1e-4)):
        for s in range(2):
            err = float((a[s] - b[s]).abs().max() / b[s].abs().max())
            assert err <= tol, (s, tol)
