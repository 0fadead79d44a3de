"""GPU: more k rows than one launch of the FP64 sweep can hold (a launch counts its threads in 32
bits: 2^24 rows of 4 waves).  j_2 in closed form at x = 20 .. 80, where its terms do not cancel;
bound 1e-10 of sum |w S|, as for the plain FP64 path's Delta (|j_2| <= 1)."""
import numpy as np
import pytest

from test_gpu_sweep import ctx, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [0, 1], ids=["fp64", "fp32"])
def test_rows_beyond_one_launch(torch_dev, ctx, prec):  # noqa: F811
    torch = torch_dev
    nk, tau0 = (1 << 24) + 3, 14000.0
    f64 = dict(dtype=torch.float64, device="cuda")
    k = torch.linspace(0.01, 0.02, nk, **f64)
    tau, w = torch.tensor([10000.0, 12000.0], **f64), torch.tensor([1.0, 0.5], **f64)
    S = torch.ones(1, nk, 2, **f64)
    S[0, :, 1] = torch.arange(nk, **f64) / nk
    if prec:
        S = S.float()
    d = ctx.los_project(2, 2, k, tau, tau0, w, S, prec=prec)[:, 0, 0].double()
    ref = torch.zeros(nk, **f64)
    for n in range(2):
        x = k * (tau0 - tau[n])
        ref += w[n] * S[0, :, n].double() * ((3 / x ** 3 - 1 / x) * torch.sin(x) - 3 / x ** 2 * torch.cos(x))
    # FP32: delta is rounded once, half an ulp of |delta| <= 0.1
    bound = 1.5e-10 + (2.0 ** -24 * 0.1 if prec else 0.0)
    assert float((d - ref).abs().max()) <= bound
    assert np.isfinite(float(d.sum()))
