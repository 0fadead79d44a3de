"""GPU parity, against the oracle, of what the FP64 sweep does in passes over the tau nodes besides
the plain columns: sampled multipoles (Delta normwise 1e-10, plain and E-mode, whose x -> 0 limit
comes in the last pass) and float data, whose delta is rounded to float after each pass (3 passes
with sources that change sign from pass to pass: 3 half units of sum |w S j|, and 1e-10)."""
import numpy as np
import pytest

import oracle
from test_gpu_sweep import ctx, torch_dev, workload  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ls", [[2, 3, 40, 41, 42, 43, 44, 90, 119], list(range(2, 120, 3)), [119]])
@pytest.mark.parametrize("mask", [0, 2, 5])
def test_sampled(torch_dev, ctx, ls, mask):  # noqa: F811
    dv = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    wl = workload(3, lmax=119, nk=1536, kmax=0.02, ntau=1700)
    d = ctx.los_project_lsample(wl.lmin, wl.lmax, ls, dv(wl.k), dv(wl.tau), wl.tau0, dv(wl.w_tau),
                                dv(wl.S), kernel_mask=mask).cpu().numpy()
    ref, A = oracle.project(wl.lmin, wl.lmax, wl.k, wl.tau, wl.tau0, wl.w_tau, wl.S, with_abs=True,
                            eps_mask=mask)
    sel = np.asarray(ls) - wl.lmin
    scale = np.maximum(A.max(axis=0, keepdims=True), 1e-300)[:, sel]
    assert float(np.max(np.abs(d - ref[:, sel]) / scale)) <= 1e-10


def test_float_passes_that_cancel(torch_dev, ctx):  # noqa: F811
    from paper_2509_25110_amd import los
    dv = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    wl = workload(3, lmax=60, nk=1536, kmax=0.006, ntau=3300)
    S = wl.S.astype(np.float32)
    S[:, :, 1100:2200] *= -1.9
    d = ctx.los_project(wl.lmin, wl.lmax, dv(wl.k), dv(wl.tau), wl.tau0, dv(wl.w_tau), dv(S),
                        prec=los.LOS_FP32).double().cpu().numpy()
    ref, A = oracle.project(wl.lmin, wl.lmax, wl.k, wl.tau, wl.tau0, wl.w_tau,
                            S.astype(np.float64), with_abs=True)
    err = np.abs(d - ref) / np.maximum(A.max(axis=0, keepdims=True), 1e-300)
    assert float(np.max(err)) <= 3 * 2.0 ** -24 + 1e-10
