"""GPU parity of the FP64 sweep where the waves of a row form groups (few live blocks: small lmax
or small k) and where many rows send the nodes through in passes, against the oracle (Delta
normwise 1e-10, as for the plain FP64 path; float data 2e-7 of sum |w S j|: half an FP32 ulp of
each source and of delta after each pass)."""
import numpy as np
import pytest

import oracle
from test_gpu_sweep import check, ctx, torch_dev, workload  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves", [2, 4, 7, 8, 12, 16])
@pytest.mark.parametrize("lmax,ntau", [(5, 60), (18, 200), (40, 130), (75, 1000)])
def test_groups(torch_dev, ctx, waves, lmax, ntau, monkeypatch):  # noqa: F811
    """1 to 5 blocks; fewer slots than groups; k from rows with one live block (of x << 1) up to
    rows with all, so that a group's slots may all end below the top block."""
    monkeypatch.setenv("LOS_PROJ_WAVES", str(waves))
    for nsrc, mask in ((1, 0), (3, 2), (4, 0)):
        wl = workload(nsrc, lmax=lmax, nk=6, kmax=2.0 * lmax / 14000, kmin=1e-5, ntau=ntau)
        check(torch_dev, ctx, wl, mask=mask)
        p = np.random.default_rng(1).permutation(wl.ntau)   # live slots scattered
        wl.tau, wl.w_tau = wl.tau[p].copy(), wl.w_tau[p].copy()
        wl.S = np.ascontiguousarray(wl.S[:, :, p])
        check(torch_dev, ctx, wl, mask=mask)


@pytest.mark.parametrize("nsrc,nk,ntau,mask", [(1, 2048, 1217, 0), (3, 1536, 1601, 2), (4, 1024, 2433, 0)])
def test_many_rows_in_passes(torch_dev, ctx, nsrc, nk, ntau, mask):  # noqa: F811
    """The smallest row counts and tau grids that go in passes (the last pass holds few nodes)."""
    check(torch_dev, ctx, workload(nsrc, lmax=30, nk=nk, kmax=0.004, ntau=ntau), mask=mask)


def test_passes_float(torch_dev, ctx):  # noqa: F811
    from paper_2509_25110_amd import los
    wl = workload(3, lmax=30, nk=1536, kmax=0.004, ntau=1700)
    dv = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    S = wl.S.astype(np.float32)
    d = ctx.los_project(wl.lmin, wl.lmax, dv(wl.k), dv(wl.tau), wl.tau0, dv(wl.w_tau), dv(S),
                        prec=los.LOS_FP32)
    ref, A = oracle.project(wl.lmin, wl.lmax, wl.k, wl.tau, wl.tau0, wl.w_tau, wl.S, with_abs=True)
    err = np.abs(d.double().cpu().numpy() - ref) / np.maximum(A.max(axis=0, keepdims=True), 1e-300)
    assert float(np.max(err)) <= 2e-7


@pytest.mark.parametrize("nk,nl,ntau", [(128, 640, 70), (129, 640, 70), (256, 2000, 512), (257, 2000, 130)])
def test_float_route(torch_dev, ctx, nk, nl, ntau, monkeypatch):  # noqa: F811
    """Few long rows of float data go to the matrix cores (the same bits as when these are asked
    for), others through the sweep (not the same bits, 2e-6 of the row's largest value apart)."""
    from paper_2509_25110_amd import los
    wl = workload(2, lmax=nl + 1, nk=nk, kmax=2.0 * nl / 14000, ntau=ntau)
    dv = lambda a: torch_dev.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    S = wl.S.astype(np.float32)
    run = lambda: ctx.los_project(wl.lmin, wl.lmax, dv(wl.k), dv(wl.tau), wl.tau0,  # noqa: E731
                                  dv(wl.w_tau), dv(S), prec=los.LOS_FP32).cpu().numpy()
    got = run()
    monkeypatch.setenv("LOS_MIXED_FUSED", "1")
    mfma = run()
    assert np.array_equal(got, mfma) == (nk in (128, 256))
    scale = np.abs(mfma).max(axis=(0, 1), keepdims=True)
    assert float(np.max(np.abs(got - mfma) / scale)) <= 2e-6
