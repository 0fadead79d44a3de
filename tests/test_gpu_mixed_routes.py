"""GPU parity of LOS_FP32 projections on both of their routes, against the CPU oracle on the same
float sources: the FP64 sweep on float data, which takes most sizes, and the matrix cores, which
take few and long rows and every size under LOS_MIXED_FUSED=1.  Delta normwise (ntau + 2) 2^-24 on
the matrix cores, as for the mixed path's other tests; 2^-24 a pass and 1e-10 by the sweep."""
import numpy as np
import pytest

import oracle
from paper_2509_25110_amd import inputs
from test_gpu_mixed import SMALL, ctx, eps_for, run_mixed, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


def err_of(torch, ctx, wl):  # noqa: F811
    d, _, S64 = run_mixed(torch, ctx, wl, 1)
    ref, A = oracle.project(wl.lmin, wl.lmax, wl.k, wl.tau, wl.tau0, wl.w_tau, S64, with_abs=True)
    return d, float(np.max(np.abs(d - ref) / np.maximum(np.max(A, axis=0, keepdims=True), 1e-300)))


EDGES = [dict(lmax=2, nk=1, ntau=5), dict(lmax=37, nk=3, ntau=129, lmin=37), dict(lmax=9, nk=4, ntau=64),
         dict(lmax=160, nk=3, ntau=200, lmin=150), dict(lmax=40, nk=2, ntau=31),
         dict(lmax=40, nk=3, ntau=3)]


@pytest.mark.parametrize("cfg", SMALL + EDGES, ids=[str(i) for i in range(len(SMALL + EDGES))])
def test_both_routes(torch_dev, ctx, cfg, monkeypatch):  # noqa: F811
    cfg = dict(cfg)
    lmin = cfg.pop("lmin", 2)
    wl = inputs.small(**dict(dict(kmax=0.05, nsrc=3), **cfg))
    wl.lmin = lmin
    assert err_of(torch_dev, ctx, wl)[1] <= 2.0 ** -24 + 1e-10
    monkeypatch.setenv("LOS_MIXED_FUSED", "1")
    assert err_of(torch_dev, ctx, wl)[1] <= eps_for(1, wl.ntau)


@pytest.mark.parametrize("nk,nl,ntau", [(128, 640, 70), (256, 2000, 512)])
def test_few_long_rows(torch_dev, ctx, nk, nl, ntau, monkeypatch):  # noqa: F811
    """The largest calls that go to the matrix cores by themselves; one row more goes through the
    sweep, and the rows of both differ by no more than the two bounds together."""
    wl = inputs.small(lmax=nl + 1, nk=nk, kmax=2.0 * nl / 14000, ntau=ntau, nsrc=2)
    got, err = err_of(torch_dev, ctx, wl)
    assert err <= eps_for(1, ntau)
    monkeypatch.setenv("LOS_MIXED_FUSED", "1")
    np.testing.assert_array_equal(got, err_of(torch_dev, ctx, wl)[0])
    monkeypatch.delenv("LOS_MIXED_FUSED")
    wl.k = np.append(wl.k, wl.k[-1] * 1.01)
    wl.S = np.concatenate([wl.S, wl.S[:, -1:]], axis=1)
    wl.w_lnk, wl.Pk = np.append(wl.w_lnk, 0.0), np.append(wl.Pk, 0.0)
    more, err = err_of(torch_dev, ctx, wl)
    assert err <= 2.0 ** -24 + 1e-10
    assert not np.array_equal(more[:nk], got)
    _, A = oracle.project(wl.lmin, wl.lmax, wl.k, wl.tau, wl.tau0, wl.w_tau,
                          wl.S.astype(np.float32).astype(np.float64), with_abs=True)
    scale = np.maximum(np.max(A, axis=0, keepdims=True), 1e-300)
    assert float(np.max(np.abs(more[:nk] - got) / scale)) <= eps_for(1, ntau) + 2.0 ** -24 + 1e-10


def test_matrix_cores_by_request_independent_of_the_call(torch_dev, ctx, monkeypatch):  # noqa: F811
    """LOS_MIXED_FUSED=1: a k grid in two calls gives bitwise the rows of one call."""
    import copy
    wl = inputs.small(lmax=700, nk=150, kmax=0.1, ntau=300, nsrc=2)
    monkeypatch.setenv("LOS_MIXED_FUSED", "1")
    whole, _, _ = run_mixed(torch_dev, ctx, wl, 1)
    for lo, hi in ((0, 47), (47, 150)):
        part = copy.copy(wl)
        part.k, part.S = wl.k[lo:hi], wl.S[:, lo:hi]
        part.w_lnk, part.Pk = wl.w_lnk[lo:hi], wl.Pk[lo:hi]
        np.testing.assert_array_equal(run_mixed(torch_dev, ctx, part, 1)[0], whole[lo:hi])
