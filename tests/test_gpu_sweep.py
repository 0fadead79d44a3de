"""GPU parity of the FP64 sweep where its split of the work can go wrong, against the
oracle (Delta normwise 1e-10, as for the plain FP64 path): every count of waves that share
a k row (fewer and more than a row has blocks or slots), tau nodes in any order (the waves
follow each other through the nodes slot by slot), tau grids that go in two passes, and
non-finite sources at nodes that carry no weight."""
import numpy as np
import pytest

import oracle
import test_gpu_tensor as tensor
from paper_2509_25110_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.fixture(scope="module")
def ctx(torch_dev):
    from paper_2509_25110_amd import los
    c = los.Context()
    yield c
    c.close()


def workload(nsrc, **kw):
    wl = inputs.small(nsrc=min(nsrc, 3), **kw)
    if nsrc == 4:
        rng = np.random.default_rng(3)
        wl.S = np.concatenate([wl.S, rng.normal(size=(1, wl.nk, wl.ntau)) * wl.S[:1]], axis=0)
    return wl


def check(torch, ctx, wl, mask=0, S=None):
    dv = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    d = ctx.los_project_kernels(wl.lmin, wl.lmax, dv(wl.k), dv(wl.tau), wl.tau0, dv(wl.w_tau),
                                dv(wl.S if S is None else S), mask)
    torch.cuda.synchronize()
    ref, A = oracle.project(wl.lmin, wl.lmax, wl.k, wl.tau, wl.tau0, wl.w_tau, wl.S, with_abs=True,
                            eps_mask=mask)
    err = np.abs(d.cpu().numpy() - ref) / np.maximum(A.max(axis=0, keepdims=True), 1e-300)
    assert float(np.max(err)) <= 1e-10


@pytest.mark.parametrize("nsrc", [1, 2, 3, 4])
@pytest.mark.parametrize("waves", [1, 2, 3, 5, 8, 12, 16])
def test_waves_sharing_a_row(torch_dev, ctx, waves, nsrc, monkeypatch):
    monkeypatch.setenv("LOS_PROJ_WAVES", str(waves))
    check(torch_dev, ctx, workload(nsrc, lmax=190, nk=5, kmax=0.03, ntau=333))
    check(torch_dev, ctx, workload(nsrc, lmax=20, nk=4, kmax=0.03, ntau=70))   # 2 blocks, 2 slots


@pytest.mark.parametrize("order", ["reversed", "shuffled"])
def test_nodes_in_any_order(torch_dev, ctx, order):
    wl = workload(3, lmax=260, nk=5, kmax=0.06, ntau=900)
    p = np.arange(wl.ntau)[::-1] if order == "reversed" else np.random.default_rng(5).permutation(wl.ntau)
    wl.tau, wl.w_tau = wl.tau[p].copy(), wl.w_tau[p].copy()
    wl.S = np.ascontiguousarray(wl.S[:, :, p])
    check(torch_dev, ctx, wl)
    check(torch_dev, ctx, wl, mask=2)


@pytest.mark.parametrize("ntau", [5500, 8192])
def test_nodes_in_two_passes(torch_dev, ctx, ntau):
    check(torch_dev, ctx, workload(4, lmax=120, nk=3, kmax=0.02, ntau=ntau))
    check(torch_dev, ctx, workload(3, lmax=70, nk=3, kmax=0.02, ntau=ntau), mask=3)  # x = 0 node last
    wl = inputs.tensor_workload(lmax=60, nk=3, kmax=0.02, ntau=ntau)
    got, _ = tensor.run_tensor(torch_dev, ctx, wl, cl=False)
    ref, A = oracle.project_tensor(wl.lmin, wl.lmax, wl.k, wl.tau, wl.tau0, wl.w_tau, wl.S,
                                   with_abs=True)
    assert tensor.normwise_err(got, ref, A, *tensor.gpu_term_scale(wl)) <= 1e-10


def test_nonfinite_sources_without_weight(torch_dev, ctx):
    """Nodes of zero weight and the node at tau0 (x = 0) take no part in plain columns, whatever
    their sources hold."""
    wl = workload(3, lmax=150, nk=4, kmax=0.04, ntau=400)
    wl.w_tau = wl.w_tau.copy()
    wl.w_tau[[3, 70, 200]] = 0.0
    S = wl.S.copy()
    S[:, :, 3], S[:, :, 70], S[:, :, 200], S[:, :, -1] = np.nan, np.inf, -np.inf, np.nan
    check(torch_dev, ctx, wl, S=S)


@pytest.mark.parametrize("ls", [
    [2, 3],                                   # first rows of the lowest block
    [17, 18, 33, 49],                         # the ends of blocks
    [5, 9, 11, 17, 21, 22, 23, 24, 25, 90],   # 3 in one block, 5 (the dense walk) in the next
    [2, 5, 7, 8] + list(range(40, 120)),      # sparse and dense blocks
    [119],
])
@pytest.mark.parametrize("mask", [0, 2])
def test_sampled_rows_of_a_block(torch_dev, ctx, ls, mask):
    """Blocks with 0, 1, 2..4 and more sampled rows, plain and E-mode (whose x -> 0 limit goes
    to l = 2)."""
    torch = torch_dev
    dv = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    for nsrc in (2, 3, 4):
        wl = workload(nsrc, lmax=119, nk=4, kmax=0.05, ntau=200)
        d = ctx.los_project_lsample(wl.lmin, wl.lmax, ls, dv(wl.k), dv(wl.tau), wl.tau0,
                                    dv(wl.w_tau), dv(wl.S), kernel_mask=mask)
        torch.cuda.synchronize()
        ref, A = oracle.project(wl.lmin, wl.lmax, wl.k, wl.tau, wl.tau0, wl.w_tau, wl.S,
                                with_abs=True, eps_mask=mask)
        sel = np.asarray(ls) - wl.lmin
        scale = np.maximum(A.max(axis=0, keepdims=True), 1e-300)[:, sel]
        assert float(np.max(np.abs(d.cpu().numpy() - ref[:, sel]) / scale)) <= 1e-10
