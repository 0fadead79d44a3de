"""GPU parity of the FP64 sweep at the limits of the rules for few blocks of multipoles, against the
oracle (Delta normwise 1e-10): up to 6 blocks with 2 waves a row, up to 8 with the nodes in passes
from 768 rows on, and one block more."""
import pytest

import oracle
import test_gpu_tensor as tensor
from paper_2509_25110_amd import inputs
from test_gpu_sweep import check, ctx, torch_dev, workload  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nsrc,nl,nk,ntau,mask", [
    (3, 96, 1600, 200, 0), (3, 97, 1600, 200, 0), (4, 96, 1100, 300, 2), (1, 81, 2100, 130, 0),
    (1, 128, 768, 1300, 0), (1, 129, 768, 1300, 0), (1, 128, 767, 1300, 0), (2, 128, 768, 1250, 2),
    (3, 128, 768, 1700, 0), (4, 128, 768, 2450, 4)])
def test_limits(torch_dev, ctx, nsrc, nl, nk, ntau, mask):  # noqa: F811
    check(torch_dev, ctx, workload(nsrc, lmax=nl + 1, nk=nk, kmax=2.0 * nl / 14000, ntau=ntau), mask=mask)


@pytest.mark.parametrize("lmax,nk,ntau", [(96, 1100, 300), (97, 1100, 300), (128, 768, 2450)])
def test_limits_tensor(torch_dev, ctx, lmax, nk, ntau):  # noqa: F811
    wl = inputs.tensor_workload(lmax=lmax, nk=nk, kmax=2.0 * lmax / 14000, ntau=ntau)
    got, _ = tensor.run_tensor(torch_dev, ctx, wl, cl=False)
    ref, A = oracle.project_tensor(wl.lmin, wl.lmax, wl.k, wl.tau, wl.tau0, wl.w_tau, wl.S,
                                   with_abs=True)
    assert tensor.normwise_err(got, ref, A, *tensor.gpu_term_scale(wl)) <= 1e-10
