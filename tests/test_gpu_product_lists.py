"""The matrix-core product where every possible tile is a workgroup (an odd and an even number of
tiles a row, whose order turns with the row), in one chunk of k rows and in several, and where its
tiles are taken from lists (batches with more than two for each workgroup the device holds): Delta
and C_l bitwise those of the table pipeline (the same values, added in the same order)."""
import numpy as np
import pytest

from paper_2509_25110_amd import inputs
from test_gpu_batch import small_batch, solve
from test_gpu_fused_tiles import table
from test_gpu_mixed import ctx, run_mixed, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nk,lmax", [(13, 700), (90, 600), (600, 500)])
@pytest.mark.parametrize("prec", [1, 2], ids=["fp32", "bf16x3"])
def test_projection(torch_dev, ctx, nk, lmax, prec, monkeypatch):  # noqa: F811
    """2 to 6 tiles a row; 9 chunks of nodes, the last ragged; the smallest k end far below l_max
    and their upper tiles are zeros."""
    wl = inputs.small(lmax=lmax, nk=nk, kmax=0.08, kmin=2e-4, ntau=521, nsrc=2)
    monkeypatch.setenv("LOS_MIXED_FUSED", "0")
    base, _, _ = run_mixed(torch_dev, ctx, wl, prec)
    monkeypatch.setenv("LOS_MIXED_FUSED", "1")
    for mib in (4096, 64, 1):  # 1 MiB: 5 to 6 rows a chunk, the last short
        monkeypatch.setenv("LOS_JTAB_MIB", str(mib))
        for shape in (4, 5):
            monkeypatch.setenv("LOS_FUSED_SHAPE", str(shape))
            d, _, _ = run_mixed(torch_dev, ctx, wl, prec)
            np.testing.assert_array_equal(d, base, err_msg="%d MiB, shape %d" % (mib, shape))


@pytest.mark.parametrize("prec", [1, 2], ids=["fp32", "bf16x3"])
def test_batch(torch_dev, ctx, prec, monkeypatch):  # noqa: F811
    b = small_batch(n=3, seed=8, lmax_range=(230, 700), nk_range=(200, 400), master_nk=420,
                    master_kmax=0.1, ntau=130)
    S, base = table(torch_dev, ctx, b, prec, monkeypatch)
    for shape in (0, 1, 3, 7):
        monkeypatch.setenv("LOS_BATCH_SHAPE", str(shape))
        plan, _, cl = solve(torch_dev, ctx, b, prec, S=S)
        plan.close()
        np.testing.assert_array_equal(cl, base, err_msg="shape %d" % shape)
