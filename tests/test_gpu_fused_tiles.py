"""The batch's fused product at the edges of its tiles, chunks and bands, against the table
pipeline (whole FP32 tables, every row written and read): the same values in the same order of
accumulation, so C_l agrees bitwise.  One model to 40 (one to eight column blocks, a second
column tile), node counts around a 64-node chunk and a 4-node piece and below one piece, and
rows whose band ends far below l_max."""
import numpy as np
import pytest

from paper_2509_25110_amd import inputs
from test_gpu_batch import ctx, dev, small_batch, solve, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


def table(torch, ctx, b, prec, monkeypatch, S=None):  # noqa: F811
    monkeypatch.setenv("LOS_BATCH_FUSED", "0")
    monkeypatch.setenv("LOS_BATCH_TILE_MB", "2")
    monkeypatch.setenv("LOS_BATCH_TILE_NC", "4")
    plan, S, cl = solve(torch, ctx, b, prec, S=S)
    assert plan.los_batch_info()["chunks"] == 1
    plan.close()
    monkeypatch.delenv("LOS_BATCH_FUSED")
    return S, cl


@pytest.mark.parametrize("n,ntau,lmax", [(1, 3, 40), (2, 4, 130), (3, 61, 257), (5, 64, 300),
                                         (6, 66, 129), (11, 67, 500), (16, 127, 260),
                                         (21, 129, 400), (40, 1003, 700)])
@pytest.mark.parametrize("prec", [1, 2], ids=["fp32", "bf16x3"])
def test_fused_edges_match_tables(torch_dev, ctx, n, ntau, lmax, prec, monkeypatch):  # noqa: F811
    b = small_batch(n=n, seed=41 + n, lmax_range=(lmax // 3, lmax), nk_range=(20, 60), master_nk=70,
                    master_kmax=2.0 * lmax / 14000, ntau=ntau)
    S, base = table(torch_dev, ctx, b, prec, monkeypatch)
    for shape in (0, 1, 3, 4, 5, 6, 7):
        monkeypatch.setenv("LOS_BATCH_SHAPE", str(shape))
        plan, _, cl = solve(torch_dev, ctx, b, prec, S=S)
        assert plan.los_batch_info()["fused_shape"] == shape
        plan.close()
        np.testing.assert_array_equal(cl, base, err_msg="shape %d" % shape)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_weight_not_finite(torch_dev, ctx, bad, monkeypatch):  # noqa: F811
    """A weight or power that is not finite reaches every multipole of its model, also those above
    the band of its k row, where no Delta is stored: as with whole tables."""
    b = small_batch(n=4, seed=5, lmax_range=(300, 600), nk_range=(40, 60), master_nk=64,
                    master_kmax=0.08, ntau=200)
    b.Pk[int(b.koff[1])] = bad          # the smallest k of model 1
    S, base = table(torch_dev, ctx, b, 1, monkeypatch)
    plan, _, cl = solve(torch_dev, ctx, b, 1, S=S)
    plan.close()
    assert not np.isfinite(cl[1, 0, :int(b.lmax[1]) - 1]).any()
    np.testing.assert_array_equal(cl, base)
