"""bench.py names the kernel and the precision that los_project really uses for float data: the FP64
sweep for LOS_FP32, the matrix cores for few and long rows, for LOS_BF16X3 and when they are asked
for."""
from types import SimpleNamespace

import pytest

import bench

C3 = SimpleNamespace(name="C3", lmin=2, lmax=5000, nl=4999, nk=8000, ntau=4000)
SWEEP = ("project_fp64_sweep_kernel", "f64 j_l and sums, f32 data")
CORES = ("jseed_kernel + fused_gemm_kernel", "f64 j_l, f32 product")


@pytest.fixture(autouse=True)
def plain_environment(monkeypatch):
    for name in ("LOS_MIXED_FUSED", "LOS_FUSED_SHAPE", "LOS_PROJ_SCHEME"):
        monkeypatch.delenv(name, raising=False)


def test_float_data(monkeypatch):
    assert bench.projection_labels(1, C3)[1:] == SWEEP
    assert bench.projection_labels(2, C3)[1:] == (CORES[0], "f64 j_l, bf16x3 product")
    assert bench.projection_labels(0, C3)[1:] == ("project_fp64_sweep_kernel", "f64")
    monkeypatch.setenv("LOS_MIXED_FUSED", "1")
    assert bench.projection_labels(1, C3)[1:] == CORES


@pytest.mark.parametrize("nl,nk,ntau,cores", [(640, 128, 70, True), (640, 129, 70, False),
                                              (639, 128, 70, False), (2000, 256, 512, True),
                                              (2000, 257, 512, False), (2000, 256, 511, False)])
def test_few_long_rows(nl, nk, ntau, cores):
    wl = SimpleNamespace(name="x", nl=nl, nk=nk, ntau=ntau)
    assert bench.projection_labels(1, wl)[1:] == (CORES if cores else SWEEP)
