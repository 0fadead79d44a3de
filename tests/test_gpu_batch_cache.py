"""GPU: the batch's tune cache does not apply a choice that was timed on earlier product kernels (lines
whose pipeline name has no version), and keeps the lines it does not use."""
from test_gpu_batch import small_batch, solve, torch_dev  # noqa: F401
import pytest

pytestmark = pytest.mark.gpu


def test_older_choice_not_applied(torch_dev, tmp_path):  # noqa: F811
    from paper_2509_25110_amd import los
    path = str(tmp_path / "tune.txt")
    b = small_batch(n=8, seed=9)
    ctx = los.Context(tune_cache=path)
    plan, S, _ = solve(torch_dev, ctx, b, 2)
    plan.close()
    key = open(path).read().splitlines()[0].rsplit(" ", 1)[0].split(" ")
    old = " ".join([key[0], "fused"] + key[2:]) + " shape=5\n"
    with open(path, "w") as f:
        f.write(old)
    plan, _, _ = solve(torch_dev, ctx, b, 2, S=S)
    shape = plan.los_batch_info()["fused_shape"]
    plan.close()
    ctx.close()
    lines = open(path).read().splitlines(True)
    assert lines[0] == old and len(lines) == 2
    assert shape != 5 and lines[1].endswith("shape=%d\n" % shape)  # 5 is not among the tuned shapes
