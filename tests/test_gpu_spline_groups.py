"""The spline evaluation's groups of 8 rows (taken from 1024 workgroups on) with a remainder of 3
rows, one and two columns per access, both output precisions, against the oracle
(oracle/spline_oracle.py); bound as for the evaluation's other tests: 1e-14 of the column's
max(|y|, h^2 |M|), and half a unit of a float result."""
import numpy as np
import pytest

from oracle import spline_oracle as so
from test_gpu_spline import ctx, dev, knots, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ntau", [3, 4])
@pytest.mark.parametrize("out_prec", [0, 1])
def test_groups_of_eight(torch_dev, ctx, ntau, out_prec):  # noqa: F811
    rng = np.random.default_rng(77)
    N, nk = 30, 8195
    q = knots(rng, N)
    k = np.sort(np.concatenate([rng.uniform(q[0], q[-1], nk - N), q]))
    Sc = rng.normal(size=(2, N, ntau))
    M = so.second_derivatives(q, Sc)
    out = ctx.los_interp_sources(dev(torch_dev, q), dev(torch_dev, Sc), dev(torch_dev, M),
                                 dev(torch_dev, k), out_prec)
    ref = so.evaluate(q, Sc, M, k)
    h2 = np.max(np.diff(q)) ** 2
    scale = np.maximum(np.abs(Sc).max(axis=1), h2 * np.abs(M).max(axis=1))[:, None, :]
    tol = 1e-14 * scale + (2.0 ** -24 * np.abs(ref) if out_prec == 1 else 0.0)
    assert np.all(np.abs(out.double().cpu().numpy() - ref) <= tol)
