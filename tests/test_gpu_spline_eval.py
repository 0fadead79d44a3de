"""The spline evaluation's search of the knot interval (64 knots at a time: one, two and three
rounds), groups of 8 rows with remainders, and one or two columns per access (odd and even tau
counts, arrays at an odd element), against the oracle (oracle/spline_oracle.py).  Wavenumbers
below, on and above the knots.  Bound as for the evaluation's other test: 1e-14 of the column's
max(|y|, h^2 |M|)."""
import numpy as np
import pytest

from oracle import spline_oracle as so
from test_gpu_spline import ctx, dev, knots, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,nk,ntau,odd", [(2, 1, 1, 0), (3, 7, 2, 0), (64, 8, 255, 0), (65, 9, 256, 1),
                                           (66, 17, 512, 0), (4097, 40, 514, 0), (4200, 33, 3, 0)])
@pytest.mark.parametrize("out_prec", [0, 1])
def test_interval_and_edges(torch_dev, ctx, N, nk, ntau, odd, out_prec):  # noqa: F811
    rng = np.random.default_rng(N + nk)
    q = knots(rng, N)
    k = np.sort(np.concatenate([rng.uniform(q[0], q[-1], max(0, nk - 4)), q[rng.integers(0, N, 4)]]))[:nk]
    Sc = rng.normal(size=(2, N, ntau))
    M = so.second_derivatives(q, Sc)

    def put(a):  # an array whose first element is at an odd place of its buffer
        a = np.ascontiguousarray(a)
        if not odd:
            return dev(torch_dev, a)
        return dev(torch_dev, np.concatenate([[0.0], a.ravel()]))[1:].view(a.shape)

    out = ctx.los_interp_sources(dev(torch_dev, q), put(Sc), put(M), dev(torch_dev, k), out_prec)
    got = out.double().cpu().numpy()
    ref = so.evaluate(q, Sc, M, k)
    h2 = np.max(np.diff(q)) ** 2
    scale = np.maximum(np.abs(Sc).max(axis=1), h2 * np.abs(M).max(axis=1))[:, None, :]
    tol = 1e-14 * scale + (2.0 ** -24 * np.abs(ref) if out_prec == 1 else 0.0)
    assert np.all(np.abs(got - ref) <= tol)
