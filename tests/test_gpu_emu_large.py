"""GPU parity of the emulator's kernels past the sizes where their larger tiles set in, ragged, against
the FP64 CPU oracle (oracle/emu_oracle.py): layers and gradients in 64 x 64 tiles (from 512 tiles
on), and the reconstruction with two column tiles a workgroup, the last workgroup with one.  Bounds
as for the emulator's other GPU tests: spectra 2e-4 relative (TE relative to sqrt(TT EE)), estimates
1e-2 relative + 2e-4, gradients normwise 2e-5 of their largest entry."""
import numpy as np
import pytest

from oracle import emu_oracle as eo
from test_gpu_emu import ctx, dev, glorot, make_emu, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nl,ncomp,width", [(1050, 40, 9, 500), (1030, 4100, 12, 64)])
def test_infer(torch_dev, ctx, n, nl, ncomp, width):  # noqa: F811
    rng = np.random.default_rng(61)
    members = 4
    emu = make_emu(ctx, nl=nl, ncomp=ncomp, width=width, depth=2, members=members)
    sizes = eo.layer_sizes(5, width, 2, 4 * ncomp)
    base = glorot(rng, sizes)
    thetas = [(base * (1 + 0.02 * rng.normal(size=base.size))).astype(np.float32)
              for _ in range(members)]
    for e, th in enumerate(thetas):
        emu.emu_set_params(e, th)
    V = rng.normal(size=(4, nl, ncomp)) / np.sqrt(nl)
    mu = rng.normal(size=(4, nl)) * 0.2 - np.array([2.0, 3.0, 0.0, 1.0])[:, None]
    mu[2] = 0.5 + 0.1 * rng.normal(size=nl)
    sigma = np.tile(0.5 / np.arange(1, ncomp + 1), (4, 1))
    t = np.exp(rng.normal(size=nl) * 0.1 - 3)
    emu.emu_set_pca(-np.ones(5), np.ones(5), mu, V, sigma, t)
    q = rng.uniform(-1, 1, size=(n, 5))
    cl, err4, _ = emu.emu_infer_spectra(dev(torch_dev, q), threshold=1e-3)
    cl, err4 = cl.cpu().numpy(), err4.cpu().numpy()
    emu.close()
    assert np.isfinite(cl).all() and np.isfinite(err4).all()
    rows = np.r_[0:18, 31:34, 63:66, 500:520, n - 30:n]  # each row is independent of the others
    cls = []
    for th in thetas:
        out, _, _ = eo.forward(th.astype(np.float64), sizes, q[rows])
        y = np.stack([mu[s] + (out[:, s * ncomp:(s + 1) * ncomp] * sigma[s]) @ V[s].T
                      for s in range(4)], axis=1)
        cls.append(eo.inverse_transform(y, t))
    cls = np.stack(cls)
    mref, _ = eo.ensemble_stats(cls)
    scale = np.abs(mref).copy()
    scale[:, 2] = np.sqrt(mref[:, 0] * mref[:, 1])
    e4 = np.max(np.abs(cls - mref[None]) / scale[None], axis=(0, 3))
    assert np.max(np.abs(cl[rows] - mref) / scale) <= 2e-4
    np.testing.assert_allclose(err4[rows], e4, rtol=1e-2, atol=2e-4)


def test_gradient(torch_dev, ctx):  # noqa: F811
    rng = np.random.default_rng(62)
    n, width, depth, ncomp = 4200, 500, 2, 9
    emu = make_emu(ctx, nl=40, ncomp=ncomp, width=width, depth=depth, members=1)
    sizes = eo.layer_sizes(5, width, depth, 4 * ncomp)
    theta = glorot(rng, sizes)
    emu.emu_set_params(0, theta)
    u = rng.uniform(-1, 1, size=(n, 5)).astype(np.float32)
    z = rng.normal(size=(n, 4 * ncomp)).astype(np.float32)
    loss, grad = emu.emu_loss_grad(0, dev(torch_dev, u), dev(torch_dev, z))
    lref, gref = eo.loss_and_grad(theta.astype(np.float64), sizes, u.astype(np.float64),
                                  z.astype(np.float64))
    assert abs(float(loss.item()) - lref) <= 2e-5 * lref
    assert np.max(np.abs(grad.cpu().numpy() - gref)) <= 2e-5 * np.max(np.abs(gref))
    emu.close()
