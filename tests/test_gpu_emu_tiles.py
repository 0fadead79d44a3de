"""GPU parity of the emulator's kernels at the edges of their tiles, against the FP64 CPU oracle
(oracle/emu_oracle.py): row counts around the 16-, 32- and 64-row tiles, multipole and
coefficient counts that fill no tile and allow no 16-byte loads, 1 to 5 members (5: more than
the fused reconstruction takes), and gradients of layers narrower and wider than a tile.

Bounds as for the emulator's other GPU tests: spectra 2e-4 relative (TE relative to
sqrt(TT EE)), estimates 1e-2 relative + 2e-4, gradients normwise 2e-5 of their largest entry
(FP32 products with FP32 accumulation against FP64)."""
import numpy as np
import pytest

from oracle import emu_oracle as eo
from test_gpu_emu import ctx, dev, glorot, make_emu, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,nl,ncomp,width,members", [
    (1, 40, 8, 64, 1), (15, 33, 7, 50, 2), (16, 129, 9, 33, 3), (17, 127, 12, 64, 4),
    (33, 65, 36, 70, 4), (65, 64, 31, 512, 2), (700, 200, 8, 512, 4), (40, 70, 8, 64, 5),
])
def test_infer_edges(torch_dev, ctx, n, nl, ncomp, width, members):  # noqa: F811
    rng = np.random.default_rng(31)
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
    lo, hi = -np.ones(5), np.ones(5)
    emu.emu_set_pca(lo, hi, mu, V, sigma, t)
    q = rng.uniform(-1, 1, size=(n, 5))
    cl, err4, flag4 = emu.emu_infer_spectra(dev(torch_dev, q), threshold=1e-3)
    cl1, err, flag = emu.emu_infer(dev(torch_dev, q), threshold=1e-3)
    torch_dev.cuda.synchronize()
    cls = []
    for th in thetas:
        out, _, _ = eo.forward(th.astype(np.float64), sizes, q)
        y = np.stack([mu[s] + (out[:, s * ncomp:(s + 1) * ncomp] * sigma[s]) @ V[s].T
                      for s in range(4)], axis=1)
        cls.append(eo.inverse_transform(y, t))
    cls = np.stack(cls)
    mref, eref = eo.ensemble_stats(cls)
    scale = np.abs(mref).copy()
    scale[:, 2] = np.sqrt(mref[:, 0] * mref[:, 1])
    e4 = np.max(np.abs(cls - mref[None]) / scale[None], axis=(0, 3))
    c = cl.cpu().numpy()
    assert np.max(np.abs(c - mref) / scale) <= 2e-4
    np.testing.assert_array_equal(c, cl1.cpu().numpy())
    np.testing.assert_allclose(err4.cpu().numpy(), e4, rtol=1e-2, atol=2e-4)
    np.testing.assert_array_equal(err.cpu().numpy(), err4.cpu().numpy().max(axis=1))
    np.testing.assert_allclose(err.cpu().numpy(), eref, rtol=1e-2, atol=2e-4)
    np.testing.assert_array_equal(flag4.cpu().numpy(), (err4.cpu().numpy() > 1e-3))
    np.testing.assert_array_equal(flag.cpu().numpy(), (err.cpu().numpy() > 1e-3))
    emu.close()


@pytest.mark.parametrize("n,width,depth,ncomp", [(1, 16, 1, 8), (31, 33, 2, 7), (33, 64, 3, 9),
                                                 (130, 100, 2, 12), (2500, 512, 1, 8)])
def test_gradient_edges(torch_dev, ctx, n, width, depth, ncomp):  # noqa: F811
    rng = np.random.default_rng(32)
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


def test_exp_sinh_range(torch_dev, ctx):  # noqa: F811
    """With all weights zero the spectra are exp(mean) and t sinh(mean) of the FP32 means: within
    2 units in the last place each (and one rounding by t), over the range where they are
    finite, around sinh's change of form at 1, and at signed zeros."""
    nl, ncomp = 4096, 8
    emu = make_emu(ctx, nl=nl, ncomp=ncomp, width=16, depth=1, members=1)
    sizes = eo.layer_sizes(5, 16, 1, 4 * ncomp)
    emu.emu_set_params(0, np.zeros_like(glorot(np.random.default_rng(0), sizes)))
    mu = np.zeros((4, nl), dtype=np.float32)
    mu[0] = np.linspace(-708, 709, nl)
    mu[1] = np.linspace(-1.5, 1.5, nl)
    mu[2] = np.concatenate([np.linspace(-710.4, 710.4, nl // 2), np.linspace(-1.1, 1.1, nl // 4),
                            np.geomspace(1e-30, 2, nl // 4)])
    mu[3] = np.geomspace(1e-30, 700, nl)
    mu[2, :2] = -0.0, 0.0
    mu[3, :2] = -0.0, 0.0
    t = np.full(nl, 0.75)
    emu.emu_set_pca(-np.ones(5), np.ones(5), mu.astype(np.float64), np.zeros((4, nl, ncomp)),
                    np.ones((4, ncomp)), t)
    cl, _, _ = emu.emu_infer_spectra(dev(torch_dev, np.zeros((3, 5))), threshold=1e-3)
    got = cl.cpu().numpy()
    ref = np.exp(mu.astype(np.longdouble))
    ref[2] = 0.75 * np.sinh(mu[2].astype(np.longdouble))
    err = np.abs(got - ref) / np.maximum(np.abs(ref), np.finfo(np.float64).tiny)
    assert np.max(err) <= 5 * 2.0 ** -53
    emu.close()
