"""GPU: the emulator's exp and sinh lose no accuracy against the device library's (largest error
0.864 and 0.858 units in the last place over FP32 arguments, measured): at most 0.864 units each.
With all weights zero, one member and t = 1 the spectra are exp(mean) and sinh(mean) of FP32 means;
the reference is the 64-bit significand of long double (its own error is below 0.001 units)."""
import numpy as np
import pytest

from oracle import emu_oracle as eo
from test_gpu_emu import ctx, dev, glorot, make_emu, torch_dev  # noqa: F401

pytestmark = pytest.mark.gpu


def units(got, ref):
    _, e = np.frexp(ref.astype(np.float64))
    return np.abs(got - ref) / np.ldexp(np.longdouble(1), e - 53)


def test_exp_sinh_units(torch_dev, ctx):  # noqa: F811
    rng = np.random.default_rng(12)
    nl, ncomp = 16000, 8
    emu = make_emu(ctx, nl=nl, ncomp=ncomp, width=16, depth=1, members=1)
    sizes = eo.layer_sizes(5, 16, 1, 4 * ncomp)
    emu.emu_set_params(0, np.zeros_like(glorot(rng, sizes)))
    worst = np.zeros(2)
    for lo, hi in ((-40, 10), (-40, 10), (-700, 709), (-1.2, 1.2), (0.8, 2.0), (1.0, 1.6), (-3, 3)):
        mu = rng.uniform(lo, hi, size=(4, nl)).astype(np.float32)
        emu.emu_set_pca(-np.ones(5), np.ones(5), mu.astype(np.float64), np.zeros((4, nl, ncomp)),
                        np.ones((4, ncomp)), np.ones(nl))
        cl, _, _ = emu.emu_infer_spectra(dev(torch_dev, np.zeros((1, 5))), threshold=1e-3)
        got = cl.cpu().numpy()[0].astype(np.longdouble)
        m = mu.astype(np.longdouble)
        worst[0] = max(worst[0], float(np.max(units(got[[0, 1, 3]], np.exp(m[[0, 1, 3]])))))
        worst[1] = max(worst[1], float(np.max(units(got[2], np.sinh(m[2])))))
    emu.close()
    print("exp %.3f, sinh %.3f units in the last place" % tuple(worst))
    assert worst[0] <= 0.864 and worst[1] <= 0.864, worst
