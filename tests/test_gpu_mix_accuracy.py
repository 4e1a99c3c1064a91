"""Rounding of the mixed-radix passes.  With f = 0 a step is a forward transform per axis,
a product with exp(-tau D lambda) and an inverse transform per axis."""
import math

import numpy as np
import pytest
import scipy.fft

from oracle import spectral

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

U = 2.0 ** -24  # unit roundoff, FP32


def _step(N, seed):
    import paper_2209_11922_amd as eife
    h, D, tau = [1.0 / n for n in N], 1e-4, 0.01
    u0 = np.random.default_rng(seed).uniform(-0.9, 0.9, tuple(n - 1 for n in reversed(N))).astype(np.float32)
    g = eife.Grid(N, h, D, "f32")
    g.set_transform(eife.binding.TX_FFT_GENERIC)
    g.set_phi(tau, 1)
    got = g.step(torch.tensor(u0, device="cuda"), 1, eife.F_ZERO).double().cpu().numpy()
    g.close()
    hat = scipy.fft.dstn(u0.astype(np.float64), type=1, norm="ortho")
    return got, scipy.fft.idstn(hat * np.exp(-tau * spectral.SineBasis(N, h, D).lam), type=1, norm="ortho")


@pytest.mark.parametrize("N", [96, 100, 240, 256, 360, 1000, 2048, 4000])
def test_line_rounds_like_its_layers(N):
    """A transform of L = 2 N points rounds once per layer of additions (log2 L of them), twice
    per set of twiddles (three stages between the first and the last at most) and once in the
    scale, each by U / sqrt(3) rms; two transforms and the stage between them (3) add up
    in squares.  Powers of a twiddle formed by a chain of products exceed this
    (L = 720: 2.7e-7 against 1.9e-7)."""
    got, ref = _step([N], N)
    err = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    bound = U * math.sqrt((2 * (math.log2(2 * N) + 6 + 1) + 3) / 3)
    print(f"N = {N}: {err:.2e}, bound {bound:.2e}")
    assert err <= bound


def _fourier(u, inverse=False):
    """The DFT along every axis by matrix products in extended precision."""
    for a, n in enumerate(u.shape):
        t = 2 * np.arctan2(np.longdouble(0), np.longdouble(-1)) / n * (np.outer(np.arange(n), np.arange(n)) % n)
        F = (np.cos(t) + (1j if inverse else -1j) * np.sin(t)) / (n if inverse else 1)
        u = np.moveaxis(np.tensordot(F, u, (1, a)), 0, a)
    return u


def test_scale_factors_do_not_add_up():
    """Periodic 48^3, FP64: both scale factors of such lines round up by 1.4e-16, which six
    transforms would add up to 8e-16.  The roundings themselves, counted as above with three
    more per transform for the split into real coefficients, come to 5.2e-16."""
    import paper_2209_11922_amd as eife
    N, D, tau = 48, 1e-4, 0.01
    u0 = np.random.default_rng(1).uniform(-0.9, 0.9, (N, N, N))
    g = eife.Grid([N] * 3, [1.0 / N] * 3, D, "f64", bc=eife.BC_PERIODIC)
    g.set_phi(tau, 1)
    got = g.step(torch.tensor(u0, device="cuda"), 1, eife.F_ZERO).cpu().numpy().astype(np.longdouble)
    g.close()
    s2 = np.sin(np.arctan2(np.longdouble(0), np.longdouble(-1)) * np.arange(N) / N) ** 2
    lam = 12 * N * N * s2 / (3 - 2 * s2)
    lam = lam[:, None, None] + lam[None, :, None] + lam[None, None, :]
    ref = _fourier(_fourier(u0.astype(np.clongdouble)) * np.exp(-np.longdouble(tau) * np.longdouble(D) * lam), inverse=True).real
    err = float(np.sqrt(((got - ref) ** 2).sum() / (ref ** 2).sum()))
    bound = 2.0 ** -53 * math.sqrt((6 * (math.log2(N) + 2 + 3) + 3) / 3)
    print(f"48^3 periodic: {err:.2e}, bound {bound:.2e}")
    assert err <= bound
