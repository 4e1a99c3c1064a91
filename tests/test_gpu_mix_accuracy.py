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
