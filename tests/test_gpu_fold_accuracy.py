"""Rounding of the folded FP32 passes: no further from the FP64 oracle than the wave-local
passes of eife_fast.hpp, which do the same transforms without the symmetry."""
import numpy as np
import pytest

import seeded_inputs
from oracle import problems, spectral, stepper

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

# relative 2-norm error of the wave-local passes (the library without eife_fold.hpp) on this run
WAVE_LOCAL = 3.56e-7


def test_folded_passes_round_no_more_than_the_wave_local_ones():
    import paper_2209_11922_amd as eife
    N, D, tau, steps = [256] * 3, 4e-4, 0.005, 3
    u0 = seeded_inputs.uniform_field(0, N).astype(np.float32)
    g = eife.Grid(N, [1.0 / 256] * 3, D, "f32")
    g.set_phi(tau, 2)
    got = g.step(torch.tensor(u0, device="cuda"), steps, eife.F_ALLEN_CAHN).double().cpu().numpy()
    g.close()
    ref = stepper.run(spectral.SineBasis(N, [1.0 / 256] * 3, D), u0.astype(np.float64), problems.allen_cahn(), tau, steps, 2)
    err = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    print(f"255^3: {err:.4e}")
    assert err <= WAVE_LOCAL
