"""GPU parity of the mixed-radix passes over the radices and block shapes they choose:
line lengths whose plans use each radix (2 ... 10, 12, 15, 16 and prime stages), the
smallest lines, lines at the longest (a block of one pair, 32 values per thread), odd
row counts and ragged column tiles.  Against the FP64 oracle at the tolerances of the
other parity tests (FP64 1e-12, FP32 1e-5 relative max-norm)."""
import numpy as np
import pytest

import seeded_inputs
from oracle import problems, spectral, stepper

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5}


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("N,bc", [
    ([2, 3], "dirichlet"), ([5, 2, 3], "dirichlet"),           # the smallest lines
    ([60, 45], "dirichlet"), ([81, 49], "dirichlet"),           # 12 x 10, 15 x 6; 9s, 7s
    ([240, 35], "dirichlet"), ([250, 33], "dirichlet"),         # 16 x 6 x 5; 10 x 5 x 10; a prime stage
    ([4095, 3], "dirichlet"), ([3, 4000], "dirichlet"),         # the longest lines, rows and columns
    ([2187, 9], "dirichlet"), ([7, 2021], "dirichlet"),         # 3^7; two large primes
    ([45, 81], "periodic"), ([100, 15, 8], "periodic"), ([225], "periodic"),
])
def test_mixed_radix_lines(N, bc, dtype):
    import paper_2209_11922_amd as eife
    per = bc == "periodic"
    h = [1.0 / n for n in N]
    D = 1e-3 if per else 0.02 ** 2
    u0 = np.random.default_rng(17).uniform(-0.9, 0.9, tuple(reversed(N))) if per else seeded_inputs.uniform_field(17, N)
    print(f"mixed-radix {N} {dtype} {bc}", flush=True)
    g = eife.Grid(N, h, D, dtype, bc=eife.BC_PERIODIC if per else eife.BC_DIRICHLET)
    g.set_transform(eife.binding.TX_FFT_GENERIC)
    g.set_phi(0.01, 2)
    u = torch.tensor(u0, dtype=g.torch_dtype, device="cuda")
    g.step(u, 3, eife.F_ALLEN_CAHN)
    torch.cuda.synchronize()
    got = u.double().cpu().numpy()
    g.close()
    basis = spectral.make_basis("C", N, h, D, bc="periodic") if per else spectral.SineBasis(N, h, D)
    ref = stepper.run(basis, u0, problems.allen_cahn(), 0.01, 3, 2)
    err = float(np.max(np.abs(got - ref)) / np.max(np.abs(ref)))
    print(f"  rel err {err:.2e}")
    assert err <= TOL[dtype]
