"""Example 5.2's boundary load from its per-time tables: the line lengths whose
specialised row passes read them (power of two, 9-multiple, whole-line FP64 of 1024
and more intervals, FP32 256-interval rows of a large 3D grid), and runs whose
evaluations cross the tables' 16-time blocks inside a step (EIFE3, variable steps).
Against the FP64 oracle, and against single-step calls, at the tolerances of the
other parity tests: relative max-norm 1e-12 (FP64), 1e-5 (FP32).
"""
import numpy as np
import pytest

from oracle import fem, problems, spectral, stepper

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5}
EPS = 0.05
T_END = 3.0 * np.sqrt(2.0) * EPS / 5.0


def _setup(N, dtype, stages, tau):
    import paper_2209_11922_amd as eife
    lengths = [np.sqrt(2.0), 0.125, 0.125][: len(N)]
    h = [L / n for L, n in zip(lengths, N)]
    wave, _, _ = problems.traveling_wave_solution(EPS)
    u0 = wave(0.0, fem.mesh(N, h)[0]) * np.ones(tuple(n - 1 for n in reversed(N)))
    g = eife.Grid(N, h, 1.0, dtype)
    g.set_forcing(EPS, 0.0)
    g.set_phi(tau, stages)
    return eife, g, h, u0, torch.tensor(u0, dtype=g.torch_dtype, device="cuda")


def _rel(got, ref):
    return float(np.max(np.abs(got - ref)) / np.max(np.abs(ref)))


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("N", [[1024], [4096], [512, 3], [1024, 4, 3], [192, 5], [256, 32, 64]],
                         ids=lambda N: "x".join(map(str, N)))
def test_specialised_rows_match_oracle(N, dtype):
    tau, steps = T_END / 256, 10  # 20 evaluations: the second block of tables is read too
    eife, g, h, u0, u = _setup(N, dtype, 2, tau)
    g.step(u, steps, eife.F_TRAVELING_WAVE, 0.0)
    got = u.double().cpu().numpy()
    g.close()
    w, w_t, _ = problems.traveling_wave_solution(EPS)
    ref = stepper.run(spectral.make_basis("C", N, h, 1.0), u0, problems.traveling_wave(EPS), tau, steps, 2,
                      boundary=(lambda t, X: w(t, X[0]), lambda t, X: w_t(t, X[0])))
    assert _rel(got, ref) <= TOL[dtype]


@pytest.mark.parametrize("stages", [1, 2, 3])
@pytest.mark.parametrize("variable", [False, True])
def test_blocks_of_tables_match_single_steps(stages, variable):
    N, steps, t0 = [64, 6, 4], 18, 0.01
    tau = T_END / 256
    taus = [tau * (1.0 + 0.3 * np.sin(1.7 * i)) if variable else tau for i in range(steps)]
    eife, g, h, u0, u = _setup(N, "f64", stages, tau)
    v = u.clone()
    if variable:
        g.step_variable(u, taus, eife.F_TRAVELING_WAVE, t0)
    else:
        g.step(u, steps, eife.F_TRAVELING_WAVE, t0)
    t = t0
    for dt in taus:
        g.set_phi(dt, stages)
        g.step(v, 1, eife.F_TRAVELING_WAVE, t)
        t += dt
    assert _rel(u.cpu().numpy(), v.cpu().numpy()) <= TOL["f64"]
    g.close()


def test_large_grid_of_256_interval_rows_matches_generic():
    """FP32 256-interval rows enough for the folded row pass, which has no traveling wave:
    these rows stay on the wave-local pass.  Against the generic passes."""
    N, tau = [256, 184, 184], T_END / 256
    assert 183 * 183 >= 16 * 8 * torch.cuda.get_device_properties(0).multi_processor_count
    out = []
    for transform in ("TX_FFT", "TX_FFT_GENERIC"):
        eife, g, _, _, u = _setup(N, "f32", 2, tau)
        g.set_transform(getattr(eife.binding, transform))
        g.step(u, 2, eife.F_TRAVELING_WAVE, 0.0)
        out.append(u.double().cpu().numpy())
        g.close()
    assert _rel(out[0], out[1]) <= TOL["f32"]
