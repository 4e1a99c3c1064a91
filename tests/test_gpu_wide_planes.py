"""Grids of more than 2^31 elements, whose z lines are longer than 32-bit offsets reach: a
sum of eigenmodes under f = 0, each of which the scheme multiplies by exp(-tau D lambda)
exactly.  The relative max-norm bound is that of the other FP32 / FP64 parity tests."""
import math

import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

MODES = [(1, 1, 1), (2, 3, 5), (7, 2, 40)]


def _eig(k, N, h, per):
    c = math.cos((2 if per else 1) * math.pi * k / N)
    return (2.0 / h) * (1.0 - c) / ((h / 6.0) * (4.0 + 2.0 * c))


def _mode(k, N, per, dtype):
    i = torch.arange(0 if per else 1, N, dtype=torch.float64, device="cuda")
    v = torch.cos(2 * math.pi * k * i / N) if per else torch.sin(math.pi * k * i / N)
    return v.to(dtype)


@pytest.mark.parametrize("N,dtype,bc,stages", [
    ([4096, 2560, 256], "f32", "dirichlet", 2), ([4096, 2560, 256], "f32", "dirichlet", 3),
    ([4096, 2760, 192], "f32", "dirichlet", 2), ([4096, 1030, 512], "f32", "dirichlet", 1),
    ([4096, 1030, 512], "f64", "dirichlet", 2), ([4096, 2100, 256], "f32", "periodic", 2),
])
def test_eigenmodes_decay(N, dtype, bc, stages):
    import paper_2209_11922_amd as eife
    per = bc == "periodic"
    print(f"wide planes {N} {dtype} {bc} {stages}", flush=True)
    h = [1.0 / n for n in N]
    g = eife.Grid(N, h, 1e-4, dtype, bc=eife.BC_PERIODIC if per else eife.BC_DIRICHLET)
    tau = 0.05
    g.set_phi(tau, stages)
    dt = g.torch_dtype
    ax = [[_mode(k[a], N[a], per, dt) for a in range(3)] for k in MODES]
    n = [len(v) for v in ax[0]]
    u = torch.zeros(n[2], n[1], n[0], dtype=dt, device="cuda")
    for x, y, z in ax:
        u.addcmul_(z.view(-1, 1, 1), torch.outer(y, x))
    g.step(u, 1, eife.F_ZERO)
    torch.cuda.synchronize()
    g.close()
    dec = [math.exp(-tau * 1e-4 * sum(_eig(k[a], N[a], h[a], per) for a in range(3))) for k in MODES]
    planes = [torch.outer(y, x).double() * d for (x, y, _), d in zip(ax, dec)]
    err = max(float((u[m].double() - sum(p * float(z[m]) for p, (_, _, z) in zip(planes, ax))).abs().max())
              for m in range(n[2]))
    del u, planes
    torch.cuda.empty_cache()
    print(f"  err {err:.2e}", flush=True)
    assert err <= {"f64": 1e-12, "f32": 1e-5}[dtype] * sum(dec)
