"""The corrector's gradient at the edges of the backward kernels' tiles: one node, full
and ragged patches of 4 rows by 64 nodes, strips that end inside a row group, several
images.  Against the reference that rounds where the kernels round: what remains is the
FP32 order of the sums and rare flips at a BF16 rounding boundary, each at most 2^-8 of
one value, so a block of the gradient agrees to 1e-2 of its norm also where only a few
nodes add up.
"""
import numpy as np
import pytest

from test_gpu_corrector import _data, _dev, _grad_bf16, _lib, _params, _rel2, cr

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,ny,nx", [(1, 1, 1), (1, 4, 64), (2, 5, 65), (1, 33, 17), (3, 9, 130), (1, 67, 300)])
def test_gradient_at_tile_edges(B, ny, nx):
    eife = _lib()
    p = _params(11)
    un, uc, uf = _data(12, B, ny, nx)
    c = eife.Corrector(nx, ny, B)
    c.set_params(p)
    c.set_scale(0.02)
    loss, g = c.grad(_dev(un), _dev(uc), _dev(uf))
    loss2, g2 = c.grad(_dev(un), _dev(uc), _dev(uf))
    c.close()
    f = lambda a: np.float32(a).astype(np.float64)  # noqa: E731
    ref = _grad_bf16(p.astype(np.float64), f(un), f(uc), f(uf), 0.02)
    bounds = np.cumsum([0] + cr.SIZES)
    for k, (lo, hi) in enumerate(zip(bounds[:-1], bounds[1:])):
        e = _rel2(g[lo:hi].astype(np.float64), ref[lo:hi])
        print(f"grad block {k}: {e:.2e}")
        assert e <= 1e-2, k
    assert loss2 == loss and np.array_equal(g, g2)
