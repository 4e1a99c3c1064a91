"""The passes over lines of 1024, 2048 and 4096 intervals against the generic passes of
the same library (which the parity tests hold to the oracle), in every layout that the
column rule chooses: one, two or four column pairs per block, few and many blocks, odd
numbers of rows and ragged last column tiles.

Two FFTs of up to 8192 points in the same precision differ by log2(8192) eps times a
small constant per transform: 1e-12 (FP64) and 5e-6 (FP32) of the largest value bound
three steps with room.
"""
import pytest
import torch

import paper_2209_11922_amd as eife
from paper_2209_11922_amd.binding import TX_FFT, TX_FFT_GENERIC

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 5e-6}
SHAPES = [(1024, 6), (2048, 6), (4096, 6), (40, 1024), (40, 2048), (40, 4096), (1100, 2048), (1100, 4096),
          (200, 18, 1024), (200, 18, 2048), (4096,)]


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("stages", [1, 2])
@pytest.mark.parametrize("N", SHAPES, ids=lambda N: "x".join(map(str, N)))
def test_long_lines_match_generic(N, stages, dtype):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    out = []
    for tx in (TX_FFT, TX_FFT_GENERIC):
        g = eife.Grid(list(N), [1.0 / n for n in N], 4e-4, dtype)
        g.set_transform(tx)
        g.set_phi(0.005, stages)
        gen.manual_seed(5)
        u = torch.rand([n - 1 for n in reversed(N)], device="cuda", generator=gen, dtype=torch.float64) * 1.8 - 0.9
        out.append(g.step(u.to(g.torch_dtype), 3, eife.F_ALLEN_CAHN, 0.1).double())
        g.close()
    err = float((out[0] - out[1]).abs().max() / out[1].abs().max())
    assert err < TOL[dtype], err
