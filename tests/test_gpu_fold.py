"""The folded FP32 passes over 256-interval lines of large 3D grids against the
generic passes of the same library (which the parity tests hold to the oracle).

Both sides round in FP32: a transform of 512 points adds about log2(512) eps times a
small constant, so three steps of the two paths may differ by a few 1e-6 relative to
the largest value; 5e-6 is the bound."""
import pytest
import torch

import paper_2209_11922_amd as eife
from paper_2209_11922_amd.binding import TX_FFT, TX_FFT_GENERIC

pytestmark = pytest.mark.gpu

# y lines at the smallest launch that takes the folded column pass; z lines with a ragged last tile (99
# columns); x lines with an odd number of rows; every axis at once
SHAPES = [(256, 256, 65), (100, 130, 256), (256, 200, 200), (256, 256, 256)]


@pytest.mark.parametrize("stages", [1, 2, 3])
@pytest.mark.parametrize("N", SHAPES)
@pytest.mark.parametrize("kind", [eife.F_ALLEN_CAHN, eife.F_MMS_U2])
def test_folded_passes_match_generic(N, stages, kind):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    u0 = torch.rand([n - 1 for n in reversed(N)], device="cuda", generator=gen) * 1.8 - 0.9
    out = []
    for tx in (TX_FFT, TX_FFT_GENERIC):
        g = eife.Grid(N, [1.0 / n for n in N], 4e-4, "f32")
        g.set_transform(tx)
        g.set_phi(0.005, stages)
        out.append(g.step(u0.clone(), 3, kind, 0.1))
    torch.cuda.synchronize()
    err = float((out[0] - out[1]).abs().max() / out[1].abs().max())
    assert err < 5e-6, err


def test_folded_passes_are_deterministic():
    u0 = torch.rand(255, 255, 255, device="cuda") * 1.8 - 0.9
    g = eife.Grid([256] * 3, [1.0 / 256] * 3, 4e-4, "f32")
    g.set_phi(0.005, 2)
    runs = [g.step(u0.clone(), 2, eife.F_ALLEN_CAHN) for _ in range(2)]
    assert torch.equal(runs[0], runs[1])
