"""GPU: the adjoint's column transform multiplies by table twiddles that are
rounded once from 64 bits, never by FP32 products of them. At sizes whose plan
ends in radix 2 or 4, one bright pixel in the central image column and n rows
(0 < n < the last radix) below the phase centre reaches the last stage through exact
additions alone, so the gradient of a baseline in v cell k is 2 exp(-2 pi i n k / N)
with the rounding of one twiddle: half a unit in the last place per part."""
import numpy as np
import pytest
import torch

import oracle
import paper_2405_13478_amd as blink

from _gpu_util import device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("uniform", [0, 1])
@pytest.mark.parametrize("N,M,n", [(32, 16, 1), (64, 32, 1), (64, 64, 2), (64, 32, 3), (512, 256, 1), (1024, 512, 1),
                                   (1024, 512, 2), (1024, 1024, 2), (1024, 512, 3), (1024, 1022, 3)])
def test_one_pixel_gradient_is_one_rounded_twiddle(N, M, n, uniform):
    H = N // 2
    k = np.arange(-H + 1, H)
    k = k[k != 0]                                 # (at u = v = 0 the two cells coincide)
    cells = np.concatenate([np.stack([np.full(k.size, c), k], 1) for c in (0, 3, H - 1)])
    uvw = np.zeros((1, len(cells), 3))
    uvw[0, :, :2] = cells                         # one cell a metre
    gbar = np.zeros((1, M, M), np.float32)
    gbar[0, M // 2 + n, M // 2] = 1.0
    to = lambda x: torch.from_numpy(x).to(device())    # noqa: E731
    vis = torch.zeros((1, 1, len(cells)), dtype=torch.complex64, device=device())
    vg, _ = blink.degrid_adjoint(to(gbar), vis, to(uvw), to(np.array([oracle.C_LIGHT])), grid_n=N, pixscale=1.0 / N,
                                 out_n=M, weighting=uniform, norm=blink.NORM_NONE)
    got = vg.cpu().numpy()[0, 0]
    turn = 2 * np.pi * (n * cells[:, 1] % N) / N
    # u = 0 holds v cells k and -k, two entries a cell: uniform weighting halves them
    size = np.where((cells[:, 0] == 0) & bool(uniform), 1.0, 2.0)
    for part, ref in ((got.real, size * np.cos(turn)), (got.imag, -size * np.sin(turn))):
        half = 0.5 * np.spacing(np.abs(ref).astype(np.float32)).astype(np.float64)
        worst = np.max(np.abs(part.astype(np.float64) - ref) / (half + 1e-15))
        assert worst <= 1.001, worst
