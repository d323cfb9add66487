"""GPU: a gridding-kernel add rounds once. With beta = 0 every kernel weight is 1,
and under uniform weighting the n baselines of one cell weigh fl(1/n): their
footprint's cells are n fused multiply-adds in the order of the baselines, bit
for bit. Row layouts by N; footprints of W + 1 rows, one of them the last row."""
import numpy as np
import pytest
import torch

import oracle
import paper_2405_13478_amd as blink
from oracle import kernel_gridding as kg

from _gpu_util import device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,W", [(32, 6), (128, 4), (512, 8), (1024, 6), (1024, 12), (2048, 6)])
def test_adds_round_once(N, W):
    n, C = 7, 16
    rng = np.random.default_rng(N + W)
    vis = (rng.standard_normal((1, C, n)) + 1j * rng.standard_normal((1, C, n))).astype(np.complex64)
    uvw = np.zeros((1, n, 3))
    uvw[0, :, :2] = 8, 3                               # (the mirrored footprint lies apart in u)
    to = lambda x: torch.from_numpy(x).to(device())    # noqa: E731
    g = blink.grid(to(vis), to(uvw), to(np.full(C, oracle.C_LIGHT)), grid_n=N, pixscale=1.0 / N, weighting=1,
                   kernel_support=W, kernel_beta=0.0)[0].cpu().numpy()
    w = np.float64(np.float32(1) / np.float32(n))
    want = np.zeros((C, 2), np.float32)
    for b in range(n):                                 # the product of two floats is exact in 64 bits
        v = np.stack([vis[0, :, b].real, vis[0, :, b].imag], -1).astype(np.float64)
        want = (want + w * v).astype(np.float32)
    iu, iv = kg.footprint(8.0, W), kg.footprint(3.0, W)
    assert len(iv) == W + 1
    got = g[:, iv[:, None] % N, iu[None] % N]
    assert np.array_equal(got.real, np.broadcast_to(want[:, :1, None], got.shape))
    assert np.array_equal(got.imag, np.broadcast_to(want[:, 1:, None], got.shape))
