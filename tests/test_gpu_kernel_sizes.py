"""GPU: kernel gridding over the grid sizes and footprint widths whose column
layout differs (signed rows without padding at the powers of two, wrapped padded
rows elsewhere), and its occupancy pass for uniform weighting, which takes one
wavefront per column: sizes whose columns do not fill the last workgroup, image
counts that are not a multiple of eight, many baselines on one cell. Images and
weight sums against the FP64 oracle, bounds as in the kernel gridding tests."""
import numpy as np
import pytest
import torch

import paper_2405_13478_amd as blink
from oracle import C_LIGHT
from oracle import kernel_gridding as kg

from _gpu_util import REL_L2_FP32, device, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,n_ant,T,C,W,uniform,sigma", [
    (12, 12, 8, 1, 2, 3, True, 0.15), (16, 16, 30, 1, 1, 4, True, 0.02), (32, 20, 40, 3, 3, 6, True, 0.2),
    (64, 32, 40, 1, 1, 16, False, 0.2), (64, 34, 90, 2, 1, 2, True, 0.15), (128, 128, 60, 1, 9, 2, True, 0.2),
    (180, 100, 30, 1, 1, 7, True, 0.2), (256, 100, 64, 1, 2, 9, False, 0.2), (512, 512, 30, 1, 1, 5, True, 0.002),
    (1024, 512, 40, 1, 1, 8, True, 0.2), (1024, 510, 20, 1, 1, 3, False, 0.2), (2048, 64, 24, 1, 1, 6, True, 0.2),
    (2048, 1024, 24, 1, 1, 4, False, 0.2)])
def test_kernel_sizes(N, M, n_ant, T, C, W, uniform, sigma):
    rng = np.random.default_rng(N * 31 + W)
    B = n_ant * (n_ant - 1) // 2
    uvw = np.zeros((T, B, 3))
    uvw[:, :, :2] = rng.normal(0, sigma * N, (T, B, 2))
    flags = (rng.random((T, B)) < 0.05).astype(np.uint8)
    pix, freq = 1.0 / N, C_LIGHT * np.linspace(0.9, 1.0, C)               # about one cell a metre
    vis = (rng.standard_normal((T, C, B)) + 1j * rng.standard_normal((T, C, B))).astype(np.complex64)
    to = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(device())    # noqa: E731
    w = torch.empty(T * C, device=device())
    img = blink.image_batch(to(vis), to(uvw), to(freq), grid_n=N, pixscale=pix, out_n=M, weighting=int(uniform),
                            flags=to(flags), weight_sum=w, kernel_support=W)
    ref, wref = kg.image_batch_conv(vis, uvw, freq, N, pix, M, 1, W, None, flags, weighting=int(uniform))
    for i in range(T * C):
        assert rel_l2(img[i].cpu().numpy(), ref[i]) <= REL_L2_FP32, i
    assert np.allclose(w.cpu().numpy(), wref, rtol=2e-6, atol=0)
