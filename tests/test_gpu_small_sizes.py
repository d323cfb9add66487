"""GPU: image batches at the power-of-two sizes below 1024 and at 2048 against the
FP64 oracle: several row pairs and columns on one wavefront, row tiles that are
partly filled, cutouts that are not a multiple of the lanes per vector, columns
of one gather step and of many, both weightings. Bound: the repository's per-image
FP32 one."""
import numpy as np
import pytest
import torch

import oracle
import paper_2405_13478_amd as blink

from _gpu_util import REL_L2_FP32, device, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,n_ant,T,C,uniform,rows_wg", [
    (32, 32, 40, 2, 2, False, 0), (32, 10, 12, 1, 3, True, 0), (64, 64, 30, 1, 2, True, 3), (64, 38, 60, 2, 1, False, 0),
    (128, 128, 120, 1, 2, True, 0), (128, 100, 30, 3, 1, False, 5), (256, 256, 90, 1, 2, False, 0),
    (256, 128, 20, 1, 1, True, 2), (512, 512, 40, 1, 1, True, 0), (512, 256, 64, 1, 1, False, 0),
    (512, 334, 100, 1, 1, False, 7), (2048, 70, 24, 1, 1, True, 2)])
def test_small_sizes(N, M, n_ant, T, C, uniform, rows_wg):
    rng = np.random.default_rng(N * 7 + M)
    B = n_ant * (n_ant - 1) // 2
    uvw = np.zeros((T, B, 3))
    uvw[:, :, :2] = rng.normal(0, 0.2 * N, (T, B, 2))
    flags = (rng.random((T, B)) < 0.05).astype(np.uint8)
    pix, freq = 1.0 / N, oracle.C_LIGHT * np.linspace(0.9, 1.0, C)        # about one cell a metre
    vis = (rng.standard_normal((T, C, B)) + 1j * rng.standard_normal((T, C, B))).astype(np.complex64)
    to = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(device())    # noqa: E731
    w = torch.empty(T * C, device=device())
    img = blink.image_batch(to(vis), to(uvw), to(freq), grid_n=N, pixscale=pix, out_n=M, weighting=int(uniform),
                            flags=to(flags), weight_sum=w, rows_wg=rows_wg)
    ref, W = oracle.image_batch(vis, uvw, freq, N, pix, M, int(uniform), 1, flags)
    for i in range(T * C):
        assert rel_l2(img[i].cpu().numpy(), ref[i]) <= REL_L2_FP32, i
    assert np.array_equal(w.cpu().numpy(), W.astype(np.float32))
