"""GPU: cells, counts and weight sums of kernel-gridded uv grids at the sizes whose
rows lie in the signed layout (256 to 2048) against the FP64 oracle, bounds as in
the kernel gridding tests; and the occupancy pass over more images than one of its
launches takes, against the same images in a call of their own."""
import numpy as np
import pytest
import torch

import paper_2405_13478_amd as blink
from oracle import C_LIGHT
from oracle import kernel_gridding as kg

from _gpu_util import device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,W,uniform", [(32, 6, 0), (256, 6, 0), (256, 9, 1), (512, 5, 1), (1024, 6, 0), (1024, 4, 1),
                                         (2048, 6, 1), (2048, 12, 0)])
def test_grid_cells_of_the_signed_layout(N, W, uniform):
    rng = np.random.default_rng(N + W)
    B = 700
    uvw = np.zeros((1, B, 3))
    uvw[0, :, :2] = rng.normal(0, 0.2 * N, (B, 2))
    uvw[0, ::7, :2] = uvw[0, 0, :2] + rng.uniform(-0.4, 0.4, (100, 2))     # many on one cell and its neighbours
    vis = (rng.standard_normal((1, 1, B)) + 1j * rng.standard_normal((1, 1, B))).astype(np.complex64)
    to = lambda x: torch.from_numpy(x).to(device())    # noqa: E731
    g, c, w, nd = blink.grid(to(vis), to(uvw), to(np.array([C_LIGHT])), grid_n=N, pixscale=1.0 / N, weighting=uniform,
                             kernel_support=W)
    xu, xv = uvw[0, :, 0], uvw[0, :, 1]                                    # one cell a metre
    keep = kg.conv_keep(xu, xv, W, N)
    om = kg.uniform_weights(xu, xv, keep, N) if uniform else None
    S, cnt, total = kg.grid_conv(vis[0, 0], xu, xv, keep, N, W, kg.kb_default_beta(W), om)
    assert 0 < (~keep).sum() == int(nd[0])
    assert np.array_equal(c.cpu().numpy()[0], cnt)
    got = g.cpu().numpy()[0].astype(np.complex128)
    assert np.linalg.norm(got - S) <= 2e-6 * np.linalg.norm(S)
    assert abs(float(w[0]) - total) <= 2e-6 * total


def test_occupancy_pass_in_several_launches():
    N, M, C = 2048, 2, 16384 + 13                      # 16,384 images of 2048^2 are one launch
    rng = np.random.default_rng(3)
    uvw = np.zeros((1, 8, 3))
    uvw[0, :, :2] = rng.uniform(-600, 600, (8, 2))
    uvw[0, 1, :2] = uvw[0, 0, :2] + 1e-3               # one cell
    uvw[0, 2, :2] = -uvw[0, 0, :2]                     # its mirror
    vis = (rng.standard_normal((1, C, 8)) + 1j * rng.standard_normal((1, C, 8))).astype(np.complex64)
    freq = C_LIGHT * np.linspace(0.9, 1.0, C)
    to = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(device())    # noqa: E731
    kw = dict(grid_n=N, pixscale=1.0 / N, out_n=M, weighting=1, kernel_support=4, chunk_images=0)
    w = torch.empty(C, device=device())
    img = blink.image_batch(to(vis), to(uvw), to(freq), weight_sum=w, **kw)
    for c0, c1 in ((0, 20), (16370, C)):
        wp = torch.empty(c1 - c0, device=device())
        part = blink.image_batch(to(vis[:, c0:c1]), to(uvw), to(freq[c0:c1]), weight_sum=wp, **kw)
        assert torch.equal(img[c0:c1], part) and torch.equal(w[c0:c1], wp)
    assert bool((w > 0).all())
