"""GPU: with a gridding kernel, a baseline whose footprint ends within rounding of
the grid's edge is kept or dropped alike by the gridding, the image and the
adjoint, as the rule says on positions rounded to double: |x| + W/2 < N/2. The
positions are chosen so that the unrounded product u s lies on the other side of
that line than its rounded value (possible where W >= N/2)."""
from fractions import Fraction

import numpy as np
import pytest
import torch

import oracle
import paper_2405_13478_amd as blink
from oracle import kernel_gridding as kg

from _gpu_util import REL_L2_FP32, device, rel_l2

pytestmark = pytest.mark.gpu


def _edge(N, W, rng):
    """(frequency, u): fl(u s) + W/2 rounds to N/2, the exact u s + W/2 to less."""
    edge = np.float64(N // 2 - W / 2)
    x = np.nextafter(edge, 0)                                       # x + W/2 is halfway below N/2
    assert x + W / 2 == N // 2
    while True:
        f = rng.uniform(100e6, 200e6)
        s = oracle.blink_oracle.uv_scale(f, N, 1.0 / N)
        u = x / s
        for u in (np.nextafter(u, 0), u, np.nextafter(u, np.inf)):
            if np.float64(u) * np.float64(s) == x and Fraction(float(u)) * Fraction(float(s)) < Fraction(float(x)):
                return f, float(u)


@pytest.mark.parametrize("uniform", [0, 1])
@pytest.mark.parametrize("N,W", [(8, 4), (16, 8), (16, 10), (32, 16)])
def test_edge_baselines_are_dropped_everywhere(N, W, uniform):
    rng = np.random.default_rng(N * W)
    f, u = _edge(N, W, rng)
    near = np.nextafter(np.nextafter(u, 0), 0)                      # just inside: kept
    uv = np.array([[u, 0.1], [0.2, u], [-u, 0.3], [-0.4, -u], [u, u], [near, -near], [0.5, near], [0.3, -0.7]])
    B = len(uv)
    uvw = np.zeros((1, B, 3))
    uvw[0, :, :2] = uv
    freq = np.array([f])
    s = oracle.blink_oracle.uv_scale(f, N, 1.0 / N)
    keep = kg.conv_keep(uv[:, 0] * s, uv[:, 1] * s, W, N)
    assert not keep[:5].any() and keep[5:].all()
    vis = (rng.standard_normal((1, 1, B)) + 1j * rng.standard_normal((1, 1, B))).astype(np.complex64)
    gbar = rng.standard_normal((1, N // 2, N // 2)).astype(np.float32)
    to = lambda x: torch.from_numpy(x).to(device())    # noqa: E731
    kw = dict(grid_n=N, pixscale=1.0 / N, weighting=uniform, kernel_support=W)
    _, counts, wsum, dropped = blink.grid(to(vis), to(uvw), to(freq), **kw)
    r = kg.image_one_conv(vis[0, 0], uv[:, 0], uv[:, 1], f, N, 1.0 / N, N // 2, 0, W, weighting=uniform)
    assert int(dropped[0]) == 5 and np.array_equal(counts.cpu().numpy()[0], r["counts"])
    assert np.isclose(float(wsum[0]), r["W"], rtol=2e-6, atol=0)
    w = torch.empty(1, device=device())
    blink.image_batch(to(vis), to(uvw), to(freq), out_n=N // 2, weight_sum=w, **kw)
    assert np.isclose(float(w[0]), r["W"], rtol=2e-6, atol=0)
    vg, _ = blink.degrid_adjoint(to(gbar), to(vis), to(uvw), to(freq), out_n=N // 2, **kw)
    ref, _ = kg.adjoint_one_conv(gbar[0], vis[0, 0], uv[:, 0], uv[:, 1], f, N, 1.0 / N, 1, W, weighting=uniform)
    got = vg.cpu().numpy()[0, 0]
    assert np.array_equal(got == 0, ~keep)
    assert rel_l2(got.view(np.float32), ref.view(np.float64)) <= REL_L2_FP32
