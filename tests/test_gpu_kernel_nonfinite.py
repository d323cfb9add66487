"""GPU: an infinite or NaN visibility in a uv grid with a gridding kernel reaches
the cells of its footprint and their mirrors and no other cell, in the signed row
layout (powers of two up to 2048) and the wrapped one, for footprints of W and of
W + 1 rows."""
import numpy as np
import pytest
import torch

import oracle
import paper_2405_13478_amd as blink
from oracle import kernel_gridding as kg

from _gpu_util import device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("uniform", [0, 1])
@pytest.mark.parametrize("N,W", [(32, 6), (64, 3), (128, 6), (180, 6), (256, 12), (512, 7), (1024, 6), (2048, 4)])
def test_nonfinite_visibility_stays_in_its_footprint(N, W, uniform):
    rng = np.random.default_rng(N + W)
    # fractional positions (W rows), whole and half ones (W + 1 rows for even and odd W)
    pos = rng.uniform(-0.25 * N, 0.25 * N, (24, 2))
    pos[::3] = np.rint(pos[::3])
    pos[1::3] = np.floor(pos[1::3]) + 0.5
    bad = [0, 1, 2, 5]
    vis = (rng.standard_normal((1, 1, 24)) + 1j * rng.standard_normal((1, 1, 24))).astype(np.complex64)
    vis[0, 0, bad] = [complex(np.inf, 1), complex(np.nan, np.nan), complex(2, -np.inf), complex(-np.inf, np.inf)]
    uvw = np.zeros((1, 24, 3))
    uvw[0, :, :2] = pos
    to = lambda x: torch.from_numpy(x).to(device())    # noqa: E731
    g, counts, _, _ = blink.grid(to(vis), to(uvw), to(np.array([oracle.C_LIGHT])), grid_n=N, pixscale=1.0 / N,
                                 weighting=uniform, kernel_support=W)
    spoiled = np.zeros((N, N), bool)
    for b in bad:
        iu, iv = kg.footprint(pos[b, 0], W), kg.footprint(pos[b, 1], W)
        assert max(abs(iu).max(), abs(iv).max()) < N // 2
        spoiled[np.ix_(iv % N, iu % N)] = spoiled[np.ix_(-iv % N, -iu % N)] = True
    got = g.cpu().numpy()[0]
    assert np.array_equal(~np.isfinite(got), spoiled)
    keep = np.ones(24, bool)
    om = kg.uniform_weights(pos[:, 0], pos[:, 1], keep, N) if uniform else None
    fine = vis[0, 0].copy()
    fine[bad] = 0
    S, cnt, _ = kg.grid_conv(fine, pos[:, 0], pos[:, 1], keep, N, W, kg.kb_default_beta(W), om)
    assert np.array_equal(counts.cpu().numpy()[0], cnt)
    assert np.linalg.norm((got - S)[~spoiled]) <= 2e-6 * np.linalg.norm(S)
