"""GPU: the X-engine's large antenna tiles (calls of many spectra of more than
64 antennas) against integer sums, bit for bit: tiles partly filled, sample
counts that end inside a 64-sample chunk, one chunk and several, and the most
negative 8-bit values (whose complement form carries the sum of the real parts)."""
import numpy as np
import pytest
import torch

import paper_2405_13478_amd as blink

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,C,A,S,extreme", [(4, 64, 65, 16, False), (16, 16, 128, 64, False), (3, 29, 129, 80, False),
                                             (8, 12, 193, 208, False), (6, 16, 256, 336, False),
                                             (2, 50, 130, 1040, True), (1, 3, 200, 272, False), (1, 1, 64, 4096, True)])
def test_large_tiles_are_exact(T, C, A, S, extreme):
    rng = np.random.default_rng(A * 1000 + S)
    volt = rng.integers(-128, 128, size=(T, C, A, S, 2)).astype(np.int8)
    if extreme:
        volt[:, :, ::3] = -128
        volt[:, :, 1::3, :, 1] = 127
    vis, autos = blink.correlate(torch.from_numpy(volt).to("cuda:0"), autos=True)
    a1, a2 = np.triu_indices(A, 1)
    for t in range(T):
        for c in range(C):
            x = volt[t, c].astype(np.float64)              # sums below 2^53: exact
            r, q = x[..., 0], x[..., 1]
            re, im = r @ r.T + q @ q.T, q @ r.T - r @ q.T
            got = vis[t, c].cpu().numpy()
            assert np.array_equal(got.real, re[a1, a2].astype(np.float32)), (t, c)
            assert np.array_equal(got.imag, im[a1, a2].astype(np.float32)), (t, c)
            assert np.array_equal(autos[t, c].cpu().numpy(), np.diag(re).astype(np.float32)), (t, c)
