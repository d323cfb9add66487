"""GPU: every form of the X-engine against integer sums, bit for bit: the one
workgroup per spectrum form at each number of 32-antenna rows that the other
correlator tests leave out, with rows that end inside a 256-byte chunk and the
most negative 8-bit values; tiles of more than 256 antennas (three and more large
tiles an edge, small ones too); and more spectra than one launch takes."""
import numpy as np
import pytest
import torch

import paper_2405_13478_amd as blink

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,C,A,S,extreme", [
    (4, 6, 20, 48, False), (3, 7, 2, 16, True), (5, 8, 50, 80, False), (10, 12, 180, 80, False), (10, 14, 193, 208, False),
    (10, 16, 256, 336, False), (4, 40, 256, 144, True),
    (1, 2, 257, 272, True), (2, 3, 300, 48, False), (4, 12, 300, 112, False), (4, 11, 385, 336, True), (1, 20, 640, 16, False)])
def test_forms_are_exact(T, C, A, S, extreme):
    rng = np.random.default_rng(A * 1000 + S)
    volt = rng.integers(-128, 128, size=(T, C, A, S, 2)).astype(np.int8)
    if extreme:
        volt[:, :, ::3] = -128
        volt[:, :, 1::3, :, 1] = 127
    vis, autos = blink.correlate(torch.from_numpy(volt).to("cuda:0"), autos=True)
    vis, autos = vis.cpu().numpy(), autos.cpu().numpy()
    a1, a2 = np.triu_indices(A, 1)
    for t in range(T):
        for c in range(C):
            x = volt[t, c].astype(np.float64)              # sums below 2^53: exact
            r, q = x[..., 0], x[..., 1]
            re, im = r @ r.T + q @ q.T, q @ r.T - r @ q.T
            assert np.array_equal(vis[t, c].real, re[a1, a2].astype(np.float32)), (t, c)
            assert np.array_equal(vis[t, c].imag, im[a1, a2].astype(np.float32)), (t, c)
            assert np.array_equal(autos[t, c], np.diag(re).astype(np.float32)), (t, c)


def test_more_spectra_than_one_launch():
    C = (1 << 22) + 37
    g = torch.Generator(device="cuda:0").manual_seed(5)
    volt = torch.randint(-128, 128, (1, C, 2, 16, 2), generator=g, device="cuda:0", dtype=torch.int8)
    vis, autos = blink.correlate(volt, autos=True)
    for c0 in range(0, C, 1 << 20):
        x = volt[0, c0:c0 + (1 << 20)].int()
        r, q = x[..., 0], x[..., 1]
        re = (r[:, 0] * r[:, 1] + q[:, 0] * q[:, 1]).sum(1).float()
        im = (q[:, 0] * r[:, 1] - r[:, 0] * q[:, 1]).sum(1).float()
        part = torch.view_as_real(vis[0, c0:c0 + (1 << 20), 0])
        assert torch.equal(part[:, 0], re) and torch.equal(part[:, 1], im)
        assert torch.equal(autos[0, c0:c0 + (1 << 20)], (r * r + q * q).sum(2).float())
