"""GPU: the adjoint's half-length passes against the FP64 oracle: every first
radix they are built for, cutouts with and without the empty middle half (M up to
and above N/2, not a multiple of the wavefront), columns of one and of several
gather steps, many baselines on u = 0 (their two rows lie in different halves),
flags, gains, and both weightings. Bound: the repository's per-image FP32 one."""
import numpy as np
import pytest
import torch

import oracle
import paper_2405_13478_amd as blink

from _gpu_util import REL_L2_FP32, device, rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,M,n_ant,uniform,gains,on_axis", [
    (32, 16, 12, False, True, False), (32, 32, 20, True, False, True), (64, 30, 16, True, True, False),
    (128, 128, 40, False, False, True), (128, 64, 33, True, True, True), (256, 134, 64, False, True, False),
    (512, 256, 24, True, False, False), (512, 400, 60, False, True, True), (1024, 512, 48, True, True, True),
    (2048, 1024, 20, False, True, False)])
def test_adjoint_half_length_passes(N, M, n_ant, uniform, gains, on_axis):
    rng = np.random.default_rng(N + M)
    a1, a2 = (x.astype(np.int32) for x in np.triu_indices(n_ant, 1))
    B = len(a1)
    u = rng.uniform(-0.4 * N, 0.4 * N, B)
    if on_axis:                                   # longer than four gather steps, or all there is
        u[: max(B // 2, min(B, 300))] = 0.0
    uvw = np.zeros((1, B, 3))
    uvw[0, :, 0], uvw[0, :, 1] = u, rng.uniform(-0.55 * N, 0.55 * N, B)
    flags = (rng.random((1, B)) < 0.05).astype(np.uint8)
    pix, freq = 1.0 / N, np.array([oracle.C_LIGHT])       # one cell a metre
    vis = (rng.standard_normal((1, 1, B)) + 1j * rng.standard_normal((1, 1, B))).astype(np.complex64)
    g = (1 + 0.1 * rng.standard_normal(n_ant) + 0.1j * rng.standard_normal(n_ant)).astype(np.complex64)
    gbar = rng.standard_normal((1, M, M)).astype(np.float32)
    to = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(device())    # noqa: E731
    kw = dict(gains=to(g), ant1=to(a1), ant2=to(a2)) if gains else {}
    vg, gg = blink.degrid_adjoint(to(gbar), to(vis), to(uvw), to(freq), grid_n=N, pixscale=pix, out_n=M,
                                  weighting=int(uniform), flags=to(flags), **kw)
    rv, rg = oracle.adjoint_batch(gbar.astype(np.float64), vis, uvw, freq, N, pix, int(uniform), 1, flags,
                                  g if gains else None, a1, a2)
    assert rel_l2(vg.cpu().numpy().view(np.float32), np.ascontiguousarray(rv).view(np.float64)) <= REL_L2_FP32
    assert np.array_equal(vg.cpu().numpy()[0, 0] == 0, rv[0, 0] == 0)        # flagged and dropped ones
    if gains:
        assert rel_l2(gg.cpu().numpy().view(np.float32), np.ascontiguousarray(rg).view(np.float64)) <= REL_L2_FP32
