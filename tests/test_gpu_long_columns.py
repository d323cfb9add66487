"""GPU: uv grids and gradients of arrays whose baselines share a few u cells, so
that a column holds several hundred entries, direct ones, mirrored ones and those
of u = 0: more than a wavefront keeps in registers, with a last step partly
filled. Every size class of the gridding call's and the adjoint's columns, both
weightings, against the FP64 oracle; bound: the repository's per-image FP32 one."""
import numpy as np
import pytest
import torch

import oracle
import paper_2405_13478_amd as blink

from _gpu_util import REL_L2_FP32, device, rel_l2

pytestmark = pytest.mark.gpu


def _long(N, rng, n_ant=64):
    a1, a2 = (x.astype(np.int32) for x in np.triu_indices(n_ant, 1))
    B = len(a1)                                                   # 2,016 at 64 antennas
    uvw = np.zeros((1, B, 3))
    # u cells 0 (a third), N/4 and its mirror column, and some spread ones
    uvw[0, :, 0] = rng.choice([0, 0, N // 4, -(N // 4)], B)
    uvw[0, ::50, 0] = rng.integers(-(N // 2) + 1, N // 2, len(uvw[0, ::50]))
    uvw[0, :, 1] = rng.uniform(-0.55 * N, 0.55 * N, B)            # a few beyond the grid
    flags = (rng.random((1, B)) < 0.05).astype(np.uint8)
    vis = (rng.standard_normal((1, 1, B)) + 1j * rng.standard_normal((1, 1, B))).astype(np.complex64)
    return a1, a2, uvw, flags, vis


def _to(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to(device())


def _check_grid(uvw, flags, vis, N, uniform):
    freq, pix = np.array([oracle.C_LIGHT]), 1.0 / N               # one cell a metre
    g, c, w, d = blink.grid(_to(vis), _to(uvw), _to(freq), grid_n=N, pixscale=pix, weighting=uniform, flags=_to(flags))
    s = oracle.blink_oracle.uv_scale(freq[0], N, pix)
    iu, iv, keep = oracle.blink_oracle.cell_index(uvw[0, :, 0], uvw[0, :, 1], s, N, flags[0])
    S, cnt = oracle.blink_oracle.grid(vis[0, 0], iu, iv, keep, N)
    G, W = oracle.blink_oracle.weight(S, cnt, uniform)
    assert np.array_equal(c.cpu().numpy()[0], cnt)
    assert float(w[0]) == W and int(d[0]) == int(((flags[0] == 0) & ~keep).sum())
    assert rel_l2(g.cpu().numpy()[0].view(np.float32), np.ascontiguousarray(G).view(np.float64)) <= REL_L2_FP32


@pytest.mark.parametrize("uniform", [0, 1])
@pytest.mark.parametrize("N", [8, 12, 32, 128, 180, 256, 512, 1024, 2048, 4096])
def test_uv_grid_of_long_columns(N, uniform):
    rng = np.random.default_rng(N + uniform)
    _, _, uvw, flags, vis = _long(N, rng)
    _check_grid(uvw, flags, vis, N, uniform)


# many entries in a tile of columns, none of which is long: around u = 0, on one
# side of it and in the last columns that can hold any
@pytest.mark.parametrize("place,uniform", [("centre", 0), ("side", 1), ("edge", 0)])
@pytest.mark.parametrize("N", [1024, 2048, 4096])
def test_uv_grid_of_full_tiles(N, place, uniform):
    rng = np.random.default_rng(N)
    _, _, uvw, flags, vis = _long(N, rng)
    first = {"centre": -8, "side": 40, "edge": N // 2 - 16}[place]
    uvw[0, :, 0] = first + rng.integers(0, 16, uvw.shape[1])
    _check_grid(uvw, flags, vis, N, uniform)


@pytest.mark.parametrize("N,M,uniform,gains", [(32, 16, 0, True), (64, 64, 1, False), (128, 64, 0, False), (256, 128, 1, True),
                                               (512, 400, 0, True), (1024, 512, 0, False), (1024, 512, 1, True),
                                               (2048, 1024, 1, False)])
def test_gradients_of_long_columns(N, M, uniform, gains):
    rng = np.random.default_rng(N * 3 + M)
    a1, a2, uvw, flags, vis = _long(N, rng)
    freq, pix = np.array([oracle.C_LIGHT]), 1.0 / N
    g = (1 + 0.1 * rng.standard_normal(64) + 0.1j * rng.standard_normal(64)).astype(np.complex64)
    gbar = rng.standard_normal((1, M, M)).astype(np.float32)
    kw = dict(gains=_to(g), ant1=_to(a1), ant2=_to(a2)) if gains else {}
    vg, gg = blink.degrid_adjoint(_to(gbar), _to(vis), _to(uvw), _to(freq), grid_n=N, pixscale=pix, out_n=M,
                                  weighting=uniform, flags=_to(flags), **kw)
    rv, rg = oracle.adjoint_batch(gbar.astype(np.float64), vis, uvw, freq, N, pix, uniform, 1, flags,
                                  g if gains else None, a1, a2)
    assert rel_l2(vg.cpu().numpy().view(np.float32), np.ascontiguousarray(rv).view(np.float64)) <= REL_L2_FP32
    assert np.array_equal(vg.cpu().numpy()[0, 0] == 0, rv[0, 0] == 0)
    if gains:
        assert rel_l2(gg.cpu().numpy().view(np.float32), np.ascontiguousarray(rg).view(np.float64)) <= REL_L2_FP32
