"""GPU: the per-timestep order of the baselines, bit for bit.

With natural weighting a grid cell is the FP32 sum of its direct entries and
then of its mirrored ones, each in sorted order (by u, ties by baseline), so the
bits of blink_grid show the order. The reference adds the same FP32 values in
the order of a numpy sort; nothing is compared with a tolerance. Sizes sit at
the edges of the sort's forms (one word or several of counts a thread, 8 or 32
baselines a thread, lists above one workgroup's); the distributions reach the
bucket ranking, its tie resolution and the radix passes."""
import numpy as np
import pytest
import torch

import paper_2405_13478_amd as blink

pytestmark = pytest.mark.gpu
C_LIGHT = 299792458.0
N = 64


def _u(kind, n, rng):
    u = rng.uniform(-30, 30, n)
    if kind == "equal":
        u[:] = 3.25
    elif kind == "zeros":
        u = np.where(rng.random(n) < 0.5, 0.0, -0.0)
    elif kind == "regular":                       # a regular array: few distinct values
        u = rng.integers(-15, 16, n) * 1.75
    elif kind == "pairs":                         # each value twice or so: ties within small buckets
        u = rng.integers(0, max(1, n // 2), n) * (50.0 / max(1, n)) - 12.0
    elif kind == "ulp":                           # neighbouring doubles among spread ones
        k = rng.integers(0, n, max(1, n // 20))
        u[k] = u[(k + 1) % n] * (1 + 2.0 ** -52 * rng.integers(0, 3, k.size))
    elif kind == "skewed":                        # three quarters of the list in 1e-7 of the range
        u[: 3 * n // 4] *= 1e-7
    elif kind == "huge":
        u[::7] *= 1e290
        u[1::11] = np.inf
        u[2::13] = np.nan
    return u


def _reference(vis, uvw, freq, flags, pix):
    T, C, B = vis.shape
    grid = np.zeros((T * C, N, N, 2), np.float32)
    counts = np.zeros((T * C, N, N), np.int32)
    dropped = np.zeros(T * C, np.int64)
    for t in range(T):
        u, v = uvw[t, :, 0], uvw[t, :, 1]
        flagged = flags[t] != 0
        usable = ~flagged & np.isfinite(u) & np.isfinite(v)
        bits = u.view(np.uint64)                  # -0.0 before +0.0, as the order's keys have them
        key = np.where(bits >> np.uint64(63) != 0, ~bits, bits | np.uint64(1 << 63))
        idx = np.flatnonzero(usable)
        idx = idx[np.lexsort((idx, key[idx]))]
        for c in range(C):
            s = (freq[c] * (np.float64(N) * pix)) / C_LIGHT
            with np.errstate(over="ignore"):
                iu, iv = np.rint(u[idx] * s), np.rint(v[idx] * s)
            keep = (np.abs(iu) < N // 2) & (np.abs(iv) < N // 2)
            k, ku, kv = idx[keep], iu[keep].astype(int), iv[keep].astype(int)
            img = t * C + c
            val = np.stack([vis[t, c, k].real, vis[t, c, k].imag], -1)
            np.add.at(grid[img], (kv % N, ku % N), val)
            np.add.at(grid[img], (-kv % N, -ku % N), val * np.float32([1, -1]))
            np.add.at(counts[img], (kv % N, ku % N), 1)
            np.add.at(counts[img], (-kv % N, -ku % N), 1)
            dropped[img] = (~flagged).sum() - keep.sum()
    return grid, counts, dropped


@pytest.mark.parametrize("n_bl,n_time,n_chan,kind", [
    (1, 1, 1, "uniform"), (63, 2, 1, "pairs"), (1024, 1, 1, "uniform"), (1025, 3, 1, "ulp"), (2049, 2, 1, "uniform"),
    (4097, 1, 2, "ulp"), (8191, 1, 1, "uniform"), (8192, 300, 1, "uniform"), (8192, 1, 2, "equal"),
    (8193, 1, 1, "uniform"), (20011, 1, 1, "ulp"), (32767, 2, 2, "uniform"), (32768, 1, 1, "pairs"),
    (32768, 1, 1, "equal"), (32769, 1, 1, "uniform"),
    (700, 1, 1, "zeros"), (700, 2, 2, "huge"), (8000, 1, 1, "huge"), (8000, 2, 1, "regular"), (8000, 1, 1, "skewed"),
    (8000, 1, 1, "pairs"), (30000, 1, 1, "regular"), (30000, 1, 2, "skewed"), (30000, 1, 1, "huge")])
def test_order_is_the_sorted_one(n_bl, n_time, n_chan, kind):
    rng = np.random.default_rng(n_bl * 31 + n_chan)
    uvw = np.zeros((n_time, n_bl, 3))
    for t in range(n_time):
        uvw[t, :, 0] = _u(kind, n_bl, rng)
        uvw[t, :, 1] = rng.uniform(-30, 30, n_bl)
    flags = (rng.random((n_time, n_bl)) < 0.07).astype(np.uint8)
    if n_time > 2:
        flags[1] = 1                              # a timestep without usable baselines
    vis = (rng.standard_normal((n_time, n_chan, n_bl)) + 1j * rng.standard_normal((n_time, n_chan, n_bl))).astype(
        np.complex64)
    freq = np.linspace(100e6, 110e6, n_chan)
    pix = C_LIGHT / (100e6 * N)                   # about one cell a metre
    dev = torch.device("cuda:0")
    to = lambda x: torch.from_numpy(x).to(dev)    # noqa: E731
    g, counts, w, dropped = blink.grid(to(vis), to(uvw), to(freq), grid_n=N, pixscale=pix, flags=to(flags))
    ref, rc, rd = _reference(vis, uvw, freq, flags, pix)
    assert np.array_equal(counts.cpu().numpy(), rc)
    assert np.array_equal(dropped.cpu().numpy(), rd)
    assert np.array_equal(w.cpu().numpy(), rc.sum((1, 2)))
    assert np.array_equal(torch.view_as_real(g).cpu().numpy(), ref)
