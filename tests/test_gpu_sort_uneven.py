"""GPU: the order of lists whose u are spread unevenly, bit for bit (see
test_gpu_sort): one long baseline beside a core, several scales, linear and
regular arrays whose baselines share a few u, at the sizes of the sort's forms and
with many timesteps at once. "missed" puts the list where the samples are not, so
that the buckets between them reach the sorts of whole buckets and the radix
passes."""
import numpy as np
import pytest
import torch

import paper_2405_13478_amd as blink

import test_gpu_sort as ts

pytestmark = pytest.mark.gpu


def _u(kind, n, rng):
    u = rng.uniform(-30, 30, n)
    if kind == "far":
        u[n // 3] = 3e8
    elif kind == "core":
        u[rng.random(n) < 0.8] *= 1e-4
    elif kind == "scales":
        u = 30 * 10.0 ** rng.uniform(-12, 0, n) * np.sign(u)
    elif kind == "linear":
        u = np.zeros(n)
    elif kind == "cylinders":
        u = rng.integers(-3, 4, n) * 7.5
    elif kind == "missed":
        threads = 256 if n <= 1024 else 1024
        rest = np.ones(n, bool)
        rest[np.arange(threads) * n // threads] = False
        u[rest] = 3.25 + 1e-9 * rng.integers(0, 3, rest.sum())
    return u


@pytest.mark.parametrize("n_bl,n_time,n_chan,kind", [
    (200, 1, 1, "linear"), (300, 3, 1, "far"), (1000, 1, 1, "linear"), (1000, 2, 2, "missed"), (1024, 1, 1, "core"),
    (1025, 1, 1, "far"), (1500, 2, 1, "cylinders"), (3000, 1, 2, "scales"), (8000, 1, 1, "missed"), (8128, 1, 1, "cylinders"),
    (8192, 2, 1, "linear"), (8193, 40, 1, "far"), (9000, 1, 1, "core"), (10752, 1, 1, "missed"), (10753, 1, 1, "scales"),
    (12000, 36, 1, "missed"), (12000, 2, 1, "missed"), (20011, 1, 1, "far"), (32640, 2, 1, "cylinders"),
    (32640, 33, 1, "core"), (32768, 1, 1, "linear"), (32768, 1, 2, "scales"), (32768, 3, 1, "missed")])
def test_order_of_uneven_lists(n_bl, n_time, n_chan, kind, monkeypatch):
    monkeypatch.setattr(ts, "_u", _u)
    ts.test_order_is_the_sorted_one(n_bl, n_time, n_chan, kind)


def test_mostly_flagged_uneven_list():
    # most samples are unusable baselines
    rng = np.random.default_rng(9)
    B = 20000
    uvw = np.zeros((1, B, 3))
    uvw[0, :, 0], uvw[0, :, 1] = _u("far", B, rng), rng.uniform(-30, 30, B)
    flags = (rng.random((1, B)) < 0.95).astype(np.uint8)
    vis = (rng.standard_normal((1, 1, B)) + 1j * rng.standard_normal((1, 1, B))).astype(np.complex64)
    freq = np.array([100e6])
    pix = ts.C_LIGHT / (100e6 * ts.N)
    to = lambda x: torch.from_numpy(x).to("cuda:0")    # noqa: E731
    g, counts, _, _ = blink.grid(to(vis), to(uvw), to(freq), grid_n=ts.N, pixscale=pix, flags=to(flags))
    ref, rc, _ = ts._reference(vis, uvw, freq, flags, pix)
    assert np.array_equal(counts.cpu().numpy(), rc)
    assert np.array_equal(torch.view_as_real(g).cpu().numpy(), ref)
