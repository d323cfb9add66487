"""GPU: the order of many long lists at once (more than 8,192 baselines and 32
timesteps), whose gathers have a launch of their own: bit for bit against the
sorted reference over the distributions that reach the bucket ranking, the heavy
buckets and the radix passes, and with delays and re-projected baselines against
the same call in blocks of few timesteps."""
import numpy as np
import pytest
import torch

import paper_2405_13478_amd as blink

from test_gpu_sort import test_order_is_the_sorted_one as _check_order

pytestmark = pytest.mark.gpu
C_LIGHT = 299792458.0


@pytest.mark.parametrize("n_bl,n_time,n_chan,kind", [
    (8193, 40, 1, "uniform"), (8193, 40, 1, "equal"), (8193, 33, 2, "ulp"), (12000, 36, 1, "skewed"), (12000, 36, 1, "huge"),
    (12000, 40, 1, "equal"), (32768, 33, 1, "regular")])
def test_split_order_is_the_sorted_one(n_bl, n_time, n_chan, kind):
    _check_order(n_bl, n_time, n_chan, kind)


@pytest.mark.parametrize("n_ant,reproject,cable", [(129, False, True), (129, True, False), (200, True, True)])
def test_split_equals_blocks_of_few_timesteps(n_ant, reproject, cable):
    T, C, N = 40, 2, 64
    rng = np.random.default_rng(n_ant)
    a1, a2 = (x.astype(np.int32) for x in np.triu_indices(n_ant, 1))
    B = len(a1)
    assert B > 8192
    uvw = rng.uniform(-25, 25, (T, B, 3))
    uvw[:, ::5, 0] = np.rint(uvw[:, ::5, 0])              # ties
    uvw[:, ::5, 1:] = 0.0
    flags = (rng.random((T, B)) < 0.05).astype(np.uint8)
    flags[7] = 1                                          # no usable baseline
    vis = (rng.standard_normal((T, C, B)) + 1j * rng.standard_normal((T, C, B))).astype(np.complex64)
    to = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")    # noqa: E731
    kw = dict(grid_n=N, pixscale=C_LIGHT / (100e6 * N), ant1=to(a1), ant2=to(a2), phase_lm=(0.2, -0.3),
              reproject=reproject, cable_m=to(rng.uniform(0, 500, n_ant)) if cable else None)
    freq = to(np.array([90e6, 100e6]))
    whole = blink.grid(to(vis), to(uvw), freq, flags=to(flags), **kw)
    for t in range(0, T, 20):
        part = blink.grid(to(vis[t:t + 20]), to(uvw[t:t + 20]), freq, flags=to(flags[t:t + 20]), **kw)
        for a, b in zip(whole, part):
            assert torch.equal(a[t * C:(t + 20) * C], b)
