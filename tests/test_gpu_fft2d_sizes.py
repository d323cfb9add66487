"""GPU: blink_fft2d at the sizes of the half-length passes (several vectors a
wavefront below 1024, two butterflies a lane at 2048) against a 64-bit
transform: one image and batches that leave the row pass a partly filled
workgroup, both signs, in place, and an output that starts 8 bytes off 16-byte
alignment (the column pass then takes its 8-byte form). The bound is 4 eps per
radix-2 level, log2(n^2) levels: an FFT's error grows by less than that."""
import numpy as np
import pytest
import torch

import paper_2405_13478_amd as blink

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,batch", [(128, 1), (128, 67), (256, 3), (256, 300), (512, 1), (512, 5), (1024, 2), (1024, 19),
                                     (2048, 1), (2048, 5)])
def test_fft2d_half_length_passes(n, batch):
    rng = np.random.default_rng(n + batch)
    x = (rng.standard_normal((batch, n, n)) + 1j * rng.standard_normal((batch, n, n))).astype(np.complex64)
    dev = torch.device("cuda:0")
    bound = 4 * np.finfo(np.float32).eps / 2 * 2 * np.log2(n)
    for sign in (1, -1):
        d = torch.from_numpy(x).to(dev)
        out = blink.fft2d(d, sign)
        assert torch.equal(torch.from_numpy(x).to(dev), d)          # the input is untouched
        pool = torch.empty(d.numel() + 1, dtype=torch.complex64, device=dev)
        odd = pool[1:].view(batch, n, n)
        assert odd.data_ptr() % 16 == 8
        blink.fft2d(d, sign, out=odd)
        blink.fft2d(d, sign, out=d)
        assert torch.equal(out, d)
        for i in {0, batch // 2, batch - 1}:
            ref = np.fft.ifft2(x[i].astype(np.complex128)) * n * n if sign > 0 else np.fft.fft2(x[i].astype(np.complex128))
            for got in (out[i], odd[i]):
                err = np.linalg.norm(got.cpu().numpy() - ref) / np.linalg.norm(ref)
                assert err <= bound, (sign, i, err, bound)
