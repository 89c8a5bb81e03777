"""Level 0 of stitch_pyramid where it is copied or converted on its own: rows that end inside a thread's
four samples or are narrower than them, at odd addresses and pitches, each source and storage type.
Copies are bit for bit; a byte is its product with FP32 1/255, rounded once to the storage type."""
import pytest
import torch

import paper_1810_03988_amd as P
from helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]
DEV = "cuda"
R255 = torch.tensor(1.0 / 255.0, dtype=torch.float32).double()


def _view(src, at, pitch):
    """src's values (C, H, W) in a buffer of their own, from element `at`, rows `pitch` apart."""
    C, H, W = src.shape
    buf = torch.zeros(at + C * H * pitch + W, dtype=src.dtype, device=DEV)
    v = torch.as_strided(buf, (C, H, W), (H * pitch, pitch, 1), at)
    v.copy_(src)
    return v


@pytest.mark.parametrize("w, h", [(3, 3), (4, 5), (7, 4), (255, 9), (256, 3), (257, 6), (1031, 17)])
@pytest.mark.parametrize("at, extra", [(0, 0), (1, 0), (3, 5)])
def test_copies_and_conversions(w, h, at, extra):
    gen = torch.Generator(device=DEV).manual_seed(w)
    for dt in (torch.float32, torch.float16):
        x = torch.randn(3, h, w, device=DEV, generator=gen).to(dt)
        got = P.pyramid(_view(x, at, w + extra), 1, "laplacian")[0]
        assert torch.equal(got, x), dt
        m = torch.arange(h * w, device=DEV).mul(37).remainder(256).to(torch.uint8).view(1, h, w)
        got = P.pyramid(_view(m, at, w + extra)[0], 1, "gaussian", dtype=dt)[0]
        assert torch.equal(got, (m.double() * R255.to(DEV)).to(dt)), dt
