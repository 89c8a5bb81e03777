"""stitch_blend on weight planes up to the size it accepts (fewer than 2^31 elements, rows under 2^23):
weights in rows so far apart that the later ones lie past 2^32 bytes, against the same weights
packed, bit for bit."""
import pytest
import torch

import paper_1810_03988_amd as P
from helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]
DEV = "cuda"


@pytest.mark.parametrize("dt, H", [
    (torch.float32, 140),      # rows 129 and up start past 2^32 bytes
    (torch.float16, 254),      # the last row ends 2^24 elements below 2^31
    (torch.uint8, 254),
])
def test_weights_in_rows_far_apart(dt, H):
    W, pitch = 70, 2 ** 23 - 4
    gen = torch.Generator(device=DEV).manual_seed(H)
    store = torch.float16 if dt == torch.float16 else torch.float32
    band = torch.rand(3, H, W, device=DEV, generator=gen).to(store)
    w = torch.rand(1, H, W - 1, device=DEV, generator=gen)       # from column 1: quads across its edge
    w = (255 * w).to(dt) if dt == torch.uint8 else w.to(dt)
    far = torch.zeros((H, pitch), dtype=dt, device=DEV)
    far[:, :W - 1] = w[0]
    want, rw = P.blend([[band]], [[w]], W, H, weight_origins=[[(1, 0)]])
    got, rg = P.blend([[band]], [[far[None, :, :W - 1]]], W, H, weight_origins=[[(1, 0)]])
    torch.cuda.synchronize()
    assert want.max() > 200
    assert torch.equal(rg[0], rw[0])
    assert torch.equal(got, want)
