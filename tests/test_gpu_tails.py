"""The small levels' single launches (pyramid tail, blend tail) against the level-by-level passes
that a batch of the same job takes: every stored band, seam-weight plane, collapse level and the
panorama, bit for bit (both sides round the same expressions)."""
import numpy as np
import pytest
import torch

import paper_1810_03988_amd as P
from helpers import gpu_available, random_partition

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]
DEV = "cuda"


def _views(plan):
    out = {}
    for k in range(plan.levels):
        out["r", 0, k] = plan.view("r", 0, k)[0]
        for i in range(plan.n):
            out["lap", i, k] = plan.view("lap", i, k)[0]
            if k >= 1:
                out["mask", i, k] = plan.view("mask", i, k)[0]
    return {key: v.clone().contiguous() for key, v in out.items() if v is not None}


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("n, W, H, L", [
    (2, 64, 16, 2),        # one blend tile exactly; no pyramid tail
    (2, 65, 17, 3),        # blend tiles one sample over, two steps
    (3, 256, 128, 4),      # pyramid tail of two levels, whole tiles
    (3, 257, 131, 5),      # three levels, remainders of one and two samples
    (2, 33, 34, 5),        # the top level 3x3
    (2, 1021, 66, 5),      # wide and low
    (5, 509, 389, 6),      # a level pass below the tail, a blend above it
    (9, 130, 258, 4),
])
def test_tails_equal_the_level_passes(n, W, H, L, storage):
    rng = np.random.default_rng(1000 * L + W)
    sizes, Hs, frames = [], [], []
    for i in range(n):
        fw, fh = int(rng.integers(20, max(24, W))), int(rng.integers(12, max(16, H)))
        A = np.eye(3) + rng.normal(0, [[0.05, 0.05, 0], [0.05, 0.05, 0], [2e-4, 2e-4, 0]])
        A[0, 2] = rng.uniform(-8, max(W - fw, 0) + 8)
        A[1, 2] = rng.uniform(-8, max(H - fh, 0) + 8)
        if i == 0:
            A[:2, 2] = 0.5                  # the canvas's first corner; the last camera its last one
        if i == n - 1:
            A[:2, 2] = W - fw, H - fh
        sizes.append((fw, fh))
        Hs.append(A)
        frames.append(torch.from_numpy(rng.integers(0, 256, (fh, fw, 3), dtype=np.uint8)).to(DEV))
    masks = random_partition(rng, n, H, W, "noise" if n % 2 else "cuts")
    got = []
    for batched in (False, True):
        plan = P.Plan(sizes, Hs, masks, W, H, L, storage=storage, keep_r0=True, bind=False)
        ws = torch.full((plan.ws_bytes + 256,), 0xFF, dtype=torch.uint8, device=DEV)
        plan.bind(ws)
        if batched:
            pano = torch.empty((H, W, 3), dtype=torch.uint8, device=DEV)
            batch = P.Batch([plan])
            batch.run([frames], [pano])
        else:
            pano = plan.frame(frames)
        torch.cuda.synchronize()
        got.append((pano.cpu(), {k: v.cpu() for k, v in _views(plan).items()}))
    assert torch.equal(got[0][0], got[1][0])
    assert got[0][1].keys() == got[1][1].keys()
    for key, a in got[0][1].items():
        b = got[1][1][key]
        bits = torch.int32 if storage == "f32" else torch.int16
        assert torch.equal(a.view(bits), b.view(bits)), key
