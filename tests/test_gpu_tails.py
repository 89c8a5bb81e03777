"""The small levels' single launches (pyramid tail, blend tail), of one frame and of a batch, against
the level-by-level passes that the same job takes in a batch whose other jobs are large: every
stored band, seam-weight plane, collapse level and the panorama, bit for bit (all round the same
expressions)."""
import numpy as np
import pytest
import torch

import paper_1810_03988_amd as P
from helpers import gpu_available, random_partition

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]
DEV = "cuda"


def _large_jobs(storage):
    """Two one-camera jobs whose middle levels are past the single launches' limits on their own:
    4.9 million pixels at 3 levels for the blends, 1.8 million at 4 for the passes."""
    out = []
    for W, H, L in ((2400, 2048, 3), (1400, 1300, 4)):
        plan = P.Plan([(W, H)], [np.eye(3)], [np.full((H, W), 255, np.uint8)], W, H, L, storage=storage)
        out.append((plan, [torch.zeros((H, W, 3), dtype=torch.uint8, device=DEV)],
                    torch.empty((H, W, 3), dtype=torch.uint8, device=DEV)))
    return out


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
    for form in ("frame", "batch", "levels"):
        plan = P.Plan(sizes, Hs, masks, W, H, L, storage=storage, keep_r0=True, bind=False)
        ws = torch.full((plan.ws_bytes + 256,), 0xFF, dtype=torch.uint8, device=DEV)
        plan.bind(ws)
        if form == "frame":
            pano = plan.frame(frames)
        else:
            pano = torch.empty((H, W, 3), dtype=torch.uint8, device=DEV)
            large = _large_jobs(storage) if form == "levels" else []
            batch = P.Batch([plan] + [p for p, _, _ in large])
            batch.run([frames] + [f for _, f, _ in large], [pano] + [o for _, _, o in large])
        torch.cuda.synchronize()
        got.append((pano.cpu(), {k: v.cpu() for k, v in _views(plan).items()}))
    bits = torch.int32 if storage == "f32" else torch.int16
    for other in got[:2]:
        assert torch.equal(other[0], got[2][0])
        assert other[1].keys() == got[2][1].keys()
        for key, a in other[1].items():
            assert torch.equal(a.view(bits), got[2][1][key].view(bits)), key


@pytest.mark.parametrize("groups", [2, 3])
def test_groups_of_small_jobs(groups):
    """Jobs whose groups take deeper single launches than the whole batch does."""
    rng = np.random.default_rng(groups)
    jobs = []
    for W, H, L in ((900, 620, 5), (310, 205, 4), (640, 480, 6), (97, 66, 2), (1000, 800, 5)):
        A = np.eye(3)
        A[:2, 2] = 3.25, 2.5
        masks = random_partition(rng, 2, H, W, "cuts")
        plan = P.Plan([(W, H)] * 2, [np.eye(3), A], masks, W, H, L)
        jobs.append((plan, [torch.from_numpy(rng.integers(0, 256, (H, W, 3), dtype=np.uint8)).to(DEV) for _ in range(2)],
                     torch.empty((H, W, 3), dtype=torch.uint8, device=DEV)))
    want = [p.frame(f).clone() for p, f, _ in jobs]
    batch = P.Batch([p for p, _, _ in jobs])
    batch.set_groups(groups)
    for _ in range(3):
        for _, _, o in jobs:
            o.zero_()
        batch.run([f for _, f, _ in jobs], [o for _, _, o in jobs])
        torch.cuda.synchronize()
        for (_, _, o), w in zip(jobs, want):
            assert torch.equal(o, w)
