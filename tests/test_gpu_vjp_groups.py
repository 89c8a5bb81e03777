"""The float-frame forward and its vector-Jacobian product where their launches split: more
cameras than one launch takes (two and three groups, the last one short), seam weights whose
rows all differ or all agree, tiles that end inside and outside a camera's region, direct terms
on some cameras, and a frame seen so steeply that the gather falls back to its wider search.
Against the FP64 oracle: FP32 outputs to 1e-6 (the rounding of the result, 2^-24, with room for
the norm's spread), the FP64 map sums to 1e-9."""
import numpy as np
import pytest
import torch

import oracle as o
import paper_1810_03988_amd as P
from helpers import gpu_available, random_partition

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]
DEV = "cuda"


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) / max(np.linalg.norm(b), 1e-300))


@pytest.mark.parametrize("n, W, H, L, kind, steep", [
    (2, 131, 67, 3, "cuts", False),      # one group
    (9, 203, 117, 3, "noise", False),    # two groups: eight and one
    (17, 150, 90, 2, "cuts", False),     # three groups
    (10, 97, 65, 1, "noise", False),     # a single level, two groups
    (3, 160, 100, 3, "cuts", True),      # depth varies over a factor of two within a pixel's square
])
def test_groups_match_the_oracle(n, W, H, L, kind, steep):
    rng = np.random.default_rng(100 * n + L)
    frames, Hs, sizes = [], [], []
    for i in range(n):
        fw, fh = int(rng.integers(33, 70)), int(rng.integers(20, 60))
        A = np.eye(3) + rng.normal(0, [[0.04, 0.04, 0], [0.04, 0.04, 0], [3e-4, 3e-4, 0]])
        A[0, 2] = rng.uniform(-8, W - fw + 8)
        A[1, 2] = rng.uniform(-8, H - fh + 8)
        if steep and i == 1:
            # depth 1 + 1.25 (x + 1) over a 7-sample frame: 1 to 3.5 within the first pixel's square
            fw, fh = 7, 5
            A = np.array([[12.0, 0.0, 14.0], [0.0, 6.0, 10.0], [1.25, 0.0, 2.25]])
        sizes.append((fw, fh))
        frames.append(rng.random((3, fh, fw)).astype(np.float32))
        Hs.append(A)
    masks = random_partition(rng, n, H, W, kind)
    plan = P.Plan(sizes, Hs, masks, W, H, L, bind=False)
    fo = o.FrameVjpOracle([f.astype(np.float64) for f in frames], Hs, masks, W, H, L)
    fd = [torch.from_numpy(f).to(DEV) for f in frames]
    want = fo.forward()
    assert np.max(np.abs(plan.forward_f32(fd).cpu().numpy() - want)) <= 1e-6
    u = rng.normal(size=(3, H, W)).astype(np.float32)
    direct = [rng.normal(size=(3, H, W)).astype(np.float32) if i % 3 == 0 else None for i in range(n)]
    for dg in (None, direct):
        d_frames, d_M = plan.backward(fd, torch.from_numpy(u).to(DEV),
                                      None if dg is None else [None if x is None else torch.from_numpy(x).to(DEV)
                                                               for x in dg])
        wf, wm = fo.vjp(u.astype(np.float64), None if dg is None else [None if x is None else x.astype(np.float64)
                                                                      for x in dg])
        for i in range(n):
            assert _rel(d_frames[i].cpu().numpy(), wf[i]) <= 1e-6, i
            assert _rel(d_M[i], wm[i]) <= 1e-9, i
