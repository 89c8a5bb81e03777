"""Which launches a frame and a batch take: small levels share one each way, and the batch that
test_gpu_tails compares with takes every level of every job by itself.  FP16 pyramids of a chain
against the FP64 oracle: a stored level of values up to 1 is within 2^-12 of what was rounded, REDUCE
averages the error of the level before, a band adds its two levels' and its own rounding; FP32
arithmetic 2e-6 as in the stages' other tests."""
import numpy as np
import pytest
import torch

import paper_1810_03988_amd as P
from helpers import gpu_available, random_partition
from test_gpu_stage_routes import _rects, _want
from test_gpu_tails import _large_jobs

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]
DEV = "cuda"


def _job(n, W, H, L, storage):
    rng = np.random.default_rng(W)
    plan = P.Plan([(W, H)] * n, [np.eye(3)] * n, random_partition(rng, n, H, W, "cuts"), W, H, L, storage=storage)
    return (plan, [torch.zeros((H, W, 3), dtype=torch.uint8, device=DEV)] * n,
            torch.empty((H, W, 3), dtype=torch.uint8, device=DEV))


def _run(jobs):
    batch = P.Batch([p for p, _, _ in jobs])
    batch.set_timing(True)
    batch.run([f for _, f, _ in jobs], [o for _, _, o in jobs])
    torch.cuda.synchronize()
    return batch.read_timing()


@pytest.mark.parametrize("storage", ["f32", "f16"])
@pytest.mark.parametrize("n, W, H, L", [(3, 256, 128, 4), (2, 33, 34, 5), (5, 509, 389, 6)])
def test_levels_of_a_batch(n, W, H, L, storage):
    small = _run([_job(n, W, H, L, storage)])
    large = _run([_job(n, W, H, L, storage)] + _large_jobs(storage))
    top = max(L, 4)
    # by itself: pass 0, then what lies above the shared launch, then one; level 0's blend and what lies above
    assert sum(c for _, c in small.values()) < 2 * L - 1
    assert sum(c for _, c in large.values()) == (top - 1) + top, large
    assert all(c <= 1 for _, c in large.values()), large


@pytest.mark.parametrize("w, h, L, canvas, origin, ch", [
    (64, 32, 4, (64, 32), (0, 0), 3), (130, 97, 6, (130, 97), (0, 0), 3), (5, 61, 3, (203, 99), (101, 17), 2),
    (119, 7, 3, (121, 40), (2, 33), 3), (1100, 960, 3, (1300, 1000), (37, 11), 3),
])
def test_half_pyramids(w, h, L, canvas, origin, ch):
    rng = np.random.default_rng(w)
    img = torch.from_numpy(rng.random((ch, h, w))).half()
    byte = torch.from_numpy(rng.integers(0, 256, (h, w), dtype=np.uint8))
    rects = _rects(w, h, L, canvas, origin)
    e = lambda k: k * 2.0 ** -12                     # of Gaussian level k, level 0 given exactly
    kw = dict(canvas=canvas, origin=origin)
    for k, (g, want) in enumerate(zip(P.pyramid(img.to(DEV), L, "gaussian", **kw),
                                      _want(img.double().numpy(), rects, 0, canvas))):
        assert np.max(np.abs(g.double().cpu().numpy() - want)) <= e(k) + 2e-6, k
    for k, (g, want) in enumerate(zip(P.pyramid(img.to(DEV), L, "laplacian", **kw),
                                      _want(img.double().numpy(), rects, 1, canvas))):
        bound = e(k) + e(k + 1) + 2.0 ** -12 if k + 1 < L else e(k)
        assert np.max(np.abs(g.double().cpu().numpy() - want)) <= bound + 2e-6, k
    for k, (g, want) in enumerate(zip(P.pyramid(byte.to(DEV), L, "gaussian", dtype=torch.float16, **kw),
                                      _want(byte[None].double().numpy() / 255.0, rects, 0, canvas))):
        assert np.max(np.abs(g.double().cpu().numpy() - want)) <= e(k + 1) + 2e-6, k
