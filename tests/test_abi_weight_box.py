"""The planner's bounding box of a camera's seam weights (its level-0 band) on sparse maps whose
first and last weights fall anywhere in a row: every width 3 .. 40 (the eight-byte scan's
remainders), empty first and last rows, single samples, against a numpy search."""
import numpy as np
import pytest

import paper_1810_03988_amd as P


@pytest.mark.parametrize("w", list(range(3, 41)))
def test_band_is_the_bounding_box_of_the_weights(w):
    rng = np.random.default_rng(w)
    for trial in range(6):
        h = int(rng.integers(3, 20))
        m = np.zeros((h, w), np.uint8)
        for _ in range(int(rng.integers(1, 4))):
            y0, x0 = int(rng.integers(0, h)), int(rng.integers(0, w))
            m[y0:y0 + int(rng.integers(1, 4)), x0:x0 + int(rng.integers(1, 1 + w // 2))] = int(rng.integers(1, 256))
        plan = P.Plan([(w, h)] * 2, [np.eye(3)] * 2, [m, 255 - m], w, h, 1, device="cpu", bind=False)
        for cam, a in enumerate((m, 255 - m)):
            ys, xs = np.nonzero(a)
            want = (xs.min(), ys.min(), xs.max() - xs.min() + 1, ys.max() - ys.min() + 1) if len(xs) else (0, 0, 0, 0)
            assert plan.regions(cam, 0)[1] == want, (w, trial, cam)
