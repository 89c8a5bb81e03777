"""PROSAC over more matches than the ranking stages at once (16384): one key over it, within a second
stage, one over two, with many equal distances and unmatched queries on both sides of a stage's end;
samples, counts and inliers equal the oracle's exactly."""
import numpy as np
import pytest

from helpers import gpu_available
from test_gpu_register import _H, _check_prosac

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("n, distances", [(16385, 5), (20001, 40000), (32769, 300)])
def test_ranking_in_stages(n, distances):
    rng = np.random.default_rng(n)
    pa = rng.integers(0, 3000, (n, 2))
    v = np.concatenate([pa, np.ones((n, 1))], 1) @ _H().T
    pb = np.rint(v[:, :2] / v[:, 2:]).astype(np.int64)
    wrong = rng.random(n) < 0.3
    pb[wrong] = rng.integers(0, 3000, (int(wrong.sum()), 2))
    match = rng.permutation(n)                    # query i's reference is match[i]
    ref = np.empty_like(pb)
    ref[match] = pb
    match[rng.choice(n, n // 7, replace=False)] = -1
    match[16380:16388] = -1
    _check_prosac(pa, ref, match, rng.integers(0, distances, n), n, rng.random((24, 4)))
