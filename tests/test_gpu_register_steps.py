"""Registration where its waves' steps end: match counts about the growth function's blocks of 64 and
the ranking's groups of 64 queries, equal distances, schedules past every growth step, a T_N too
small for the corrected quotient, searches over few and many T', reference counts about two
points a lane, tables about the eight read at once.  Samples, counts, inliers and matches equal
the oracle's exactly, the refit to the other prosac tests' tolerance."""
import numpy as np
import pytest

import paper_1810_03988_amd as P
from oracle import register_oracle as ro
from helpers import gpu_available
from test_gpu_register import _apply, _check_prosac, _descriptor_sets, _dev, _H

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


@pytest.mark.parametrize("M, T_N, nhyp", [
    (5, 200000.0, 70), (67, 200000.0, 130), (68, 40.0, 130), (69, 1e-280, 130), (132, 300.0, 400),
    (133, 200000.0, 200), (260, 2.0 ** 53, 64), (1030, 1000.0, 900),
])
def test_growth_ranking_and_search(M, T_N, nhyp):
    rng = np.random.default_rng(M)
    unmatched = M // 9
    n = M + unmatched
    pa = rng.integers(0, 700, (n, 2))
    pb = np.array([np.rint(_apply(_H(), p)) for p in pa]).astype(np.int64)
    wrong = rng.random(n) < 0.2
    pb[wrong] = rng.integers(0, 800, (int(wrong.sum()), 2))
    match = rng.permutation(n)                    # query i's reference is match[i]
    ref = np.empty_like(pb)
    ref[match] = pb
    dist = rng.integers(0, 6, n)                  # many ties
    match[rng.choice(n, unmatched, replace=False)] = -1
    _check_prosac(pa, ref, match, dist, n, rng.random((nhyp, 4)), T_N=T_N)


@pytest.mark.parametrize("na, nb, nd, tables", [(3, 1, 32, 1), (70, 63, 96, 7), (65, 65, 128, 8), (40, 129, 160, 9),
                                                (9, 300, 512, 16)])
def test_matching(na, nb, nd, tables):
    rng = np.random.default_rng(nd + tables)
    da, db = _descriptor_sets(rng, na, nb, nd)
    pos = rng.integers(0, nd, (tables, 6))
    want_idx, want_d = ro.lsh_match(da, db, pos, nd)
    m = P.Matcher(na, nb, nd, pos, nd)
    got_idx, got_d = m.run(_dev(da.view(np.int32)), _dev([na]), _dev(db.view(np.int32)), _dev([nb]))
    assert got_idx.tolist() == want_idx.tolist() and got_d.tolist() == want_d.tolist()
