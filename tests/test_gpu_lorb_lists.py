"""L-ORB detection by lists: tiles with no corner, with a few, and with many times a block's threads
near one (noise and dense dots at low thresholds, every test passing at 0), the extreme
thresholds, areas that end about a tile's edge -- points, responses and descriptors equal to the
oracle's."""
import numpy as np
import pytest

from helpers import gpu_available
from test_gpu_lorb import _check

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]


def _image(kind, rng, h, w):
    if kind == "noise":
        g = rng.integers(0, 256, (h, w))
    elif kind == "binary":
        g = 255 * (rng.random((h, w)) < 0.08)
    elif kind == "dots":
        g = np.full((h, w), 30)
        g[::4, ::4] = 220
        g[2::4, 2::4] = 10
    else:                                       # one corner, the rest flat
        g = np.full((h, w), 90)
        g[h // 2, w // 2] = 250
    return np.repeat(g.astype(np.uint8)[..., None], 3, axis=2)


@pytest.mark.parametrize("kind, tf", [("noise", 1), ("noise", 120), ("binary", 20), ("binary", 254), ("dots", 5),
                                      ("dots", 0), ("single", 60)])
@pytest.mark.parametrize("aw, ah", [(64, 16), (65, 17), (127, 31)])
def test_lists(kind, tf, aw, ah):
    rng = np.random.default_rng(tf + aw)
    frame = _image(kind, rng, ah + 40, aw + 44)
    _check(frame, [(20, 18, aw, ah), (0, 0, aw + 44, ah + 40)], tf=tf, t=-(1 << 60) if kind == "dots" else 0, n=3000,
           nd=96)
