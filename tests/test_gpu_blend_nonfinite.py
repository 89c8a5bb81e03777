"""An infinite or undefined band sample reaches its own pixel of the blend and no other: the same
blend with a finite sample in its place has the same bits everywhere else.  Samples at the ends of
windows that begin and end inside a thread's four pixels, at a window's first sample, in the
level-by-level blend (R kept in the band's memory) and in that of all levels at once."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1810_03988_amd.stitch import StitchLevels, check, image_hwc, level_dims, levels_struct, lib
from helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]
DEV = "cuda"


@pytest.mark.parametrize("dt", [torch.float32, torch.float16])
@pytest.mark.parametrize("L, by_level", [(1, True), (2, True), (2, False), (3, False)])
@pytest.mark.parametrize("x0, width, at", [(1, 30, 0), (3, 9, 8), (2, 2, 1), (17, 33, 32), (6, 20, 0)])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_a_sample_reaches_its_own_pixel(x0, width, at, L, by_level, dt, value):
    W, H, y0, height, row = 70, 40, 3, 30, 0 if at == 0 else 17
    rng = np.random.default_rng(x0 * width)
    dims = level_dims(H, W, L)
    bands = [[torch.from_numpy(rng.normal(0.3, 0.2, (3, *d))).to(DEV).to(dt) for d in dims] for _ in range(2)]
    bands[1][0] = bands[1][0][:, y0:y0 + height, x0:x0 + width].contiguous()
    wts = [[torch.from_numpy(rng.uniform(0.1, 0.9, (1, *d))).to(DEV).to(dt) for d in dims] for _ in range(2)]
    wts[1][0] = torch.from_numpy(rng.integers(1, 256, (1, H, W), dtype=np.uint8)).to(DEV)
    borg = [[(0, 0)] * L, [(x0, y0)] + [(0, 0)] * (L - 1)]
    zeros = [(0, 0)] * L

    def blend(sample):
        mine = [[b.clone() for b in c] for c in bands]
        mine[1][0][1, row, at] = sample
        r = mine[0] if by_level else [torch.empty((3, *d), dtype=dt, device=DEV) for d in dims]
        pano = torch.empty((H, W, 3), dtype=torch.uint8, device=DEV)
        bs = (StitchLevels * 2)(*[levels_struct(b, org, W, H) for b, org in zip(mine, borg)])
        ws = (StitchLevels * 2)(*[levels_struct(w, zeros, W, H) for w in wts])
        n = lib().stitch_blend_workspace_bytes(2, L)
        buf = torch.empty(n + 256, dtype=torch.uint8, device=DEV)
        check(lib().stitch_blend(2, bs, ws, ctypes.byref(image_hwc(pano)), ctypes.byref(levels_struct(r, zeros, W, H)),
                                 (buf.data_ptr() + 255) // 256 * 256, n, torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        return r, pano

    (rf, pf), (rn, pn) = blend(0.25), blend(value)
    own = torch.zeros((3, H, W), dtype=torch.bool, device=DEV)
    own[1, y0 + row, x0 + at] = True
    assert not torch.isfinite(rn[0][own]).any()
    assert torch.equal(rn[0][~own], rf[0][~own])
    for k in range(1, L):
        assert torch.equal(rn[k], rf[k]), k
    assert torch.equal(pn[~own.any(0)], pf[~own.any(0)])
