"""The level-by-level blend, four pixels a thread: windows that begin and end inside a thread's four
pixels or are narrower than them, byte and sample weights, widths about a quad and a tile,
panoramas at odd pitches -- against the blend of all levels at once, which reads every pixel on its
own, bit for bit (the same products in the same order)."""
import ctypes

import numpy as np
import pytest
import torch

import paper_1810_03988_amd as P
from paper_1810_03988_amd.stitch import HWC, U8, StitchImage, StitchLevels, check, level_dims, levels_struct, lib
from helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]
DEV = "cuda"


@pytest.mark.parametrize("dt", [torch.float32, torch.float16])
@pytest.mark.parametrize("W, H, L, pitch, at", [
    (64, 16, 2, 192, 0), (65, 17, 3, 195, 1), (67, 33, 2, 208, 3), (130, 50, 4, 391, 2), (9, 40, 2, 27, 0),
])
def test_windows_and_pitches(W, H, L, pitch, at, dt):
    rng = np.random.default_rng(W * L)
    dims = level_dims(H, W, L)
    bands, wts, borg, worg = [], [], [], []
    for i in range(3):
        b, w, bo, wo = [], [], [], []
        for k, (h, wd) in enumerate(dims):
            def window():
                if i == 0:
                    return 0, 0, wd, h
                x, y = int(rng.integers(0, wd)), int(rng.integers(0, h))
                return x, y, int(rng.integers(1, wd - x + 1)), int(rng.integers(1, h - y + 1))
            x, y, ww, hh = window()
            if i == 2:
                ww = min(ww, 3)                     # narrower than a quad
            b.append(torch.from_numpy(rng.normal(0.4, 0.3, (3, hh, ww))).to(DEV).to(dt))
            bo.append((x, y))
            x, y, ww, hh = window()
            byte = (i + k) % 2 == 0
            w.append(torch.from_numpy(rng.integers(0, 256, (1, hh, ww), dtype=np.uint8)).to(DEV) if byte else
                     torch.from_numpy(rng.random((1, hh, ww))).to(DEV).to(dt))
            wo.append((x, y))
        bands.append(b), wts.append(w), borg.append(bo), worg.append(wo)
    pano, rs = P.blend(bands, wts, W, H, band_origins=borg, weight_origins=worg)
    # R in camera 0's band memory: one level a launch
    zeros = [(0, 0)] * L
    inplace = [[x.clone() for x in bands[0]]] + bands[1:]
    bs = (StitchLevels * 3)(*[levels_struct(b, o, W, H) for b, o in zip(inplace, borg)])
    ws = (StitchLevels * 3)(*[levels_struct(w, o, W, H) for w, o in zip(wts, worg)])
    r = levels_struct(inplace[0], zeros, W, H)
    buf = torch.full((at + pitch * H + 16,), 7, dtype=torch.uint8, device=DEV)
    out = StitchImage(buf.data_ptr() + at, W, H, 3, U8, HWC, pitch, 0)
    n = lib().stitch_blend_workspace_bytes(3, L)
    wsp = torch.empty(n + 256, dtype=torch.uint8, device=DEV)
    check(lib().stitch_blend(3, bs, ws, ctypes.byref(out), ctypes.byref(r), (wsp.data_ptr() + 255) // 256 * 256, n,
                             torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    rows = torch.as_strided(buf, (H, pitch), (pitch, 1), at)
    assert torch.equal(rows[:, :3 * W].reshape(H, W, 3), pano)
    assert (rows[:-1, 3 * W:] == 7).all() and (buf[:at] == 7).all() and (buf[at + pitch * (H - 1) + 3 * W:] == 7).all()
    for k in range(L):
        assert torch.equal(inplace[0][k], rs[k]), k
