"""stitch_pyramid, stitch_blend and stitch_warp where their launches divide: whole chains in one
launch, one level at a time where buffers overlap, level 0 formed from g0 or in place, rows shorter
than one wide read, rectangles at odd places, frames narrower than a tap pair's eight bytes.
Against the FP64 oracle on the rectangles (samples outside count 0): five FP32 sums of five
non-negative terms up to 1 a level lose at most 2^-22 a level, 2e-6 over six and their
differences; a warped sample takes six roundings of values up to 1, 1e-6.  Routes against each
other bit for bit."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as o
import paper_1810_03988_amd as P
from oracle import stitch_oracle as so
from paper_1810_03988_amd.stitch import StitchImage, check, image_chw, level_dims, levels_struct, lib
from helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]
DEV = "cuda"


def _rects(w, h, L, canvas, origin):
    return [(origin[0] >> k, origin[1] >> k,
             min(-(-(origin[0] + w) // (1 << k)), -(-canvas[0] // (1 << k))) - (origin[0] >> k),
             min(-(-(origin[1] + h) // (1 << k)), -(-canvas[1] // (1 << k))) - (origin[1] >> k)) for k in range(L)]


def _pyramid(g0, outs, rects, kind, canvas):
    """The C entry point on given buffers."""
    C, h, w = g0.shape
    src = StitchImage(g0.data_ptr(), w, h, C, {torch.uint8: 0, torch.float32: image_chw(outs[0]).dtype,
                                               torch.float16: image_chw(outs[0]).dtype}[g0.dtype], 1,
                      g0.stride(1) * g0.element_size(), g0.stride(0) * g0.element_size())
    s = levels_struct(outs, [(x, y) for x, y, _, _ in rects], *canvas)
    n = lib().stitch_pyramid_workspace_bytes(len(outs))
    ws = torch.empty(n + 256, dtype=torch.uint8, device=DEV)
    check(lib().stitch_pyramid(ctypes.byref(src), kind, ctypes.byref(s), (ws.data_ptr() + 255) // 256 * 256, n,
                               torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()


def _want(g, rects, kind, canvas):
    """Pyramid of g (float64) placed on its rectangle, every level 0 outside its own."""
    W, H = canvas
    full, out = [], []
    for k, (x, y, w, h) in enumerate(rects):
        z = np.zeros((g.shape[0], *level_dims(H, W, len(rects))[k]))
        z[:, y:y + h, x:x + w] = g if k == 0 else so.reduce_full(full[-1])[:, y:y + h, x:x + w]
        full.append(z)
    for k, (x, y, w, h) in enumerate(rects):
        v = full[k]
        if kind == 1 and k + 1 < len(rects):
            v = v - so.expand_full(full[k + 1], *v.shape[1:])
        out.append(v[:, y:y + h, x:x + w])
    return out


@pytest.mark.parametrize("w, h, L, canvas, origin, ch", [
    (64, 32, 4, (64, 32), (0, 0), 3),          # one tile
    (65, 33, 4, (65, 33), (0, 0), 1),          # one sample over it
    (130, 97, 6, (130, 97), (0, 0), 3),        # five steps: two launches
    (5, 61, 3, (203, 99), (101, 17), 2),       # rows shorter than a wide read, odd origin
    (119, 7, 3, (121, 40), (2, 33), 3),        # ends at the canvas's right and bottom edge
    (1100, 960, 3, (1300, 1000), (37, 11), 3), # a level of its own launch
    (9, 9, 1, (40, 40), (3, 5), 3),
])
@pytest.mark.parametrize("kind", [0, 1])
def test_pyramid_routes(w, h, L, canvas, origin, ch, kind):
    rng = np.random.default_rng(w + L)
    img = rng.random((ch, h, w)).astype(np.float32)
    rects = _rects(w, h, L, canvas, origin)
    want = _want(img.astype(np.float64), rects, kind, canvas)
    for dt in (torch.float32, torch.float16):
        g0 = torch.from_numpy(img).to(DEV).to(dt)
        new = lambda: [torch.full((ch, rh, rw), float("nan"), dtype=dt, device=DEV) for _, _, rw, rh in rects]
        apart = new()
        _pyramid(g0, apart, rects, kind, canvas)
        inplace = new()
        inplace[0].copy_(g0)
        _pyramid(inplace[0], inplace, rects, kind, canvas)
        shared = new()
        src = g0.clone()
        if L > 1:                                # level 1 lies in g0's own memory
            shared[1] = src.view(-1)[:shared[1].numel()].view(shared[1].shape)
        _pyramid(src, shared, rects, kind, canvas)
        for k in range(L):
            if dt == torch.float32:
                assert np.max(np.abs(apart[k].cpu().numpy() - want[k])) <= 2e-6, k
            assert torch.equal(apart[k], inplace[k]), k
            assert torch.equal(apart[k], shared[k]), k


@pytest.mark.parametrize("w, h, L, canvas, origin", [
    (7, 40, 3, (90, 60), (11, 3)), (8, 40, 3, (90, 60), (0, 0)), (201, 77, 5, (260, 77), (33, 0)),
])
def test_byte_weights(w, h, L, canvas, origin):
    rng = np.random.default_rng(w)
    m = rng.integers(0, 256, (1, h, w), dtype=np.uint8)
    rects = _rects(w, h, L, canvas, origin)
    want = _want(m / 255.0, rects, 0, canvas)
    got = P.pyramid(torch.from_numpy(m[0]).to(DEV), L, "gaussian", canvas=canvas, origin=origin)
    half = P.pyramid(torch.from_numpy(m[0]).to(DEV), L, "gaussian", canvas=canvas, origin=origin, dtype=torch.float16)
    for k in range(L):
        assert np.max(np.abs(got[k].cpu().numpy() - want[k])) <= 2e-6, k
    assert torch.equal(half[0], (torch.from_numpy(m).to(DEV).double() / 255.0).half()) or \
        np.max(np.abs(half[0].double().cpu().numpy() - want[0])) <= 2.0 ** -11


@pytest.mark.parametrize("fw, fh", [(1, 4), (2, 3), (3, 1), (4, 5), (61, 18)])
def test_warp_of_narrow_frames(fw, fh):
    rng = np.random.default_rng(fw)
    src = rng.integers(0, 256, (fh, fw, 3), dtype=np.uint8)
    H = np.array([[1.9, 0.2, 4.3], [-0.1, 2.2, 3.7], [1e-3, -2e-3, 1.0]])
    W, Hh = 2 * fw + 21, 2 * fh + 18             # rows beyond a multiple of sixteen
    got = P.warp(torch.from_numpy(src).to(DEV), H, -3, -2, W, Hh).cpu().numpy()
    want = o.warp(src, o.hinv_spec(H), np.arange(-2, Hh - 2), np.arange(-3, W - 3))
    assert np.max(np.abs(got - want)) <= 1e-6


@pytest.mark.parametrize("W, H, L", [(64, 16, 2), (131, 66, 4), (700, 900, 5)])
def test_blend_with_r_in_the_bands_memory(W, H, L):
    rng = np.random.default_rng(W)
    dims = level_dims(H, W, L)
    bands = [torch.from_numpy(rng.normal(size=(3, *d)).astype(np.float32)).to(DEV) for d in dims]
    wts = [torch.from_numpy(rng.random((1, *d)).astype(np.float32)).to(DEV) for d in dims]
    pano, rs = P.blend([bands], [wts], W, H)
    inplace = [b.clone() for b in bands]
    out = torch.empty_like(pano)
    zeros = [(0, 0)] * L
    bs = levels_struct(inplace, zeros, W, H)
    wsx = levels_struct(wts, zeros, W, H)
    n = lib().stitch_blend_workspace_bytes(1, L)
    ws = torch.empty(n + 256, dtype=torch.uint8, device=DEV)
    from paper_1810_03988_amd.stitch import image_hwc
    check(lib().stitch_blend(1, ctypes.byref(bs), ctypes.byref(wsx), ctypes.byref(image_hwc(out)), ctypes.byref(bs),
                             (ws.data_ptr() + 255) // 256 * 256, n, torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert torch.equal(out, pano)
    for k in range(L):
        assert torch.equal(inplace[k], rs[k]), k
