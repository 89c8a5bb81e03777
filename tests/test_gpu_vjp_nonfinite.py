"""Non-finite frame samples and upstream gradients in the float-frame forward and its
vector-Jacobian product: they reach the results they have a share in, through every tap of every
operator, and no other.  The reference lists every tap (samples outside an array count 0, and so
does a product with a seam weight of 0).  Where its result is finite ours agrees as on finite
inputs (FP32 outputs to 1e-6 of the largest), and where it isn't, ours isn't; an infinity that
stays one (a sum with no opposite infinity and no NaN) keeps its sign."""
import numpy as np
import pytest
import torch

import oracle as o
import paper_1810_03988_amd as P
from oracle.stitch_oracle import expand_full, reduce_full
from helpers import gpu_available

pytestmark = [pytest.mark.gpu, pytest.mark.skipif(not gpu_available(), reason="needs a GPU")]
DEV = "cuda"
NAN, INF = float("nan"), float("inf")


def _mul(g, v):
    return np.where(g == 0.0, 0.0, g * v)


def _forward(fo):
    L = fo.L
    B = [0.0] * L
    for gm, f, M, c in zip(fo.gm, fo.frames, fo.M, fo.cells):
        g = [fo._warp(f, M, c)[0]]
        for _ in range(L - 1):
            g.append(reduce_full(g[-1]))
        for k in range(L):
            B[k] = B[k] + _mul(gm[k], g[k] - (expand_full(g[k + 1], *g[k].shape[1:]) if k + 1 < L else 0.0))
    R = B[-1]
    for k in range(L - 2, -1, -1):
        R = B[k] + expand_full(R, *B[k].shape[1:])
    return R


def _vjp(fo, u, direct):
    L = fo.L
    dR = [u]
    for _ in range(L - 1):
        dR.append(o.expand_T(dR[-1]))
    out = []
    for i, f in enumerate(fo.frames):
        dL = [_mul(fo.gm[i][k], dR[k]) for k in range(L)]
        g = dL[L - 1]
        for k in range(L - 1, 0, -1):
            g = (g if k == L - 1 else dL[k] + g) - o.expand_T(dL[k - 1])
            g = o.reduce_T(g, *fo.dims[k - 1])
        g = dL[0] + g if L > 1 else g
        if direct is not None:
            g = g + direct[i]
        out.append(fo._warp_T(f, fo.M[i], fo.cells[i], g)[0])
    return out


def _agree(got, want, what):
    got = got.astype(np.float64)
    fin = np.isfinite(want)
    bad = np.argwhere(np.isfinite(got) != fin)
    assert bad.size == 0, f"{what}: {len(bad)} samples differ in being finite, first {bad[0]}: {want[tuple(bad[0])]}"
    assert np.max(np.abs(got[fin] - want[fin]), initial=0.0) <= 1e-6 * max(1.0, np.max(np.abs(want[fin]), initial=0.0)), what
    inf = np.isinf(want)
    assert np.array_equal(got[inf], want[inf]), what
    assert fin.any() and not fin.all(), f"{what}: the case shows nothing"


def _shift(x, y):
    return np.array([[1.0, 0.0, x], [0.0, 1.0, y], [0.0, 0.0, 1.0]])


def _cuts(W, H, at):
    m = np.zeros((2, H, W), np.uint8)
    m[0, :, :at] = 255
    m[1, :, at:] = 255
    return [m[0], m[1]]


@pytest.mark.parametrize("value", [NAN, INF])
@pytest.mark.parametrize("L, at", [(2, (7, 0)), (4, (7, 0)), (4, (11, 39)), (4, (0, 17)), (5, (5, 20))])
def test_forward(L, at, value):
    """A frame at the canvas's left edge, seam weights everywhere: its region ends inside the canvas."""
    W, H, fw, fh = 301, 41, 40, 41
    f = np.random.default_rng(L).random((3, fh, fw)).astype(np.float32)
    f[:, at[0], at[1]] = value
    masks = [np.full((H, W), 255, np.uint8)]
    plan = P.Plan([(fw, fh)], [_shift(0.25, 0.5)], masks, W, H, L, bind=False)
    fo = o.FrameVjpOracle([f.astype(np.float64)], [_shift(0.25, 0.5)], masks, W, H, L)
    got = plan.forward_f32([torch.from_numpy(f).to(DEV)]).cpu().numpy()
    with np.errstate(invalid="ignore"):
        _agree(got, _forward(fo), "R_0")


@pytest.mark.parametrize("value", [NAN, INF])
@pytest.mark.parametrize("L", [3, 4, 5])
def test_the_first_column_stays_left(L, value):
    """An upstream gradient's first column has no share in the frame's right half."""
    W, H = 301, 49
    rng = np.random.default_rng(L)
    f = rng.random((3, H, W)).astype(np.float32)
    u = rng.normal(size=(3, H, W)).astype(np.float32)
    u[:, 23, 0] = value
    plan = P.Plan([(W, H)], [_shift(0.25, 0.5)], [np.full((H, W), 255, np.uint8)], W, H, L, bind=False)
    got = plan.backward([torch.from_numpy(f).to(DEV)], torch.from_numpy(u).to(DEV))[0][0]
    assert not torch.isfinite(got[:, 23, :2]).any()
    assert torch.isfinite(got[:, :, W // 2:]).all()


@pytest.mark.parametrize("value", [NAN, INF])
@pytest.mark.parametrize("L, x", [(1, 9), (2, 0), (3, 0), (4, 0), (2, 77), (4, 40), (3, 118), (4, 117)])
def test_upstream_gradient(L, x, value):
    """A camera over the whole canvas."""
    W, H = 119, 37
    rng = np.random.default_rng(x)
    f = rng.random((3, H, W)).astype(np.float32)
    u = rng.normal(size=(3, H, W)).astype(np.float32)
    u[:, 19, x] = value
    masks = [np.full((H, W), 255, np.uint8)]
    plan = P.Plan([(W, H)], [_shift(0.25, 0.5)], masks, W, H, L, bind=False)
    fo = o.FrameVjpOracle([f.astype(np.float64)], [_shift(0.25, 0.5)], masks, W, H, L)
    got = plan.backward([torch.from_numpy(f).to(DEV)], torch.from_numpy(u).to(DEV))[0]
    with np.errstate(invalid="ignore"):
        _agree(got[0].cpu().numpy(), _vjp(fo, u.astype(np.float64), None)[0], "d_frame")


@pytest.mark.parametrize("value", [NAN, INF])
@pytest.mark.parametrize("L", [2, 3, 4])
@pytest.mark.parametrize("x", [150, 157, 159, 160, 163])
def test_upstream_gradient_at_a_seam(x, L, value):
    """Two frames over the whole canvas that meet at a seam, with direct terms: dG_0 is wanted beyond the
    cameras' regions, whose dG_1 ends beside the seam."""
    W, H = 333, 37
    rng = np.random.default_rng(x)
    frames = [rng.random((3, H, W)).astype(np.float32) for _ in range(2)]
    Hs = [_shift(0.25, 0.5), _shift(-0.5, 0.25)]
    u = rng.normal(size=(3, H, W)).astype(np.float32)
    u[:, 18, x] = value
    direct = [rng.normal(size=(3, H, W)).astype(np.float32) for _ in range(2)]
    masks = _cuts(W, H, 160)
    plan = P.Plan([(W, H)] * 2, Hs, masks, W, H, L, bind=False)
    fo = o.FrameVjpOracle([f.astype(np.float64) for f in frames], Hs, masks, W, H, L)
    dev = lambda v: torch.from_numpy(v).to(DEV)
    got = plan.backward([dev(f) for f in frames], dev(u), [dev(d) for d in direct])[0]
    with np.errstate(invalid="ignore"):
        want = _vjp(fo, u.astype(np.float64), [d.astype(np.float64) for d in direct])
    for i in range(2):
        if np.isfinite(want[i]).all():
            assert np.isfinite(got[i].cpu().numpy()).all(), i
        else:
            _agree(got[i].cpu().numpy(), want[i], f"d_frame {i}")
