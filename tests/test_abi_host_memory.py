"""Entry points that take host memory report running out of it: with every allocation failing, a status
comes back instead of an exception that ends the process, and the plan stays usable."""
import os
import shutil
import subprocess
import sys

import pytest

from paper_1810_03988_amd.build import ROOT

SHIM = r"""
#include <cstdlib>
#include <new>
static bool armed = false;
extern "C" void arm(int on) { armed = on != 0; }
void* operator new(std::size_t n) {
  if (armed) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
"""

CALLS = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)   # before the library, whose allocations it serves
import numpy as np
import paper_1810_03988_amd as P
from paper_1810_03988_amd.stitch import CHW, F32, StitchImage, last_error, lib
W, H = 96, 64
plan = P.Plan([(W, H)], [np.eye(3)], [np.full((H, W), 255, np.uint8)], W, H, 3, device="cpu", bind=False)
buf = np.zeros(1 << 24, np.uint8)
ws = (buf.ctypes.data + 255) // 256 * 256
im = StitchImage(ws, W, H, 3, F32, CHW, 4 * W, 4 * W * H)
one = (StitchImage * 1)(im)
d = (ctypes.c_double * 9)()
n = lib().stitch_frame_backward_workspace_bytes(plan._h)
assert n < 1 << 23
calls = dict(
    bind=lambda: lib().stitch_plan_bind(plan._h, ws, plan.ws_bytes, None),
    forward=lambda: lib().stitch_frame_forward_f32(plan._h, one, ctypes.byref(im), ws, n, None),
    backward=lambda: lib().stitch_frame_backward(plan._h, one, ctypes.byref(im), None, one, d, ws, n, None))
call = calls[sys.argv[2]]
shim.arm(1)
status = call()
shim.arm(0)
assert status == 8 and "memory" in last_error(), (status, last_error())
print("STATUS", status)
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="needs g++")
@pytest.mark.parametrize("call", ["bind", "forward", "backward"])
def test_running_out_is_a_status(call, tmp_path):
    src, so, py = tmp_path / "shim.cpp", tmp_path / "shim.so", tmp_path / "calls.py"
    src.write_text(SHIM)
    py.write_text(CALLS)
    subprocess.run(["g++", "-O1", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    r = subprocess.run([sys.executable, str(py), str(so), call], env=dict(os.environ, PYTHONPATH=str(ROOT)),
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "STATUS" in r.stdout, (r.returncode, r.stderr[-2000:])
