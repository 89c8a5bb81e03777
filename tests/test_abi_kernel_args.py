"""Kernels that read a descriptor argument through the constant address space take it from the argument
segment: in unoptimised device code, where a by-value parameter is a private copy, no pointer into
private memory becomes one into the constant address space (scalar memory reads at a private address)."""
import re
import shutil
import subprocess
from pathlib import Path

import pytest

from paper_1810_03988_amd.build import CSRC, ROOT, hipcc

OPT = Path(hipcc()).resolve().parent.parent / "llvm" / "bin" / "opt"
# references and locals that hold pointers become values; by-value structs stay private copies
PASSES = "always-inline,function(infer-address-spaces,mem2reg,infer-address-spaces,mem2reg)"


@pytest.mark.skipif(not (shutil.which(hipcc()) and OPT.exists()), reason="needs hipcc and opt")
@pytest.mark.parametrize("source", ["kernels.hip", "lorb.hip", "register.hip", "grad.hip"])
def test_no_private_pointer_becomes_a_constant_one(source, tmp_path):
    ll, out = tmp_path / "raw.ll", tmp_path / "out.ll"
    subprocess.run([hipcc(), "--offload-arch=gfx950", "-O0", "-Xclang", "-disable-O0-optnone", "-std=c++17",
                    f"-I{ROOT / 'include'}", f"-I{CSRC}", "--cuda-device-only", "-S", "-emit-llvm", "-o", str(ll),
                    str(CSRC / source)], check=True, capture_output=True)
    subprocess.run([str(OPT), "-mcpu=gfx950", "-passes=" + PASSES, "-S", "-o", str(out), str(ll)], check=True,
                   capture_output=True)
    kernels = found = 0
    for body in re.split(r"(?m)^define ", out.read_text())[1:]:
        kernels += "amdgpu_kernel" in body.split("\n", 1)[0]
        private = set()
        for line in body.splitlines():
            m = re.match(r"\s+(%[\w.]+) = (.*)", line)
            if not m:
                continue
            name, rhs = m.groups()
            used = set(re.findall(r"%[\w.]+", rhs))
            if rhs.startswith("alloca"):
                private.add(name)
            elif re.match(r"(addrspacecast|getelementptr|select|phi)\b", rhs) and used & private:
                if rhs.startswith("addrspacecast") and rhs.rstrip().endswith("to ptr addrspace(4)"):
                    found += 1
                else:
                    private.add(name)
    assert kernels > 0
    assert found == 0, f"{found} private pointers read as constant memory"
