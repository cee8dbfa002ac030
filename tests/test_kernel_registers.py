"""Vector registers of the built pair kernels: the waves on a SIMD that their
timings rest on (512 registers, in steps of 8).  Reads the metadata of this
package's own library; no GPU needed."""
import os
import re
import shutil
import subprocess

import pytest

from paper_1709_02410_amd import rpywall

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def vgprs(tmp_path_factory):
    objdump, readelf = (os.path.join(LLVM, t) for t in ("llvm-objdump", "llvm-readelf"))
    if not os.path.exists(rpywall.LIB_PATH) or not os.path.exists(objdump):
        pytest.skip("librpywall.so not built, or no LLVM tools")
    d = str(tmp_path_factory.mktemp("co"))
    lib = shutil.copy(rpywall.LIB_PATH, d)
    subprocess.run([objdump, "--offloading", os.path.basename(lib)], cwd=d, check=True, capture_output=True)
    out = {}
    for f in os.listdir(d):
        if f.endswith("gfx950"):
            notes = subprocess.run([readelf, "--notes", f], cwd=d, check=True, capture_output=True, text=True).stdout
            out.update((n, int(v)) for n, v in
                       re.findall(r"\.name:\s+(\S+)\n(?:.*\n)*?\s+\.vgpr_count:\s+(\d+)", notes))
    assert out
    return out


@pytest.mark.parametrize("what,pattern,waves", [
    ("VJP, FP32, groups of 256", r"10sym_kernelI.*VjpBodyIfE.*Li4ELi1ELb0E", 4),
    ("VJP, FP32, groups of 64", r"10sym_kernelI.*VjpBodyIfE.*Li1ELi1ELb0E", 4),
    ("product, FP32, groups of 256", r"10sym_kernelI.*ProductBodyIfLi1ELi0E.*Li4ELi1ELb0E", 6),
    ("product, FP64, groups of 256", r"10sym_kernelI.*ProductBodyIdLi1ELi0E.*Li4ELi1ELb0E", 4),
    ("periodic, FP32, groups of 256", r"10sym_kernelI.*ProductBodyIfLi1ELi1E.*Li4ELi1ELb0E", 5),
    ("periodic, FP32, packed groups of 64", r"10sym_kernelI.*ProductBodyIfLi1ELi1E.*Li1ELi1ELb0E", 5),
    ("periodic, FP64, groups of 256", r"10sym_kernelI.*ProductBodyIdLi1ELi2E.*Li4ELi1ELb0E", 4),
])
def test_waves_per_simd(vgprs, what, pattern, waves):
    found = {n: v for n, v in vgprs.items() if re.search(pattern, n)}
    assert len(found) == 1, found
    (v,) = found.values()
    print(what, v)
    assert -(-v // 8) * 8 * waves <= 512, (what, v, waves)
