"""No kernel spills vector registers to scratch, but for the residual epilogue of the 256x256 tile with its split last round (256
accumulators, 16 registers).  Read from the code objects that this repository's own build leaves."""
import glob
import os
import re
import subprocess

import pytest

from paper_2605_11678_amd import build

LLVM = "/opt/rocm/llvm/bin/"
ALLOWED = {"gemm_fast_split_tailILi1E": 16}


def test_vector_register_spills(tmp_path):
    objs = sorted(glob.glob(os.path.join(build.PKG, "_build", "kernels_*.o")))
    tools = [LLVM + t for t in ("llvm-objcopy", "clang-offload-bundler", "llvm-readelf")]
    if not objs or not all(os.path.exists(t) for t in tools):
        pytest.skip("no objects of a build, or no LLVM tools")
    n = 0
    for o in objs:
        fat, co = str(tmp_path / "fat.bin"), str(tmp_path / "k.co")
        subprocess.run([tools[0], "--dump-section=.hip_fatbin=" + fat, o, str(tmp_path / "copy.o")], check=True)
        subprocess.run([tools[1], "--type=o", "--unbundle", "--input=" + fat, "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", "--output=" + co], check=True)
        notes = subprocess.run([tools[2], "--notes", co], check=True, capture_output=True, text=True).stdout
        for name, spill in re.findall(r"\.name: +(_Z\S+).*?\.vgpr_spill_count: +(\d+)", notes, re.S):
            n += 1
            assert int(spill) <= max([v for k, v in ALLOWED.items() if k in name], default=0), (name, spill)
    assert n > 50
