"""CPU-only check of the widest pass kernels' registers: a lane of 32 limbs needs
close to the 256 vector registers that two waves per SIMD leave it, and one
more halves the waves."""
import importlib.util
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2501_07535_amd", "csrc")

SRC = """#include "ntt_impl.hpp"
namespace moma {
template __global__ void ntt_pass_kernel<32, 1, false, false, kArithFull>(NttPassArgs, NttC<32, true>);
template __global__ void ntt_pass_kernel<32, 1, false, false, kArithLazy>(NttPassArgs, NttC<32>);
template __global__ void ntt_batch_kernel<32, 1, false, false, true>(const NttPassArgs*, const NttC<32, true>*, const uint2*,
                                                                     u32);
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc is not available")
def test_kernels_of_32_limbs_leave_room_for_two_waves(tmp_path):
    spec = importlib.util.spec_from_file_location("moma_build_script", os.path.join(ROOT, "paper_2501_07535_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    src.write_text(SRC)
    r = subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", f"-I{CSRC}", f"-I{ROOT}/include", str(src), "-o",
                        str(asm)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    text = asm.read_text()
    waves = [int(v) for v in re.findall(r"^; Occupancy: (\d+)", text, re.M)]
    scratch = [int(v) for v in re.findall(r"^; ScratchSize: (\d+)", text, re.M)]
    assert len(waves) == 3 and min(waves) >= 2, waves
    assert max(scratch) == 0, scratch
