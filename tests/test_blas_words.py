"""The elementwise multiplies at the narrowest limb counts, which stay on 32-bit words.

On the CPU, the compiled kernels: fewer VALU instructions than the digit form
takes at the same limb count, as calls bound by memory need.  On the GPU, parity
at the limb counts on both sides of the line, with every kind of scaling."""
import importlib.util
import os
import random
import re
import shutil
import subprocess

import pytest

import moma_inputs as mi

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2501_07535_amd", "csrc")

SRC = """#include "blas.hip"
namespace moma {
template <int L, bool FW>
__global__ void digits_kernel(const u32* pa, const u32* pb, u32* pout, u64 n, BarrettC<L, FW> c) {
  const u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  u32 a[L], b[L], r[L];
#pragma unroll
  for (int j = 0; j < L; j++) {
    a[j] = __builtin_nontemporal_load(pa + (u64)j * n + i);
    b[j] = __builtin_nontemporal_load(pb + (u64)j * n + i);
  }
  barrett_mul_digits<L, FW>(r, a, b, c);
#pragma unroll
  for (int j = 0; j < L; j++) __builtin_nontemporal_store(r[j], pout + (u64)j * n + i);
}
template __global__ void digits_kernel<2, false>(const u32*, const u32*, u32*, u64, BarrettC<2>);
template __global__ void digits_kernel<3, false>(const u32*, const u32*, u32*, u64, BarrettC<3>);
template __global__ void digits_kernel<4, false>(const u32*, const u32*, u32*, u64, BarrettC<4>);
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc is not available")
def test_word_products_issue_fewer_instructions(tmp_path):
    spec = importlib.util.spec_from_file_location("moma_build_script", os.path.join(ROOT, "paper_2501_07535_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    src, asm = tmp_path / "k.hip", tmp_path / "k.s"
    # the library's own instances, at the narrow limb counts only
    text = open(os.path.join(CSRC, "blas.hip")).read()
    (tmp_path / "blas.hip").write_text(text[:text.index("static int launch_blas_LK")].rsplit("template", 1)[0] + """
template __global__ void blas_kernel<2, OP_VMUL, false, false>(const u32*, const u32*, u32*, u64, BlasC<2, false>);
template __global__ void blas_kernel<3, OP_VMUL, false, false>(const u32*, const u32*, u32*, u64, BlasC<3, false>);
template __global__ void blas_kernel<4, OP_VMUL, false, false>(const u32*, const u32*, u32*, u64, BlasC<4, false>);
}
""")
    src.write_text(SRC)
    r = subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", f"-I{tmp_path}", f"-I{CSRC}", f"-I{ROOT}/include",
                        str(src), "-o", str(asm)], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    products = {}
    for m in re.finditer(r"^(_ZN4moma\S*?(blas|digits)_kernelILi(\d)E\S*):(.*?)s_endpgm", asm.read_text(), re.S | re.M):
        products[m.group(2), int(m.group(3))] = len(re.findall(r"^\tv_mad_u64_u32", m.group(4), re.M))
    for L in (2, 3, 4):
        assert products["blas", L] < products["digits", L], products


@pytest.mark.gpu
@pytest.mark.parametrize("limbs,bits", [(2, 29), (2, 34), (2, 60), (2, 62), (2, 64), (3, 61), (3, 92), (3, 93), (3, 96),
                                        (4, 93), (4, 124), (4, 128), (5, 125), (5, 156)])
def test_products_on_both_sides_of_the_line(limbs, bits):
    import paper_2501_07535_amd as moma
    from gpu_util import from_dev, say, to_dev
    rng = random.Random(100 * limbs + bits)
    say(f"limbs={limbs} bits={bits}")
    for q in ((1 << bits) - 1, (1 << (bits - 1)) + 1, rng.getrandbits(bits) | 1 << (bits - 1) | 1):
        edge = [0, 1, q - 1, q - 2, q >> 1, (1 << 32) % q, (1 << (bits - 1)) % q]
        va = edge * len(edge) + [rng.randrange(q) for _ in range(470)]
        vb = [e for e in edge for _ in edge] + [rng.randrange(q) for _ in range(470)]
        da, db = to_dev(mi.ints_to_rows(va, limbs)), to_dev(mi.ints_to_rows(vb, limbs))
        want = mi.ints_to_rows([x * y % q for x, y in zip(va, vb)], limbs)
        assert (from_dev(moma.vmul(da, db, q)) == want).all(), q
        for al in (0, 1, q - 1, rng.randrange(q)):
            ax = mi.ints_to_rows([(al * x + y) % q for x, y in zip(va, vb)], limbs)
            assert (from_dev(moma.axpy(al, da, db, q)) == ax).all(), (q, al)
        outs = [to_dev(mi.ints_to_rows(va, limbs)) for _ in range(2)]
        batch = moma.Batch([((da, db), outs[0], q, None, moma.JOB_VMUL), ((da, db), outs[1], q, al, moma.JOB_AXPY)])
        batch.run()
        assert (from_dev(outs[0]) == want).all() and (from_dev(outs[1]) == ax).all(), q
