"""The sums into a workgroup's decoder-gradient image in LDS, which all its waves
add to at once by compare-and-swap: every read of the image there is an atomic one
in the compiled code (an ordinary load of a word that another wave swaps may be
repeated, and the swap then succeed on a sum of an older value)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2507_03836_amd import build as B

KERNEL = """
#include "mlp_train_dev.h"
__global__ void k(const float* x, float* out) {
  __shared__ __attribute__((aligned(16))) float image[%d];
  for (int e = threadIdx.x; e < %d; e += blockDim.x) image[e] = 0.0f;
  __syncthreads();
  %s
  __syncthreads();
  out[blockIdx.x * blockDim.x + threadIdx.x] =
      __hip_atomic_load(image + threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
"""
TILES = """
  fh::f4v v[%d];
  for (int t = 0; t < %d; ++t)
    for (int i = 0; i < 4; ++i) v[t][i] = x[(t * 4 + i) * blockDim.x + threadIdx.x];
  fh::lds_add_tiles(image, v);
"""


@pytest.mark.parametrize("adds", ["scalar", "tiles 1", "tiles 4"])
def test_image_is_read_atomically(tmp_path, adds):
    hipcc = shutil.which(B.HIPCC) or shutil.which("hipcc")
    if hipcc is None:
        pytest.skip("no hipcc")
    if adds == "scalar":
        src = KERNEL % (64, 64, "fh::lds_add(image + threadIdx.x % 64, x[threadIdx.x]);")
    else:
        n = int(adds.split()[1])
        src = KERNEL % (256 * n, 256 * n, TILES % (n, n))
    f, ir = tmp_path / "k.hip", tmp_path / "k.ll"
    f.write_text(src)
    subprocess.run([hipcc, *B.FLAGS, "--cuda-device-only", "-S", "-emit-llvm", str(f), "-o", str(ir)],
                   check=True, capture_output=True, cwd=os.fspath(tmp_path))
    loads = re.findall(r"= load (?:atomic |volatile )?[^\n]*addrspace\(3\)[^\n]*", ir.read_text())
    assert re.search(r"cmpxchg[^\n]*addrspace\(3\)", ir.read_text())
    assert loads and all(l.startswith("= load atomic") for l in loads), loads
