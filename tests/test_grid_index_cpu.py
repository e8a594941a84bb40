"""The gathers' per-axis node offsets against node_base, on the host, up to the largest grid a batch takes."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2412_12089_amd", "csrc")

SRC = r"""
#include "mpm_device.h"
#include <cstdio>
#include <cstdlib>
using namespace mpmx;

int main() {
  long bad = 0;
  for (int T : {3, 24, 203, 204, 256}) {
    EnvDev e = {};
    e.n = 4 * T;
    e.T = T;
    e.tile_off = 7;
    const float* grid = nullptr;   // addresses are compared, never read
    unsigned seed = 1;
    for (int r = 0; r < 4000; ++r) {
      int b[3];   // every second base lies in the last tile of each axis
      for (int a = 0; a < 3; ++a) b[a] = r % 2 ? e.n - 3 - (int)(rand_r(&seed) % 6) : (int)(rand_r(&seed) % (e.n - 2));
      const StencilAddr s = stencil_addr(e, b);
      for (int o = 0; o < 27; ++o) {
        const int i = o / 9, j = o / 3 % 3, k = o % 3;
        const uintptr_t got = (uintptr_t)(env_group1(e, grid) + (size_t)(uint32_t)(s.x[i] + s.y[j] + s.z[k]));
        const uintptr_t want = (uintptr_t)(node_base(e, b[0] + i, b[1] + j, b[2] + k) + G1) * sizeof(float);
        if (got != want && ++bad < 4) std::printf("T %d base %d %d %d node %d: %zu, not %zu\n", T, b[0], b[1], b[2], o, (size_t)got, (size_t)want);
      }
    }
  }
  std::printf("%ld wrong\n", bad);
  return bad != 0;
}
"""


def test_stencil_offsets_match_node_base(tmp_path):
    hipcc = os.environ.get("HIPCC") or shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "index.hip", tmp_path / "index"
    src.write_text(SRC)
    subprocess.run([hipcc, "-O1", "-std=c++17", "--cuda-host-only", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
