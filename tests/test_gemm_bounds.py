"""Where the GEMM's LDS-bound loads read, computed on the host by the kernels' own function."""
import os
import subprocess

from tests.libqe import ROOT

SOURCE = r"""
#include "gemm_util.h"
#include <stdio.h>
int main() {
  for (int k = 1; k <= 400; ++k)
    for (int ld = (k + 15) / 16 * 16; ld <= 512; ld += 16)
      for (int rows = 1; rows <= 40; rows += 13)
        for (int row = 0; row < rows; ++row)
          for (int c = 0; c < 8; ++c) {
            const long at = qe::chunk_offset(row, ld, c, k);
            if (at + 16 > long(rows - 1) * ld + (k + 15) / 16 * 16) return printf("k %d ld %d rows %d row %d chunk %d reads past the operand\n", k, ld, rows, row, c), 1;
            if (16 * c < k && at != long(row) * ld + 16 * c) return printf("k %d ld %d row %d chunk %d moved\n", k, ld, row, c), 1;
          }
  // the last row of an operand just below 2 GiB
  if (qe::chunk_offset((1 << 24) - 1, 127 + 1, 7, 4096) != uint32_t(((1u << 24) - 1) * 128u + 112u)) return puts("32 bits"), 1;
  return 0;
}
"""


def test_loads_of_the_first_k_tile_stay_inside_the_operand(tmp_path):
    """Row strides down to the reduction rounded up to 16, which the entry point accepts: no 16-byte load of the
    first K tile ends past the last row, and every chunk that holds part of the reduction is read in its place.
    The large tiles load whole first tiles also where the reduction is shorter than one."""
    src, exe = tmp_path / "bounds.hip", tmp_path / "bounds"
    src.write_text(SOURCE)
    subprocess.run(["/opt/rocm/bin/hipcc", "--offload-arch=gfx950", "--cuda-host-only", "-std=c++17", "-O1", "-w", "-I",
                    os.path.join(ROOT, "paper_2609_23536_amd", "csrc"), str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
