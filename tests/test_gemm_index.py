"""The register-staged GEMM loads inside its rows (CPU; a host build of the index)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2604_21290_amd", "csrc")
CXX = shutil.which("g++") or shutil.which("c++")

PROGRAM = r"""
#include <cstdio>
#include "gemm_index.h"
int main() {
  const int steps[] = {128, 192, 256, 384};
  for (int step : steps)
    for (int rowb = 16; rowb <= 3 * 384; rowb += 16) {
      const int stages = (rowb + step - 1) / step;
      // the deepest pipeline requests three stages past the one it multiplies
      for (int s = 0; s < stages + 3; ++s)
        for (int slot = 0; slot < step; slot += 16) {
          const int at = slot + gl::gemm_slot_offset(s, step, slot, rowb);
          const bool in = s * step + slot < rowb;
          if (at < 0 || at + 16 > rowb || (in && at != s * step + slot)) {
            std::printf("step %d row %d stage %d slot %d: byte %d\n", step, rowb, s, slot, at);
            return 1;
          }
        }
    }
  return 0;
}
"""


@pytest.mark.skipif(CXX is None, reason="no host compiler")
def test_every_staged_vector_lies_in_its_row(tmp_path):
    src, exe = tmp_path / "index.cpp", tmp_path / "index"
    src.write_text(PROGRAM)
    subprocess.run([CXX, "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
