"""LDS layout of the one-workgroup sweep, on the CPU: every wave's slice starts on
a 16-byte boundary (it is read 16 bytes at a time) behind the residuals and ends
inside what the host asks for, whatever the numbers of cells and variables."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2310_08230_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "small_layout.h"

template <typename R>
int check(int waves) {
  for (int64_t cells = 0; cells < 40; ++cells)
    for (int64_t vars = 1; vars < 40; ++vars) {
      const int64_t at = small_slices_at<R>(cells, vars), all = small_reals<R>(cells, vars, true, waves);
      for (int w = 0; w < waves; ++w)
        if ((at + w * CHUNK_SLICE) * int64_t(sizeof(R)) % 16) return 1;
      if (at < cells + 1 + vars || at + waves * CHUNK_SLICE > all) return 2;
      if (small_reals<R>(cells, vars, false, waves) != cells + 1 + vars) return 3;
    }
  return 0;
}

int main() {
  const int f = check<float>(12), d = check<double>(8);
  std::printf("%d %d\n", f, d);
  return f | d;
}
"""


def test_slices_are_aligned_and_inside(tmp_path):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)], capture_output=True, text=True).stdout.split() == ["0", "0"]
