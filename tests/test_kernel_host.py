"""CPU tests of the host-side functions that the kernels and their launches use
(csrc/fabft_kernels.h), compiled with g++ into a small program."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2507_16676_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


def run_cpp(tmp_path, body):
    src, exe = tmp_path / "t.cpp", tmp_path / "t"
    src.write_text('#include <cstdio>\n#include <cstdlib>\n#include "fabft_kernels.h"\n'
                   "using namespace fabft;\n" + body)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I",
                    os.path.join(rocm, "include"), str(src), "-o", str(exe)], check=True)
    return subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)


def test_wide_loads_stay_inside_the_rows(tmp_path):
    """The loads of the d = 256 forward (tiles 0 to t_end + 1, four steps of 16
    rows): the scalar offset never exceeds the buffer's size, so the range check
    (vector offset >= size - scalar offset) cannot wrap; the lanes it lets
    through are exactly the rows below Lk of the tiles [0, t_end), each from its
    own address."""
    r = run_cpp(tmp_path, r"""
int main() {
  const int ends[] = {1, 2, 3, 65535, 65536};
  for (int far = 0; far < 2; ++far)
    for (int i = 1; i <= 200; ++i) {
      const int Lk = far ? 4194240 - i : i;       // up to the largest accepted Lk
      const int all = (Lk + 63) / 64;
      for (int t_end : ends) {
        if (t_end > all) t_end = all;
        const uint32_t size = wide_load_size(Lk, t_end);
        const int first = t_end > 3 ? t_end - 3 : 0;
        for (int t = first; t < t_end + 2; ++t)
          for (int j = 0; j < 4; ++j) {
            const uint32_t so = wide_load_start(4 * t + j, size);
            if (so > size) { printf("Lk %d t_end %d t %d j %d: start past the size\n", Lk, t_end, t, j); return 1; }
            for (int row = 0; row < 16; ++row)
              for (uint32_t col = 0; col < kWideRowBytes; col += 16) {
                const uint32_t vo = row * kWideRowBytes + col;
                const bool loads = vo < size - so;
                const long long krow = 64LL * t + 16 * j + row;
                const bool wanted = t < t_end && krow < Lk;
                if (loads != wanted || (loads && (long long)so + vo != krow * 512 + col)) {
                  printf("Lk %d t_end %d key row %lld: loads %d\n", Lk, t_end, krow, (int)loads);
                  return 1;
                }
              }
          }
      }
    }
  return 0;
}
""")
    assert r.returncode == 0, r.stdout
