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


# d, causal, check (0 off, 1 sum, 2 weighted), heads, Lq, Lk, half workgroups:
# both sides of each line of the rule on 256 CUs, with the measured time of
# half over full workgroups
HALF = [
    # as many rounds of the CUs in both forms, two: 1.03, 1.015, 1.04, 1.01; without a
    # check and weighted 0.98, 0.99; one query tile 0.93; three: 1.015, 0.98
    (64, 0, 1, 32, 4096, 4096, 0), (64, 0, 1, 64, 2048, 2048, 0), (64, 0, 1, 13, 8192, 8192, 0),
    (64, 0, 1, 128, 1024, 1024, 0), (64, 0, 0, 32, 4096, 4096, 1), (64, 0, 2, 32, 4096, 4096, 1),
    (64, 0, 1, 48, 4096, 4096, 0), (64, 0, 1, 64, 4096, 4096, 1),
    (64, 0, 1, 192, 1024, 1024, 1), (64, 0, 1, 512, 256, 4096, 1),
    # a half round saved: 0.82, 0.84, 0.77
    (64, 0, 1, 24, 4096, 4096, 1), (64, 0, 1, 34, 4096, 4096, 1), (64, 1, 1, 300, 256, 2048, 1),
    # no mask, no more full workgroups than CUs: 0.98 and 1.04, 1.07
    (64, 0, 1, 192, 256, 448, 1), (64, 0, 1, 96, 512, 512, 0), (64, 0, 1, 32, 2048, 2048, 0),
    # the same, causal: 0.82, 1.03, 1.03, 1.11, 0.89
    (64, 1, 1, 66, 512, 512, 1), (64, 1, 1, 80, 512, 512, 0), (64, 1, 1, 128, 512, 512, 0),
    (64, 1, 1, 128, 350, 350, 0), (64, 1, 1, 192, 130, 130, 1),
    # causal over more keys than queries, two full rounds: 1.08 (off 1.035, weighted
    # 1.05), 1.02 (off 0.975, weighted 0.97), 1.05 (off 0.975), 0.95; not full 0.92
    (64, 1, 1, 64, 2048, 4096, 0), (64, 1, 0, 64, 2048, 4096, 0), (64, 1, 2, 64, 2048, 4096, 0),
    (64, 1, 1, 64, 2048, 8192, 0), (64, 1, 0, 64, 2048, 8192, 1), (64, 1, 2, 64, 2048, 8192, 1),
    (64, 1, 1, 256, 512, 1024, 0), (64, 1, 0, 256, 512, 1024, 1), (64, 1, 1, 128, 1024, 2048, 1),
    (64, 1, 1, 200, 512, 2048, 1),
    # every half workgroup on its own CU
    (64, 0, 1, 12, 128, 128, 1), (96, 1, 1, 32, 256, 256, 1), (128, 1, 1, 32, 512, 512, 1),
    (128, 1, 1, 32, 128, 128, 0),
    # causal, long rows: 32 heads of 2,048 and 64 of 1,024; of 4,096
    (128, 1, 1, 32, 2048, 2048, 1), (128, 1, 1, 64, 1024, 1024, 0), (64, 1, 1, 32, 4096, 4096, 0),
    # short rows of many heads
    (64, 1, 1, 270, 700, 700, 1), (96, 0, 1, 384, 512, 512, 1), (128, 0, 1, 384, 512, 512, 0),
]


def test_half_workgroup_rule(tmp_path):
    rows = ",\n".join("{%s}" % ", ".join(map(str, r)) for r in HALF)
    r = run_cpp(tmp_path, f"""
int main() {{
  const int c[][7] = {{{rows}}};
  for (auto& x : c) printf("%d", (int)half_is_faster(x[0], x[1], x[2] != 0, x[2] == 2, x[3], x[4], x[5], 256));
  // a device whose CU count is unknown, and more workgroups than a grid holds
  printf("%d%d", (int)half_is_faster(64, false, true, false, 12, 128, 128, 0),
         (int)half_is_faster(64, false, true, false, 1 << 30, 300, 300, 256));
}}
""")
    assert r.returncode == 0
    got = [int(x) for x in r.stdout]
    assert got[-2:] == [0, 0]
    assert [(x, g) for x, g in zip(HALF, got) if x[-1] != g] == []


def test_global_check_threads(tmp_path):
    """One wave for short heads, sixteen while every head has a CU of its own and
    for long heads of many bytes, four otherwise."""
    r = run_cpp(tmp_path, """
int main() {
  const int c[][4] = {{12, 64, 64, 64}, {12, 65, 64, 1024}, {5000, 16, 128, 64}, {5000, 1, 256, 64},
                      {256, 2048, 128, 1024}, {257, 256, 64, 256}, {2048, 1024, 64, 1024},
                      {2047, 1024, 64, 256}, {5000, 1023, 64, 256}, {1, 1 << 20, 256, 1024},
                      {300, 65536, 256, 1024}};
  for (auto& x : c)
    if (global_threads(x[0], x[1], x[2]) != x[3]) printf("%d %d %d\\n", x[0], x[1], x[2]);
  return 0;
}
""")
    assert r.returncode == 0 and r.stdout == "", r.stdout
