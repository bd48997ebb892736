"""The row solver's work counters on the CPU: with the largest corridor, the
smallest workgroup and 63 arcs per vertex, thousands of relabels and passes of
one launch stay within what the lanes' 32-bit counts and a wave's total hold,
and the sums come out whole."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <stdio.h>
#include "fr_internal.h"
int main() {
  const int64_t nr = 577000, tpb = 256, waves = tpb / 64, relabels = 5000;
  const int64_t rows_gr = (nr * 2 + tpb - 1) / tpb + 1, rows_pass = (nr * 4 + tpb - 1) / tpb + 1;
  RowWork w;  // every lane of every wave at the largest count
  int64_t sum[2] = {0, 0}, want[2] = {0, 0};
  auto flush = [&]() {
    for (int j = 0; j < 2; j++) {
      const int64_t total = 64 * (int64_t)w.arcs[j];
      if (w.arcs[j] < 0 || total > 0x7fffffffll) return false;
      sum[j] += waves * total;
      w.arcs[j] = 0;
    }
    return true;
  };
  for (int64_t s = 0; s < relabels; s++) {
    w.gr_items += nr;
    w.arcs[1] += (int32_t)(63 * rows_gr);
    w.arcs[0] += (int32_t)(63 * rows_pass);
    want[0] += waves * 64 * 63 * rows_pass;
    want[1] += waves * 64 * 63 * rows_gr;
    if (w.due() && !flush()) return 1;
  }
  if (!flush()) return 2;
  if (sum[0] != want[0] || sum[1] != want[1]) return 3;
  if (w.gr_items != relabels * nr) return 4;
  puts("ok");
  return 0;
}
"""


def test_row_work_counts(tmp_path):
    src, exe = tmp_path / "w.cpp", tmp_path / "w"
    src.write_text(SOURCE)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_1012_0006_amd", "csrc"), str(src),
                           "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.returncode
