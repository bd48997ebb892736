"""The multi-try stopping rule on the CPU: its form in doubles decides as the
128-bit form does, at the edges of the range it is taken for and next to the
decision's own boundary."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include <stdio.h>
#include <stdlib.h>
#include "fr_internal.h"
static uint64_t state = 88172645463325252ull;
static uint64_t next() {
  state ^= state << 13;
  state ^= state >> 7;
  return state ^= state << 17;
}
int main() {
  const int64_t ps[] = {1, 2, 3, 2048, 4094, 4095, 4096};
  const int64_t s1s[] = {-4096, -4095, -4094, -1, 0, 1, 4094, 4095, 4096};
  const int64_t s2s[] = {0, 1, (1 << 23) + 1, (1 << 24) - 2, (1 << 24) - 1, 1 << 24};
  const int64_t als[] = {1, 2, 3, 512, 1022, 1023, 1024};
  int64_t checked = 0, near = 0;
  for (int i = 0; i < 400000; i++) {
    const int64_t p = i % 2 ? ps[next() % 7] : 1 + next() % 4095;
    const int64_t s1 = i % 3 ? s1s[next() % 9] : (int64_t)(next() % 8191) - 4095;
    const int64_t s2 = i % 5 ? s2s[next() % 6] : next() % (1 << 24);
    const int64_t al = i % 7 ? als[next() % 7] : 1 + next() % 1023;
    const __int128 lhs = ((__int128)p * s1 * s1 - (__int128)al * ((__int128)p * s2 - s1 * s1)) * 65536;
    const int64_t edge = (int64_t)(lhs / ((__int128)p * p));
    const int64_t betas[] = {0, 45426, 1408000, (1 << 21) - 1, edge - 1, edge, edge + 1};
    for (const int64_t b : betas) {
      if (b < 0 || b >= (1 << 21)) continue;  // floor(ln n 2^16), n < 2^31
      checked++;
      near += b >= edge - 1 && b <= edge + 1;
      if (mt_stop(p, s1, s2, (int32_t)al, b) != mt_stop_int(p, s1, s2, (int32_t)al, b)) {
        printf("p %ld S1 %ld S2 %ld alpha %ld beta %ld\n", p, s1, s2, al, b);
        return 1;
      }
    }
  }
  return near > 10000 && checked > 1000000 ? 0 : 2;
}
"""


def test_double_form_is_exact(tmp_path):
    src, exe = tmp_path / "s.cpp", tmp_path / "s"
    src.write_text(SOURCE)
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "include"),
                           "-I" + os.path.join(ROOT, "paper_1012_0006_amd", "csrc"), str(src),
                           "-o", str(exe)])
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, (r.returncode, r.stdout)
