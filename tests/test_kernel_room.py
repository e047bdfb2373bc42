"""The persistent selection's occupancy answers (csrc/gmc_occupancy.h), against
fake driver calls on the CPU: a kernel's LDS grant never shrinks, and sizes that
come in turn are asked for once."""
import os
import shutil
import subprocess

import pytest

from paper_2608_02134_amd import binding as B

PROGRAM = r"""
#include <stdio.h>
#include <algorithm>
#include "gmc_occupancy.h"
int main() {
  gmc::KernelRoom room;
  size_t limit = 64 * 1024;     // what the fake driver has granted
  int grants = 0, asks = 0;
  auto grant = [&](size_t n) { ++grants; if (n > 140 * 1024) return false; limit = n; return true; };
  auto ask = [&](size_t n, int* b) { ++asks; if (n > limit) return false; *b = int(160 * 1024 / (n + 24 * 1024)); return true; };
  const size_t turn[] = {0, 100 * 1024, 70 * 1024, 30 * 1024, 150 * 1024};
  size_t most = 64 * 1024;
  for (int pass = 0; pass < 3; ++pass)
    for (size_t n : turn) {
      const int want = n > 140 * 1024 ? 0 : int(160 * 1024 / (n + 24 * 1024));
      if (room.blocks(n, grant, ask) != want) { printf("wrong answer for %zu\n", n); return 1; }
      if (n <= 140 * 1024) most = std::max(most, n);
      if (limit < most) { printf("the grant fell to %zu\n", limit); return 1; }
    }
  if (grants != 2 || asks != 4) { printf("%d grants, %d queries\n", grants, asks); return 1; }
  // more sizes than are kept: answers stay right, memory stays bounded
  for (int pass = 0; pass < 2; ++pass)
    for (size_t n = 1024; n <= 40 * 1024; n += 1024)
      if (room.blocks(n, grant, ask) != int(160 * 1024 / (n + 24 * 1024))) { printf("wrong answer for %zu\n", n); return 1; }
  if (limit != 100 * 1024) { printf("the grant moved to %zu\n", limit); return 1; }
  printf("ok\n");
  return 0;
}
"""


def test_grants_only_grow_and_answers_are_kept(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if not cxx:
        pytest.skip("no C++ compiler")
    src, exe = tmp_path / "room.cpp", tmp_path / "room"
    src.write_text(PROGRAM)
    csrc = os.path.join(os.path.dirname(B.LIB_PATH), "csrc")
    subprocess.run([cxx, "-std=c++17", "-I", csrc, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
