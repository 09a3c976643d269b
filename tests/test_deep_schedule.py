"""The addresses of the matrix-core bound GEMM's K loop, on the host: every load it issues, the
unused ones past its K range included, stays inside the weight group or activation row it is
meant for, whatever the hardware's range check covers."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2606_26744_amd", "csrc")

# The loop's issue order: a prologue of D weight units and CU / 2 + 1 activation pairs, then
# unit u issues weight unit u + D and pair u / 2 + CU / 2 + 1.
WALK = r"""
#include <cstdio>
#include "deep_schedule.hpp"
using namespace hdf;
int main() {
  for (int k0 = 0; k0 < 40; ++k0)
    for (int k1 = k0 + 1; k1 < 80; ++k1)
      for (int CU = 2; CU <= 4; CU += 2) {
        const int ku0 = 2 * k0, nu = 2 * (k1 - k0), np = nu / 2, D = kDeepRing - 1;
        auto weight = [&](int u) {
          for (int ss = 0; ss < 2; ++ss) {
            const int at = deep_weight_offset(ku0, u, nu, ss);
            if (at < ku0 * 8192 || at + 4080 + 16 > deep_weight_bytes(k1)) return false;
            if (u < nu && at != (ku0 + u) * 8192 + ss * 4096) return false;
          }
          return true;
        };
        auto pair = [&](int pr) {
          const int at = deep_act_offset(ku0, pr, np);
          return at >= k0 * 128 && at + 128 <= k1 * 128 && (pr >= np || at == (k0 + pr) * 128);
        };
        bool ok = true;
        for (int x = 0; x < D; ++x) ok = ok && weight(x);
        for (int v = 0; v <= CU / 2; ++v) ok = ok && pair(v);
        for (int u = 0; u < nu; ++u) ok = ok && weight(u + D) && pair(u / 2 + CU / 2 + 1);
        if (!ok) {
          std::printf("K steps %d..%d, %d units a barrier\n", k0, k1, CU);
          return 1;
        }
      }
  return 0;
}
"""


def test_every_load_stays_in_its_operand(tmp_path):
    cxx = shutil.which("g++") or shutil.which("amdclang++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(WALK)
    subprocess.run([cxx, "-std=c++17", "-O1", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
