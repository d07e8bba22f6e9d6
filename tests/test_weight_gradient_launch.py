"""CPU-only: which launches of two weight gradients the persistent groupXTY accepts.  That launch fetches the order indices for every stage,
also when both operands lie expert-sorted, so without them it has to be refused; maps with order indices of their own as well."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2403_08245_amd")

PROGRAM = r"""
#include "common.h"
#include <stdio.h>
int main() {
  static int32_t order[64], other[64], offsets[10];
  static float out[4];
  auto ask = [&](const char *name, const int32_t *o, const int32_t *a, const int32_t *b, const int32_t *a3, bool further) {
    DWArgs w{out, out, out, offsets, 9, 64, 1416, 1032};
    w.a_map = RowMap{a, 1};
    w.b_map = RowMap{b, 1};
    w.a3_map = RowMap{a3, 1};
    if (further) {
      w.A3 = w.B3 = out;
      w.dW3 = out;
      w.M3 = 1032;
      w.N3 = 2832;
    }
    w.order = o;
    printf("%s %d\n", name, (int)dw_stream_supported(w));
  };
  ask("one_sorted", nullptr, nullptr, nullptr, nullptr, false);
  ask("one_mapped", nullptr, order, order, nullptr, false);
  ask("two_without_order", nullptr, nullptr, nullptr, nullptr, true);
  ask("two_mapped_without_order", nullptr, nullptr, order, order, true);
  ask("two_sorted", order, nullptr, nullptr, nullptr, true);
  ask("two_mapped_b", order, nullptr, order, nullptr, true);
  ask("two_mapped_a3", order, nullptr, nullptr, order, true);
  ask("two_mapped", order, nullptr, order, order, true);
  ask("two_mapped_a", order, order, nullptr, nullptr, true);
  ask("two_other_b", order, nullptr, other, nullptr, true);
  ask("two_other_a3", order, nullptr, order, other, true);
  return 0;
}
"""


def test_two_weight_gradients_need_the_order_indices(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not shutil.which(hipcc):
        pytest.skip("no hipcc")
    import paper_2403_08245_amd as m
    src, exe = tmp_path / "ask.hip", tmp_path / "ask"
    src.write_text(PROGRAM)
    folder, name = os.path.split(os.path.abspath(m.lib._name))
    subprocess.run([hipcc, "--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-Wno-unused-command-line-argument",
                    "-I", os.path.join(PKG, "csrc"), "-I", os.path.join(ROOT, "include"), str(src), "-L" + folder, "-l:" + name, "-Wl,-rpath," + folder, "-o", str(exe)],
                   check=True, capture_output=True, text=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    got = {k: v == "1" for k, v in (line.split() for line in out.splitlines())}
    taken = {"one_sorted", "one_mapped", "two_sorted", "two_mapped_b", "two_mapped_a3", "two_mapped"}
    assert {k for k, v in got.items() if v} == taken
    assert len(got) == 11
