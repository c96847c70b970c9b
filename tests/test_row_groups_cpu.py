"""The test by which the QKV epilogue takes 32 rows for consecutive keys of V^T
holds only for rows that are: every group of every launch form of many packed
batches, against the positions of all its rows.  Host compilation of the
library's own index functions."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2510_01565_amd", "csrc")
CXX = shutil.which("g++") or shutil.which("c++")
ROCM_INCLUDE = "/opt/rocm/include"

SOURCE = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "dit_internal.h"
using namespace dit;

static long groups, taken, wrong, missed, ends_only_wrong;

// rows [row_base, row_base + M) of a launch, in groups of 32
static void launch(const BatchMeta& m, int row_base, int M) {
  for (int g = 0; g + 31 < M; g += 32) {
    const RowEntry a = make_row_entry(m, row_base + g), b = make_row_entry(m, row_base + g + 31);
    bool in_line = true, one_request = true;
    for (int q = 1; q < 32; ++q) {
      const RowEntry e = make_row_entry(m, row_base + g + q);
      in_line = in_line && e.pos == a.pos + q;
      one_request = one_request && e.req == a.req;
    }
    const bool got = rows_consecutive(a, b, 32);
    ++groups;
    taken += got;
    wrong += got && !in_line;
    missed += !got && in_line && one_request;
    ends_only_wrong += b.pos == a.pos + 31 && !in_line;
  }
}

static void batch(int n, const int* gh, const int* gw, const int* nt) {
  BatchMeta m;
  memset(&m, 0, sizeof m);
  m.n_req = n;
  for (int r = 0; r < n; ++r) {
    const int ni = gh[r] * gw[r];
    m.txt_off[r + 1] = m.txt_off[r] + nt[r];
    m.img_off[r + 1] = m.img_off[r] + ni;
    m.joint_off[r + 1] = m.joint_off[r] + nt[r] + ni;
    m.pad_off[r + 1] = m.pad_off[r] + (nt[r] + ni + kSeqPad - 1) / kSeqPad * kSeqPad;
    m.n_txt[r] = nt[r];
    m.grid_w[r] = gw[r];
  }
  m.T_txt = m.txt_off[n];
  m.T_img = m.img_off[n];
  m.T = m.T_txt + m.T_img;
  launch(m, 0, m.T);               // a single-stream block: text rows, then image rows
  launch(m, 0, m.T_txt);           // a double-stream block's two groups
  launch(m, m.T_txt, m.T_img);
}

int main() {
  for (int ni = 1; ni <= 31; ++ni)  // two requests around every seam
    for (int nt = 1; nt <= 399; ++nt) {
      const int gh[2] = {1, 16}, gw[2] = {ni, 16}, t[2] = {nt, 0};
      batch(2, gh, gw, t);
    }
  srand(1);
  for (int k = 0; k < 20000; ++k) {
    int gh[16], gw[16], t[16];
    const int n = 1 + rand() % (k % 4 == 0 ? 16 : 4);
    for (int r = 0; r < n; ++r) {
      gh[r] = 1 + rand() % 12;
      gw[r] = 1 + rand() % 12;
      t[r] = rand() % 3 ? rand() % 130 : 0;
    }
    batch(n, gh, gw, t);
  }
  printf("%ld %ld %ld %ld %ld\n", groups, taken, wrong, missed, ends_only_wrong);
  return 0;
}
"""


@pytest.mark.skipif(CXX is None or not os.path.isdir(ROCM_INCLUDE), reason="no host compiler or HIP headers")
def test_consecutive_rows_are_consecutive(tmp_path):
    src, exe = tmp_path / "rows.cpp", tmp_path / "rows"
    src.write_text(SOURCE)
    r = subprocess.run([CXX, "-O2", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I", CSRC, "-I", ROCM_INCLUDE,
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    groups, taken, wrong, missed, ends_only = map(int, subprocess.run([str(exe)], capture_output=True, text=True,
                                                                      check=True).stdout.split())
    assert groups > 200000 and taken > 50000
    assert wrong == 0    # a group taken for consecutive rows is consecutive
    assert missed == 0   # and every group of consecutive rows of one request is taken
    assert ends_only > 50  # the batches do hold groups whose end positions alone look consecutive
