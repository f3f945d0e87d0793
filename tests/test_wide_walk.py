"""The wide kernel's walk through its weight stream (WideWalk, the code the
kernel runs, compiled here for the host): the fragments a wave multiplies are
the steps of its part in order, and every fragment it fetches, the ones ahead
of its last step too, lies within kWideTail bytes of the weights' end.  Walked
as the kernel does, over filter rows, parts of the reduction, channel splits
and channel counts down to one step.  Blobs hold those bytes."""
import subprocess

import pytest
import torch

from paper_2007_09835_amd import build, rt3d

TAIL = 35 * 1024

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "rt3d_internal.h"
static_assert(rt3d::kWideTail == TAIL, "the bytes a blob keeps behind the weights");
using namespace rt3d;

template <int FM, int WK>
long walk(int rows32, int ks, int c16, int c16_total) {
  const int frags = (rows32 + 1) / 2 * 2, stot = ks * c16_total;
  const long a_bytes = static_cast<long>(frags) * stot * 1024;
  const int nchunks = (c16_total + c16 - 1) / c16;
  const int sc_full = ks * c16, sc_last = ks * (c16_total - (nchunks - 1) * c16);
  long bad = 0;
  for (int row = 0; row < (rows32 + FM - 1) / FM * FM; row += FM)
    for (int kpart = 0; kpart < WK; ++kpart)
      for (int ch0 = 0; ch0 < nchunks; ++ch0)
        for (int ch1 = ch0 + 1; ch1 <= nchunks; ++ch1) {
          const int n_full = (sc_full - kpart + WK - 1) / WK;
          std::vector<long> want;   // steps of this part
          for (int ch = ch0; ch < ch1; ++ch)
            for (int s = kpart; s < (ch == nchunks - 1 ? sc_last : sc_full); s += WK)
              want.push_back(static_cast<long>(ch) * sc_full + s);
          WideWalk<FM, WK> w{};
          w.start(row, stot, ch0, sc_full, n_full, kpart);
          // the ring but its last slot, then one step ahead per step multiplied
          for (size_t s = 0; s < want.size() + kWideRing - 1; ++s) {
            for (int i = 0; i < FM; ++i) {
              if (static_cast<long>(w.off[i]) + 1024 > a_bytes + kWideTail) ++bad;
              if (s < want.size() && w.off[i] != (static_cast<long>(row + i) * stot + want[s]) * 1024) ++bad;
            }
            w.next();
          }
        }
  return bad;
}

int main() {
  long total = 0;
  for (int rows32 : {1, 2, 3, 8})
    for (int ks : {1, 2, 3, 9, 27})
      for (int c16 : {1, 2, 3, 8})
        for (int c16_total : {1, 2, 3, 4, 9, 16}) {
          if (c16 > c16_total) continue;
          const long bad = walk<1, 1>(rows32, ks, c16, c16_total) + walk<1, 2>(rows32, ks, c16, c16_total) +
                           walk<1, 4>(rows32, ks, c16, c16_total) + walk<2, 1>(rows32, ks, c16, c16_total) +
                           walk<2, 2>(rows32, ks, c16, c16_total) + walk<2, 4>(rows32, ks, c16, c16_total);
          if (bad) std::printf("rows32=%d ks=%d c16=%d of %d: %ld\n", rows32, ks, c16, c16_total, bad);
          total += bad;
        }
  return total != 0;
}
"""


def test_weight_walk_stays_in_the_blob(tmp_path):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", f"-DTAIL={TAIL}", "-I", build.CSRC, str(src), "-o", str(exe)],
                   check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout[:2000]


@pytest.mark.parametrize("c_in,c_out,thw,k", [(16, 32, (2, 7, 7), (1, 1, 1)), (16, 32, (2, 7, 7), (3, 3, 3)),
                                              (144, 130, (4, 14, 14), (1, 3, 3)), (512, 64, (8, 28, 28), (3, 1, 1)),
                                              (64, 96, (8, 28, 28), (3, 3, 3))])
def test_blobs_hold_the_bytes_behind_the_weights(c_in, c_out, thw, k, monkeypatch):
    monkeypatch.delenv("RT3D_TUNE", raising=False)
    build.build(force=False)
    d = rt3d.make_desc(1, c_in, c_out, thw, k, pad=tuple(v // 2 for v in k), dtype="bf16")
    blob, info = rt3d.rt3d_dense_pack(d, torch.zeros((c_out, c_in, *k), dtype=torch.bfloat16))
    a_off = int.from_bytes(bytes(info.plan)[104:112], "little")
    steps = k[0] * k[1] * k[2] * -(-c_in // 16)
    assert a_off > 0
    assert len(blob) >= a_off + -(-c_out // 64) * 2 * steps * 1024 + TAIL
