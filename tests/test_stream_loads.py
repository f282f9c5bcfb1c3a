"""The load bookkeeping of the Gram form's tile ring (stream_loads.h), replayed
on the host for every wave, d_h, weight type, kind of start vectors and
alignment: when a wave goes on to tile i, its loads of that tile have landed
whatever the order in which later ones complete, and the loads of the tiles
requested after it stay in flight."""

import os
import shutil
import subprocess

import pytest

from conftest import ROOT

PROGRAM = r"""
#include <cstdio>
#include <deque>
#include "stream_loads.h"
using namespace sn;

int main() {
  long checked = 0;
  for (int dh : {16, 32, 64, 128})
    for (int es : {2, 4})
      for (int vst : {0, 1024, 2048})
        for (int vec = 0; vec < 2; ++vec)
          for (int heads = vst ? 1 : 0; heads <= (vst == 0 ? 0 : vst == 1024 ? 1 : es == 2 ? 8 : 16); ++heads)
            for (int n = 1; n <= 20; ++n) {
              const int nst = ring_slots(dh, vst), nvi = vst ? vector_instructions(es, vec, heads) : 0;
              int rows = 0, instructions = 0;  // of one tile, over the waves
              for (int wv = 0; wv < kHWaves; ++wv) {
                const int own = tile_loads(dh, wv) + (vst ? vector_loads(nvi, wv) : 0);
                if (own > tile_loads(dh, 0) + (vst ? 2 : 0)) return printf("dh %d wave %d: %d loads\n", dh, wv, own), 1;
                rows += tile_loads(dh, wv);
                std::deque<int> queue;  // tiles of the outstanding loads, oldest first
                auto issue = [&](int i) {
                  for (int x = 0; x < tile_loads(dh, wv); ++x) queue.push_back(i);
                  int mine = 0;
                  for (int x = vector_first(wv); x < nvi; x += kHWaves) queue.push_back(i), ++mine;
                  if (i == 0) instructions += mine;
                };
                for (int i = 0; i < nst - 1 && i < n; ++i) issue(i);
                for (int i = 0; i < n; ++i) {
                  const bool ahead = i + nst - 2 < n;
                  const size_t most = ahead ? outstanding_ahead(nst, own) : 0, before = queue.size();
                  if (most > 63) return printf("count %zu\n", most), 1;
                  while (queue.size() > most) queue.pop_front();
                  if (!queue.empty() && queue.front() <= i)
                    return printf("dh %d es %d vst %d vec %d heads %d n %d wave %d: a load of tile %d is outstanding at %d\n",
                                  dh, es, vst, vec, heads, n, wv, queue.front(), i), 1;
                  if (ahead && before > 0 && queue.size() != (size_t)((nst - 2) * own))
                    return printf("dh %d wave %d: loads of later tiles waited for\n", dh, wv), 1;
                  if (i + nst - 1 < n) issue(i + nst - 1);
                  ++checked;
                }
              }
              if (rows * 1024 != tile_bytes(dh) || instructions != nvi) return printf("dh %d: loads missing\n", dh), 1;
              if (vst && nvi * vector_rows_per_load(es, vec) * (128 / es * 4) > vst) return printf("vst\n"), 1;
            }
  printf("%ld\n", checked);
  return 0;
}
"""


def test_every_load_has_landed_before_its_tile_is_used(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("needs a host C++ compiler")
    src, exe = tmp_path / "replay.cpp", tmp_path / "replay"
    src.write_text(PROGRAM)
    subprocess.run([cxx, "-std=c++17", "-I" + os.path.join(ROOT, "paper_2602_18851_amd", "csrc"), "-o", str(exe),
                    str(src)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
    assert int(res.stdout) > 10000
