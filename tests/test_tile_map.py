"""The map from workgroups to row tiles of the one-vector step's dot and update
passes (csrc/tilemap.h) and the row chunks of the block process
(csrc/rowchunks.h), on the CPU: every (tile, launch position, index) is
taken exactly once, workgroups that share a tile stay on one XCD where the map
keeps them there, and no XCD is left with much more than its share."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_0704_3486_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <set>
#include <tuple>
#include "tilemap.h"

template <bool DOWN, bool BY_XCD>
int check(int nt, int nb, int nk, double most, int rows) {
  const unsigned per = nb * nk;
  const size_t grid = tile_grid(per, nt, rows, BY_XCD);
  std::set<std::tuple<int, int, int>> seen;
  int load[kXcds] = {}, prev = DOWN ? nt : -1;
  for (size_t i = 0; i < grid; ++i) {
    int t = -1, z = -1, in = -1;
    if (!tile_of<DOWN, BY_XCD>((unsigned)i, per, nb, nt, rows, t, z, in)) continue;
    if (t < 0 || t >= nt || z < 0 || z >= nb || in < 0 || in >= nk) return 1;
    if (!seen.insert({t, z, in}).second) return 2;
    ++load[i % kXcds];
    // the walk goes by groups of kXcds tiles (dealt out: by tiles)
    const bool dealt = !BY_XCD && dealt_out(nt, rows);
    const int g = dealt ? t : t / kXcds, p = dealt ? prev : (prev < 0 ? -1 : prev / kXcds);
    if (prev >= 0 && prev < nt && (DOWN ? g > p : g < p)) return 3;
    prev = t;
  }
  if (seen.size() != (size_t)nt * nb * nk) return 4;
  int mx = 0;
  for (int l : load) mx = l > mx ? l : mx;
  return mx > most * ((double)nt * nb * nk / kXcds) + 1.0 ? 5 : 0;
}

int main() {
  for (int nt = 1; nt <= 140; ++nt)
    for (int nb : {1, 2, 3, 5, 8, 64})
      for (int nk : {1, 3, 8}) {
        int r = 0;
        for (int rows : {512 * nt, 512 * nt - 496}) {  // a full last tile, and one of 16 rows
          // 25 tiles by XCD: four where the share is 3.125
          if (!r) r = check<false, false>(nt, nb, nk, 1.28, rows);
          if (!r) r = check<true, false>(nt, nb, nk, 1.28, rows);
          if (!r && nt > kXcds) r = check<true, true>(nt, nb, nk, 8.0, rows);
          // up to eight tiles: no XCD idles for the lack of an eighth of the rows
          if (!r && nt <= kXcds && !dealt_out(nt, rows) && 8 * rows < 7 * kXcds * kTileRows) r = 6;
        }
        if (r) return printf("tiles %d slots %d index %d: %d\n", nt, nb, nk, r), 1;
      }
  return 0;
}
"""


def test_every_tile_once_and_even_shares(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "d.cpp", tmp_path / "d"
    src.write_text(DRIVER)
    subprocess.run([cxx, "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


CHUNKS = r"""
#include <cstdio>
#include "rowchunks.h"

int main() {
  for (int V = 16; V <= 200000; V += V < 12000 ? 1 : 7) {
    const int N = 12 * V;
    int rpw = 0;
    const int nch = row_chunks(N, rpw), up = update_chunk(rpw);
    if (nch < 1 || nch > (N < kSmallRows ? 48 : 128) || rpw % 8 || (long long)nch * 4 * rpw < N ||
        (long long)(nch - 1) * 4 * rpw >= N)
      return printf("rows %d: %d chunks of 4 x %d\n", N, nch, rpw), 1;
    // the update's chunks hold whole workgroups, and are the dot pass's where those do
    if (up % 128 || up < 4 * rpw || up >= 4 * rpw + 128 || (rpw % 32 == 0 && up != 4 * rpw))
      return printf("rows %d: update chunks of %d rows\n", N, up), 1;
    // large lattices: 128 chunks but for rounding their rows up to whole lines, so an XCD takes at most
    // 16 chunks of 4 (N / 512 + 8) rows, 1 + 4096 / N times an eighth of N
    if (N > 65536 && 16.0 * 4 * rpw > (1.0 + 4096.0 / N) * N / 8)
      return printf("rows %d: %d chunks\n", N, nch), 1;
  }
  int rpw = 0;
  if (row_chunks(12 * 20736, rpw) != 128) return printf("12^4: %d rows a wavefront\n", rpw), 1;
  return 0;
}
"""


def test_row_chunks(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "c.cpp", tmp_path / "c"
    src.write_text(CHUNKS)
    subprocess.run([cxx, "-O1", "-std=c++17", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
