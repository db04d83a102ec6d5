"""Host replay of the tile condensation's copies of a basis row (cc_tile.h, the
index arithmetic that prep_tile_body itself uses): the first fill of every
segment and the refill of every chunk, a word at a time.  Every word read lies in
the row or in the DENSE_F32_PAD floats past it, which every float32 dense basis
has, and every position a band row needs is in its slot when the row is taken.
Around whole rings, with one and two segments, all three configurations."""
import ctypes
import subprocess

import pytest

SOURCE = r"""
#define __host__
#define __device__
#include "cc_tile.h"
#include <algorithm>
#include <vector>
using namespace cc;

// Words that the copies of one row read past its end; -1: a position that a
// band row needs was not in its slot.
extern "C" int replay(int cfg, int nf, int bw, int nseg) {
  const int CH = TILE_CH[cfg - 1], R = tile_ring(cfg, nf, bw), row = nf * 9;
  int past = 0;
  for (int seg = 0; seg < nseg; ++seg) {
    const int pa = tile_segment(nf, R, seg, nseg), pb = std::min(nf, tile_segment(nf, R, seg + 1, nseg));
    std::vector<int> ring(R * 9);                    // the row's word in each of the ring's
    auto copy = [&](int to, int from) {
      for (int i = 0; i < TILE_PIECE; ++i) {
        past = std::max(past, from + i + 1 - row);
        ring[to + i] = from + i;
      }
    };
    for (int k = 0; k < R * 9 / TILE_PIECE; ++k) copy(k * TILE_PIECE, (int)tile_fill_piece(pa, k, nf));
    int slot = 0;
    for (int p0 = pa; p0 < pb; p0 += CH) {
      for (int p = p0; p < std::min(p0 + CH, nf); ++p)
        for (int k = p; k <= std::min(nf - 1, p + bw); ++k)
          for (int c = 0; c < 9; ++c)
            if (ring[k % R * 9 + c] != k * 9 + c) return -1;
      if (p0 + R < nf && p0 + CH < pb) {
        for (int k = 0; k < CH * 9 / TILE_PIECE; ++k)
          copy(slot * 9 + k * TILE_PIECE, (int)(tile_piece(p0 + R, 0) + tile_piece(0, k)));
        slot = (slot + CH) % R;
      }
    }
  }
  return past;
}
extern "C" int pad() { return DENSE_F32_PAD; }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    import paper_2510_12053_amd.build as build
    d = tmp_path_factory.mktemp("tile")
    (d / "replay.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I", build.CSRC, str(d / "replay.cpp"), "-o",
                    str(d / "replay.so")], check=True)
    return ctypes.CDLL(str(d / "replay.so"))


@pytest.mark.parametrize("nseg", [1, 2])
@pytest.mark.parametrize("cfg,bands", [(1, (0, 40, 128)), (2, (5, 256, 289, 482, 640)), (3, (5, 121, 300, 700))])
def test_copies_stay_in_the_basis(lib, cfg, bands, nseg):
    for bw in bands:
        for rings in (64, 128, 192, 256, 384, 512, 768, 867, 896, 1024, 1536, 2304):
            for nf in (rings - 1, rings, rings + 1, rings + 6, rings + 63):
                past = lib.replay(cfg, nf, min(bw, nf - 1), nseg)
                assert 0 <= past <= lib.pad(), (cfg, nf, bw, nseg, past)
