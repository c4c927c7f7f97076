"""Geometry of the forward transform's tiles on the CPU (csrc/fwd_tile.h,
compiled for the host): every output of a tile is formed once, and the
details of a 32 x 32 piece are summed in the same lanes and the same order
whether the tile is 32 or 64 a side, so that a problem's inner products do
not depend on the batch that sets the side."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2202_11945_amd", "csrc")

CHECK = r"""
#include "fwd_tile.h"
#include <cstdio>
#include <map>
#include <set>
#include <tuple>
#include <vector>
using namespace fewha;
constexpr int NT = 512;
// (piece, class, row and lane in it, level) -> the outputs that the lane adds, in order, in piece coordinates
typedef std::map<std::tuple<int, int, int, int>, std::vector<std::tuple<int, int>>> Order;
template <int T, int J>
bool level(Order& order) {
  using W = FwdWin<T>;
  constexpr int RL = W::run(J), D = W::D(J), D1 = W::D1(J);
  std::set<std::tuple<int, int>> high, low, rest;
  for (int u = 0; u < W::rounds(J, NT); ++u)
    for (int th = 0; th < NT; ++th) {
      const int wave = th / 64, lane = th % 64;
      const FwdPlace k = fwd_place<T, J>(wave * 64 + u * NT, lane);
      if (k.c < 0 || k.r < 0 || k.c >= W::W(J) || (k.on && k.r >= W::runs(J))) return false;  // reads stay inside
      if (!k.on) continue;
      if (k.cls != FWD_REST && (k.c >= D || RL * (k.r + 1) > D)) return false;
      for (int p = 0; p < RL; ++p) {
        const int y = RL * k.r + p;
        auto& seen = k.cls == FWD_HIGH ? high : k.cls == FWD_LOW ? low : rest;
        if (!seen.insert({y, k.c}).second) return false;
        if (k.cls == FWD_REST) continue;
        // details are formed in the first round, in the rows of lanes that k_fdwt_dir adds up for their piece
        const int piece = y / D1 * W::side + k.c / D1, q = lane / 16;
        const int cls_wave = k.cls == FWD_HIGH ? 0 : W::pieces;
        int i = 0;
        if (J == 3)
          i = wave == k.cls && q == piece ? 0 : 4;
        else
          while (i < 4 && !(W::wave_of(k.cls, piece, i) + cls_wave == wave && W::place_of(piece, i) == q)) ++i;
        if (u != 0 || i == 4) return false;
        order[{piece, k.cls, 16 * i + lane % 16, J}].push_back({y % D1, k.c % D1});
      }
    }
  // details once each; the coarse window from the low and the other columns, once each
  if ((int)high.size() != D * D || (int)low.size() != D * D) return false;
  for (const auto& e : low)
    if (!rest.insert(e).second) return false;
  return (int)rest.size() == W::W(J) * W::W(J);
}
template <int T>
bool tile(Order& o) {
  return level<T, 1>(o) && level<T, 2>(o) && level<T, 3>(o);
}
int main() {
  Order o32, o64, all;
  if (!tile<32>(o32) || !tile<64>(o64)) return std::puts("a tile's outputs"), 1;
  for (int piece = 0; piece < 4; ++piece)
    for (const auto& e : o32)
      all[{piece, std::get<1>(e.first), std::get<2>(e.first), std::get<3>(e.first)}] = e.second;
  if (all != o64) return std::puts("order of the sums"), 1;
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs a host compiler")
def test_forward_tiles_cover_and_sum_alike(tmp_path):
    src, exe = tmp_path / "check.cpp", tmp_path / "check"
    src.write_text(CHECK)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(exe), str(src)], check=True)
    res = subprocess.run([str(exe)], capture_output=True, text=True)
    assert res.returncode == 0, res.stdout
