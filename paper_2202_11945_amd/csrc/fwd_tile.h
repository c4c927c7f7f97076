// Geometry of the forward transform's three-level tiles (k_fdwt_dir): plain
// constant expressions, so that the host can check them.
#pragma once

namespace fewha {

// Windows, LDS strides and column tasks of a T x T input tile (T = 32 or 64).
template <int T>
struct FwdWin {
  static constexpr int D(int j) { return T >> j; }                     // detail outputs per direction
  // coarse window (W(0): the input): W(3) = T / 8, W(j) = 2 W(j + 1) + 4
  static constexpr int W(int j) { return (T >> j) + 4 * ((8 >> j) - 1); }
  static constexpr int SR(int j) { return W(j) + D(j) + 1; }          // LDS stride of the row pass's output
  static constexpr int SX(int j) { return W(j) + 1; }                 // ... of the coarse window
  // output pairs of a task: four at the finest level, as few as the threads
  // allow below (a pass there costs its latency, not its reads)
  static constexpr int run(int j) { return j == 1 ? 4 : j == 2 ? 2 : 1; }
  static constexpr int runs(int j) { return W(j) / run(j); }
  // Column tasks, each a column and a run of pairs, in classes of whole
  // waves: x-high columns (both halves in y are details), x-low columns
  // under the tile (coarse and detail), the rest of the coarse window.
  //
  // The details of a 32 x 32 piece of the tile lie in the same lanes for
  // either T: at the finest level in 4 rows of 16 lanes of each of the first
  // two classes, at the second in 2 of the same rows, at the third in a row
  // of its own (row p of the first two waves is piece p).  k_fdwt_dir sums
  // every row by itself and the rows of a piece in turn, so a layer's inner
  // products do not depend on the tile side, which the number of tiles in a
  // launch decides.
  static constexpr int side = T / 32, pieces = side * side;
  static constexpr int D1(int j) { return 32 >> j; }                   // a piece's detail outputs per direction
  static constexpr int rows(int j) { return D1(j) * D1(j) / run(j) / 16; }
  static constexpr int at_rest = 2 * 64 * pieces;
  static constexpr int rest(int j) { return W(j) * runs(j) - 16 * pieces * rows(j); }
  // levels 1 and 2, row i of a piece: its wave within the class (T = 64: the second class's
  // waves in pairs swapped, so that level 2, which takes every other one,
  // has the two classes on different SIMDs), its place in the wave
  static constexpr int turn(int cls) { return T == 64 ? cls : 0; }
  static constexpr int wave_of(int cls, int piece, int i) {
    return T == 32 ? 0 : (2 * (piece / side) + i / 2) ^ turn(cls);
  }
  static constexpr int place_of(int piece, int i) { return T == 32 ? i : 2 * (i % 2) + piece % side; }
  // T = 64: level 2 leaves every other wave of the first class to the rest
  static constexpr bool between(int j) { return T == 64 && j == 2; }
  static constexpr int rounds(int j, int nt) { return between(j) || j == 3 ? 1 : (at_rest + rest(j) + nt - 1) / nt; }
};

enum { FWD_HIGH, FWD_LOW, FWD_REST };

// The column task of level J at place w0 + lane (w0: a multiple of 64): its
// class, column c and run r of pairs.
struct FwdPlace {
  int cls;
  bool on;
  int c, r;
};
template <int T, int J>
constexpr FwdPlace fwd_place(int w0, int lane) {
  using W = FwdWin<T>;
  constexpr int D1 = W::D1(J), R1 = D1 / W::run(J);
  if (J == 3) {  // no rest
    const int piece = lane / 16, l = lane % 16;
    const bool on = w0 < 2 * 64 && piece < W::pieces;
    return FwdPlace{w0 == 0 ? FWD_HIGH : FWD_LOW, on, on ? D1 * (piece % W::side) + l % D1 : 0,
                    on ? R1 * (piece / W::side) + l / D1 : 0};
  }
  static_assert(!W::between(J) || W::rest(J) <= 64 * W::side, "the rest fits the waves left to it");
  const bool between = W::between(J) && w0 < W::at_rest / 2 && w0 / 64 % 2 == 1;
  if (w0 < W::at_rest && !between) {
    const int cls = w0 < W::at_rest / 2 ? FWD_HIGH : FWD_LOW;
    const int w = (w0 / 64 % W::pieces) ^ W::turn(cls);
    if (J == 1)  // two runs of a 64 tile's columns, four of a 32 tile's
      return FwdPlace{cls, true, T == 32 ? lane % 16 : lane % 32, T == 32 ? lane / 16 : 2 * w + lane / 32};
    const int q = lane / 16, l = lane % 16;
    const int i = T == 32 ? q : 2 * (w % 2) + q / 2;  // row of the piece
    const int py = T == 32 ? 0 : w / 2, px = T == 32 ? 0 : q % 2;
    const bool on = i < W::rows(J);
    return FwdPlace{cls, on, D1 * px + l % D1,
                    on ? R1 * py + i * (16 / D1) + l / D1 : 0};
  }
  // columns past the tile in its runs, then every column in the runs past it
  constexpr int D = W::D(J), past = W::W(J) - D, first = past * (D / W::run(J)), p = past > 0 ? past : 1;
  const int e = (between ? w0 / 128 * 64 : w0 - W::at_rest) + lane;
  const bool on = e < W::rest(J);
  return FwdPlace{FWD_REST, on, !on ? 0 : e < first ? D + e % p : (e - first) % W::W(J),
                  !on ? 0 : e < first ? e / p : D / W::run(J) + (e - first) / W::W(J)};
}

}  // namespace fewha
