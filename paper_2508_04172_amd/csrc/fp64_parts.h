// How a batch of the FP64 contraction is dealt to its tiles: the rules on
// sizes, and what of the basis rows each part may read.  Host code, compiled on
// its own by the CPU tests.
#pragma once

#include <algorithm>

#include "rbfl_internal.h"

namespace rbfl {

// Tiles of the FP64 contraction by a batch's count of 32 x 32 output tiles: below
// kTinyTiles 32 x 32 (k_gemm_small_fp64), below kMidTiles 64 x 64 (variant 4's),
// from there on the handle's variant.  A large tile waits for one workgroup's
// chain of chunks while there is less than a round of them (64 x 128, 808 rows:
// 75-79 us for 512 to 1021 proposals of 1280 columns, 33 and 50 us with 32 x 32
// tiles), and its last rounds are coarse; a wave with one 16 x 16 tile reads as
// much LDS as it multiplies.  us for 32 x 32 / 64 x 64 / best large tile, 808
// rows x 1280 columns: 88 / 95 / 117 at 2048 proposals (2560 tiles), 129 / 118 /
// 118 at 3000 (3760), 331 / 288 / 316 at 8192, 633 / 519 / 526 at 16384 (20480);
// 3008 rows x 2560 columns: 299 / 329 / 411 at 1021 (2560), 435 / 408 / 413 at
// 1500 (3760), 1138 / 982 / 1152 at 4000, 2343 / 1922 / 1921 at 8192 (20480).
// All give the same bits.
constexpr int64_t kTinyTiles = 2880, kMidTiles = 22000;
inline int64_t tiles32(const EvalConsts &hc, int64_t nb) { return (nb + 31) / 32 * col_tiles(hc, 32); }

// How many of a batch's first proposals the variant's tile takes; the rest goes
// to the smaller ones.  None below kMidTiles.  The 8-wave tiles (256 x 128, one
// workgroup per CU; 128 x 128, two) leave half the chip idle in a short last
// round, so they hand it over where the smaller tiles take less: with two per CU
// up to 0.4 of a round (which would cost half of one) and from 0.5 to 0.75 (a
// whole one): 7.30 to 6.84 ms at 30011 proposals of 3008 rows and 2560 columns
// (9.2 rounds).
inline int64_t main_part(const EvalConsts &hc, int64_t nb, int variant) {
  if (tiles32(hc, nb) < kMidTiles) return 0;
  if (variant != 5 && variant != 6) return nb;
  const int64_t qt = variant == 5 ? 256 : 128, round = variant == 5 ? 256 : 512, n_ct = hc.Kp / 128;
  const int64_t tiles = (nb + qt - 1) / qt * n_ct, rest = tiles % round;
  const bool hand_over = 4 * rest < 3 * round && (variant == 5 || 5 * rest < 2 * round || 2 * rest > round);
  return hand_over ? std::min(nb, (tiles - rest) / n_ct * qt) : nb;
}

// One launch of the contraction: proposals first .. first + count - 1 of a batch
// whose basis rows are Bt[r][q], q < rows_ld(batch).  Its tiles may load entries
// first .. first + read_end - 1 of a row: past the part's last proposal they load
// zeros only, never the next row or, of the last row, what lies behind it.
struct Fp64Part {
  int64_t first, count, read_end;
};
struct Fp64Parts {
  Fp64Part main, rest;      // the variant's tile; the smaller ones
};
// pinned: the variant's tile takes the whole batch whatever its size.
inline Fp64Parts fp64_parts(const EvalConsts &hc, int64_t nb, int variant, bool pinned) {
  const int64_t n1 = pinned ? nb : main_part(hc, nb, variant);   // a whole number of tiles, or the batch
  return {{0, n1, rows_ld(n1)}, {n1, nb - n1, rows_ld(nb - n1)}};
}

}  // namespace rbfl
