// Runtime-radix Stockham transforms of 7-smooth lengths (radices of
// mixed_plan.h): argument blocks shared by the host planner and the device
// code.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "mixed_plan.h"

namespace dpfft {

// Radix plan of one line length L = prod radix[p].  Thread j of a line owns
// butterflies b = j + T*q of every pass, at most mixed_qmax(R) of them.
struct MixedPlan {
  int32_t L;
  int32_t P;                  // passes
  int32_t T;                  // threads per line
  int32_t C;                  // lines per workgroup
  int32_t radix[kMaxPasses];
  int32_t ns[kMaxPasses];     // product of the earlier radices
  int32_t tw2_shift;          // w_L^e = hi[e >> s] * lo[e & (2^s - 1)]
  int32_t pitch;              // LDS elements per line (ELEM_FAST layout)
  uint64_t codes;             // radix[p] in bits 5p..5p+4 (the device reads only this)
  int32_t tw_lds;             // LDS element offset of the pass-twiddle table
};

struct MixedArgs {
  MixedPlan mp;
  int64_t in_b, in_l, in_e;
  int64_t out_b, out_l, out_e;
  int64_t lines;             // lines per batch item
  int64_t tiles_per_batch;   // ceil(lines / C)
  const float2 *tw2;         // 2^s lo entries, then ceil(L / 2^s) hi entries
  const float2 *tw4_lo;      // four-step twiddles of N (two-level)
  const float2 *tw4_hi;
  int32_t tw4_shift;
  float scale;
  uint32_t flags;
};

// Fewest threads per line of short rows, whose lanes load T neighbouring
// elements at a time: with few threads a wave touches many lines at once and
// its L1 loses them before their next elements.  Without the bound a line of 10
// to 25 points is one radix of one thread (4 M points, no bound and bound: 12
// points 26.6 us, 20.2; 18, 29.5 and 19.4; 24, 30.0 and 18.7; 25, 31.2 and 21.4;
// 64 M points of 24, 468 us and 324).  20 points keep two threads: three do not
// divide 5 x 4 (64 M points 7% slower).
constexpr int mixed_row_tmin(int64_t L) { return L < 10 ? 1 : L > 16 && L != 20 ? 3 : 2; }

// The same for batches of rows, where it shows up to 360 points (4 M points: 56
// points 18.7 us, 16.1; 80, 19.2 and 17.4; 120, 20.4 and 15.9; 64 M points of 288,
// 232 and 184), as the most points per thread.  Longer lines have enough
// threads, and a bound would cost them the wide radices (375 points: 38 threads
// take 20% more than 25); so would 10 points per thread at 98 and 105 (14 x 7
// and 15 x 7 from 7 and 8 threads: 10% and 15%) and at 48 (12 x 4, 8%).
constexpr int mixed_rows_tmin(int64_t L) {
  const int64_t most = L <= 48 ? 12 : L <= 96 ? 10 : L <= 120 ? 14 : 20;
  const int t = L <= 360 ? (int)((L + most - 1) / most) : 1;
  return t > mixed_row_tmin(L) ? t : mixed_row_tmin(L);
}

// Host: radix plan of a 7-smooth L (radix_plan of mixed_plan.h) with tmin to
// tmax threads per line; order 0: largest radix first, 1: smallest first.
// Returns false if L has a prime factor above 7 or no plan within those.
bool mixed_radices(int64_t L, MixedPlan *mp, int order = 0, int tmax = 1024, int tmin = 1);

// Host: whether every pass's butterflies are owned by the plan's threads.
bool mixed_covers(const MixedPlan &mp);

// Host: the factorization of a 7-smooth L into the elementary radices (16s,
// then 8/4/2, then 7, 5, 9 for pairs of 3, 3), as "16x7x3"; the passes run
// products of them.
std::string mixed_factors(int64_t L);

// Four-step twiddle of a column step: none, applied, applied with streamed
// stores (tiles of whole 128-byte lines only: with 64-byte pieces, 8 columns
// of 1000 x 1000, they took 281 us against 268).
enum : int { TW4_NONE = 0, TW4_PLAIN = 1, TW4_STREAM = 2 };

// Host: the kernel instance for (map, omap, TW4_*, swap mode); nullptr if none.
const void *mixed_kernel(int map, int omap, int tw4, int sw);

// Host: the real-row kernel (N = 2L reals -> L + 1 bins, or the inverse).
const void *mixed_real_kernel(bool inverse);

// LDS elements of the tile data of a workgroup, and total LDS bytes (tile
// data, the pass-twiddle table that follows it and, for column tiles with the
// four-step twiddle, kFourStepVals values per line).
constexpr int kFourStepVals = 5;
int mixed_tile_elems(const MixedPlan &mp, int map, int omap);
int mixed_lds_bytes(const MixedPlan &mp, int map, int omap, bool tw4);

}  // namespace dpfft
