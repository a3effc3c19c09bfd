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

// Host: radix plan of a 7-smooth L (radix_plan of mixed_plan.h) with at most
// tmax threads per line; order 0: largest radix first, 1: smallest first.
// Returns false if L has a prime factor above 7 or no plan within tmax.
bool mixed_radices(int64_t L, MixedPlan *mp, int order = 0, int tmax = 1024);

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
