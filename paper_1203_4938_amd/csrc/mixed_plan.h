// Radix plans of the runtime-radix transforms: which radices, in which order,
// and how many threads per line.  Constant expressions, so the compile-time
// ragged tiles and the host planner take the same plan for a length.
#pragma once
#include <stdint.h>

namespace dpfft {

constexpr int kMaxPasses = 12;

// Radices with a device pass.  The composite ones run as products of their
// factors in registers (coprime factors without twiddles), so most lines of up
// to 625 points take two passes through LDS (243, 343, 512 and 560 three) and
// most of up to 15625 three (11760 four, 12005 five).
constexpr int kMixedRadices[] = {25, 24, 21, 20, 18, 16, 15, 14, 12, 10, 9, 8, 7, 6, 5, 4, 3, 2};
constexpr int kNumMixedRadices = sizeof(kMixedRadices) / sizeof(int);

// Butterflies of one pass a thread may own (16 to 25 elements in registers).
constexpr int mixed_qmax(int R) { return R >= 14 ? 1 : R >= 10 ? 2 : (16 + R - 1) / R; }

struct RadixPlan {
  int P = 0;                 // passes
  int T = 0;                 // threads per line
  int R[kMaxPasses] = {};
  int64_t cost = -1;
};

namespace rplan {
// Vector instructions of a radix-R butterfly, roughly.
constexpr int butterfly_ops(int R) {
  switch (R) {
    case 2: return 4;
    case 3: return 16;
    case 4: return 16;
    case 5: return 40;
    case 6: return 44;
    case 7: return 84;
    case 8: return 56;
    case 9: return 120;
    case 10: return 100;
    case 12: return 112;
    case 14: return 196;
    case 15: return 200;
    case 16: return 170;
    case 18: return 276;
    case 20: return 240;
    case 21: return 364;
    case 24: return 296;
    case 25: return 460;
  }
  return 1000;
}

constexpr int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Share (in threads) of a CU's 16 waves (the passes take up to 128 registers)
// that a line's workgroup holds: 256 threads' worth of lines or, above, one
// line, in whole waves, and what is left over when no further workgroup fits.
constexpr int64_t wave_share(int T) {
  const int C = T < 256 ? 256 / T : 1, w = ceil_div(C * T, 64);
  return 64 * 16 / (16 / w) / C;
}

// Modelled time of one line with T threads: every pass costs its latency
// (LDS round trip and barrier) plus its butterflies, on the waves the line
// holds.  Of the weights tried (pass 100, 200, 500, 800; a fixed cost per tile
// of 0 to 3000) these gave the fastest plans: 720-point rows 146 us against
// 172 for 50 M points, 60-point rows 214 against 240, within 2% elsewhere.
constexpr int64_t kPassCost = 100, kElemCost = 20;
constexpr int64_t plan_cost(int L, const int *R, int P, int T) {
  int64_t c = 0;
  for (int p = 0; p < P; ++p) {
    const int q = ceil_div(L / R[p], T);
    if (q > mixed_qmax(R[p])) return -1;
    c += kPassCost + (int64_t)q * (kElemCost * R[p] + butterfly_ops(R[p]));
  }
  return c * wave_share(T);
}

struct Search {
  int L, tmax, tmin;
  RadixPlan best;
  int R[kMaxPasses] = {};
  // all multisets of `left` radices, none before kMixedRadices[i0], with product n
  constexpr void run(int n, int i0, int p, int left) {
    if (left == 0) {
      if (n == 1) finish(p);
      return;
    }
    for (int i = i0; i < kNumMixedRadices; ++i) {
      const int r = kMixedRadices[i];
      if (n % r) continue;
      int64_t top = 1;  // the rest must be reachable with radices <= r
      for (int k = 0; k < left && top < n; ++k) top *= r;
      if (top < n) break;
      R[p] = r;
      run(n / r, i, p + 1, left - 1);
    }
  }
  constexpr void finish(int P) {
    for (int p = 0; p < P; ++p)
      for (int q = 1; q <= mixed_qmax(R[p]); ++q) {
        const int T = ceil_div(L / R[p], q);
        if (T > tmax || T < tmin) continue;
        const int64_t c = plan_cost(L, R, P, T);
        if (c < 0 || (best.cost >= 0 && c >= best.cost)) continue;
        best.cost = c;
        best.P = P;
        best.T = T;
        for (int k = 0; k < P; ++k) best.R[k] = R[k];
      }
  }
};
}  // namespace rplan

// The plan of a 7-smooth L with tmin to tmax threads per line (tmax >=
// ceil(L / 16)): the cheapest of the fewest passes, or of one pass more where
// those leave much of a CU unused.  Largest radix first (the first pass has no
// twiddles); order 1 takes the same radices smallest first.  P = 0 with T = 0
// if there is none (L = 1 has P = 0 and T = 1).
constexpr RadixPlan radix_plan(int L, int order, int tmax, int tmin = 1) {
  if (L == 1) {
    RadixPlan one;
    one.T = 1;
    return one;
  }
  rplan::Search s{L, tmax, tmin, {}};
  int P = 1;
  for (; P <= kMaxPasses && s.best.cost < 0; ++P) s.run(L, 0, 0, P);
  // a pass more may need fewer threads, and so leave less of a CU unused:
  // 4900 points in three passes of 350 threads 258 us for 50 M points, in four
  // of 245 threads 212 (with a fuller CU fewer passes win: 5880 points, both 420
  // threads, 213 us in three and 270 in four)
  const RadixPlan few = s.best;
  if (few.T > 0 && 4 * few.T < 3 * rplan::wave_share(few.T)) {
    s.run(L, 0, 0, P);
    if (rplan::wave_share(s.best.T) >= rplan::wave_share(few.T)) s.best = few;
  }
  RadixPlan r = s.best;
  if (order == 1)
    for (int p = 0; p < r.P / 2; ++p) {
      const int t = r.R[p];
      r.R[p] = r.R[r.P - 1 - p];
      r.R[r.P - 1 - p] = t;
    }
  return r;
}

}  // namespace dpfft
