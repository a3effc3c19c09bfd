// Runtime-radix Stockham line kernels (any 7-smooth length that fits LDS).
//
// Same data decomposition as the power-of-two kernels -- a workgroup owns C
// lines, T threads per line, passes in Stockham autosort order -- but the
// radix sequence is read at run time, so one compiled instance serves every
// length (the ragged batches use hundreds of them).  Because the element sets
// of consecutive passes differ when the radix changes, every pass reads its
// inputs from LDS (the first pass from HBM) and writes its outputs back to LDS
// (the last pass to HBM), in place, with a barrier between the reads and the
// writes.  Pass twiddles w_{Ns R}^{k r} = w_L^{k r L/(Ns R)} are rebuilt from a
// two-level table of w_L made in FP64 on the host.
#include <string>

#include "mixed_device.h"
#include "real_pair.h"

namespace dpfft {

// longest line a workgroup transforms
constexpr int64_t kMixedMaxLine = 16384;

template <int MAP, int OMAP, int TW4, int SW>
__global__ void __launch_bounds__(1024) k_mixed(const cf *__restrict__ in, cf *__restrict__ out,
                                                MixedArgs a) {
  extern __shared__ cf lds[];
  const MixedPlan &mp = a.mp;
  const int tid = threadIdx.x;
  const uint32_t tile = (a.flags & F_REMAP) ? xcd_remap(blockIdx.x, gridDim.x) : blockIdx.x;
  const int64_t bb = tile / a.tiles_per_batch;
  const int64_t line0 = (int64_t)(tile - bb * a.tiles_per_batch) * mp.C;
  LineShape sh{mp.L, mp.T, mp.C, mp.pitch, mp.P, mp.tw2_shift, mp.codes, a.tw2,
               a.tw4_lo, a.tw4_hi, a.tw4_shift, a.scale, mp.tw_lds, a.lines};
  TileLine t;
  t.c = MAP == ELEM_FAST ? tid / mp.T : tid % mp.C;
  t.j = MAP == ELEM_FAST ? tid % mp.T : tid / mp.C;
  t.line0 = line0;
  t.line = line0 + t.c;
  t.valid = tid < mp.C * mp.T && t.line < a.lines;
  t.src = in + bb * a.in_b + t.line * a.in_l;
  t.dst = out + bb * a.out_b + t.line * a.out_l;
  t.in_e = a.in_e;
  t.out_e = a.out_e;
  t.c2 = OMAP == ELEM_FAST ? tid / mp.T : tid % mp.C;
  t.j2 = OMAP == ELEM_FAST ? tid % mp.T : tid / mp.C;
  t.valid2 = tid < mp.C * mp.T && line0 + t.c2 < a.lines;
  t.dst2 = out + bb * a.out_b + (line0 + t.c2) * a.out_l;
  mixed_tile<MAP, OMAP, TW4, SW>(sh, t, lds, mp.C * mp.T);
}

// Real rows: lines of N = 2L reals <-> L + 1 bins, L 7-smooth, the L-point
// transform of the samples read as complex pairs and the pairing of k with
// L - k in one launch (tw4_lo, tw4_hi: the two-level table of w_N).  Forward,
// every pass leaves its outputs in LDS and the pairing reads both elements
// of a pair there; inverse, the pairs are formed on the way in, swapped for
// the swap(FFT(swap)) form, and the first pass reads them from LDS.  A
// separate pairing launch moves the line through HBM once more: 16 images of
// 1080 x 1920: rows and pairing launches 53 + 41 us, 63 us fused (inverse 39 +
// 52 us, 70 us).
template <bool INV>
__global__ void __launch_bounds__(1024) k_mixed_real(const cf *__restrict__ in,
                                                     cf *__restrict__ out, MixedArgs a) {
  extern __shared__ cf lds[];
  const MixedPlan &mp = a.mp;
  const int tid = threadIdx.x, L = mp.L, T = mp.T;
  const int64_t bb = blockIdx.x / a.tiles_per_batch;
  const int64_t line0 = (int64_t)(blockIdx.x - bb * a.tiles_per_batch) * mp.C;
  const int c = tid / T, j = tid % T;
  const bool valid = tid < mp.C * T && line0 + c < a.lines;
  const cf *src = in + bb * a.in_b + (line0 + c) * a.in_l;
  cf *dst = out + bb * a.out_b + (line0 + c) * a.out_l;
  lcf *row = as_lds(lds) + c * mp.pitch;
  const uint32_t msk = (1u << a.tw4_shift) - 1u;
  auto wn = [&](int k) { return cmul(a.tw4_hi[(uint32_t)k >> a.tw4_shift], a.tw4_lo[(uint32_t)k & msk]); };

  lcf *twl = as_lds(lds) + mp.tw_lds;
  const int ntw = tw2_entries(L, mp.tw2_shift), nth = mp.C * T;
  int ntw0 = 0;  // table entries the first pass copies
  if constexpr (INV) {
    for (int i = tid; i < ntw; i += nth) stc(twl, i, a.tw2[i]);
    if (valid) {
      for (int k = j; k <= L / 2; k += T) {
        cf xk = src[k], xr = src[L - k], zk, zr;
        if (k == 0) xk.y = xr.y = 0.f;
        real_pair_inv(xk, xr, wn(k), zk, zr);
        stc(row, k + (k >> 4), cswap(zk));
        const int r = L - k;
        if (k != 0 && r != k) stc(row, r + (r >> 4), cswap(zr));
      }
    }
    __syncthreads();
  } else {
    ntw0 = ntw < nth ? ntw : nth;
    for (int i = tid + nth; i < ntw; i += nth) stc(twl, i, a.tw2[i]);
    if (mp.P == 0) {
      if (valid && j == 0) stc(row, 0, src[0]);
      __syncthreads();
    }
  }
  if (INV && mp.P == 0) {
    if (valid && j == 0) dst[0] = cscale(cswap(ldc(row, 0)), a.scale);
    return;
  }
  int ns = 1;
  for (int p = 0; p < mp.P; ++p) {
    const int R = (int)((mp.codes >> (5 * p)) & 31u);
    mixed_pass_any<ELEM_FAST, ELEM_FAST, TW4_NONE>(
        R, as_glb(src), as_glb(dst), as_lds(lds), twl, as_glb(a.tw2), ntw0, nullptr, nullptr, twl, L, T,
        mp.C, mp.pitch, ns, mp.tw2_shift, 0, c, j, valid, !INV && p == 0, INV && p == mp.P - 1,
        INV ? 2 : 0, 1, 1, 0, a.scale);
    ns *= R;
  }
  if constexpr (!INV) {
    if (valid) {
      for (int k = j; k <= L / 2; k += T) {
        const int r = L - k, rz = k == 0 ? 0 : r;
        cf xk, xr;
        real_pair_fwd(ldc(row, k + (k >> 4)), ldc(row, rz + (rz >> 4)), wn(k), xk, xr);
        dst[k] = xk;
        if (r != k) dst[r] = xr;
      }
    }
  }
}

const void *mixed_real_kernel(bool inverse) {
  return inverse ? (const void *)&k_mixed_real<true> : (const void *)&k_mixed_real<false>;
}

// ---------------------------------------------------------------------------
// host helpers
// ---------------------------------------------------------------------------
bool mixed_radices(int64_t L, MixedPlan *mp, int order, int tmax, int tmin) {
  if (L < 1 || L > kMixedMaxLine) return false;
  for (int64_t n = L; n > 1;) {
    const int p = n % 2 == 0 ? 2 : n % 3 == 0 ? 3 : n % 5 == 0 ? 5 : n % 7 == 0 ? 7 : 0;
    if (!p) return false;
    n /= p;
  }
  const RadixPlan r = radix_plan((int)L, order, tmax, tmin);
  if (r.T == 0) return false;
  mp->L = (int32_t)L;
  mp->P = r.P;
  mp->T = r.T;
  int ns = 1;
  mp->codes = 0;
  for (int p = 0; p < r.P; ++p) {
    mp->radix[p] = r.R[p];
    mp->ns[p] = ns;
    ns *= r.R[p];
    mp->codes |= (uint64_t)r.R[p] << (5 * p);
  }
  int lg = 0;
  while ((int64_t(1) << lg) < L) ++lg;
  mp->tw2_shift = (lg + 1) / 2;
  mp->pitch = (int32_t)(L + (L >> 4) + 1);
  return true;
}

bool mixed_covers(const MixedPlan &mp) {
  for (int p = 0; p < mp.P; ++p)
    if (mp.L / mp.radix[p] > mp.T * mixed_qmax(mp.radix[p])) return false;
  return true;
}

std::string mixed_factors(int64_t L) {
  int cnt[8] = {};
  for (int p : {2, 3, 5, 7})
    for (; L % p == 0; L /= p) ++cnt[p];
  std::string s;
  auto push = [&](int r, int times) {
    for (int i = 0; i < times; ++i) s += (s.empty() ? "" : "x") + std::to_string(r);
  };
  push(16, cnt[2] / 4);
  if (cnt[2] % 4) push(1 << (cnt[2] % 4), 1);
  push(7, cnt[7]);
  push(5, cnt[5]);
  push(9, cnt[3] / 2);
  push(3, cnt[3] % 2);
  return s;
}

int mixed_tile_elems(const MixedPlan &mp, int map, int omap) {
  auto need = [&](int m) {
    if (m == ELEM_FAST) return (int64_t)mp.C * mp.pitch;
    const int64_t u = (int64_t)mp.L * mp.C;
    return u + (u >> 4) + 1;
  };
  int64_t n = need(map);
  if (omap != map) n = n > need(omap) ? n : need(omap);
  return (int)n;
}

int mixed_lds_bytes(const MixedPlan &mp, int map, int omap, bool tw4) {
  return (mixed_tile_elems(mp, map, omap) + tw2_entries(mp.L, mp.tw2_shift) +
          (tw4 ? kFourStepVals * mp.C : 0)) * (int)sizeof(cf);
}

const void *mixed_kernel(int map, int omap, int tw4, int sw) {
#define MK(M, O, TW, S) \
  if (map == M && omap == O && tw4 == TW && sw == S) return (const void *)&k_mixed<M, O, TW, S>;
  // single-pass rows: forward, inverse (swap in+out), 2D row pass inverse (swap in)
  MK(ELEM_FAST, ELEM_FAST, TW4_NONE, 0)
  MK(ELEM_FAST, ELEM_FAST, TW4_NONE, 1)
  MK(ELEM_FAST, ELEM_FAST, TW4_NONE, 3)
  // column tiles: 2D column pass (fwd, inv = swap out), four-step first pass (fwd, swap in)
  MK(LINE_FAST, LINE_FAST, TW4_NONE, 0)
  MK(LINE_FAST, LINE_FAST, TW4_NONE, 2)
  MK(LINE_FAST, LINE_FAST, TW4_NONE, 3)
  MK(LINE_FAST, LINE_FAST, TW4_PLAIN, 0)
  MK(LINE_FAST, LINE_FAST, TW4_PLAIN, 1)
  MK(LINE_FAST, LINE_FAST, TW4_STREAM, 0)
  MK(LINE_FAST, LINE_FAST, TW4_STREAM, 1)
  // four-step second pass: rows stored transposed (fwd, swap out)
  MK(ELEM_FAST, LINE_FAST, TW4_NONE, 0)
  MK(ELEM_FAST, LINE_FAST, TW4_NONE, 2)
#undef MK
  return nullptr;
}

}  // namespace dpfft
