// The four-step core of long real-input transforms with the pairing of bins
// inside it (N = 2L reals, L = N1 N2 a power of two; see real_pair.h).
//
// Forward, second pass.  Row k1 of the intermediate becomes Z[k1 + N1 k2], and
// bin k = k1 + N1 k2 pairs with L - k = (N1 - k1) + N1 (N2 - 1 - k2): rows k1 and
// N1 - k1 hold each other's partners, in reverse order.  A tile therefore takes
// C/2 rows and their C/2 mirrors, leaves the transformed rows in LDS as every
// transposed store does, and reads both elements of a pair there.  Rows 0 and
// N1/2 are their own mirrors (row 0 pairs k2 with N2 - k2) and share the first
// tile's lines 0 and C/2.
//
// Inverse, first pass.  Column n2 of the bins, read as the matrix X[n1 N2 +
// n2], pairs (n1, n2) with (N1 - 1 - n1, N2 - n2): the tile takes C/2 columns
// and their mirrors, exchanges the raw bins through LDS, forms the values whose
// inverse transform holds the samples, and goes on as the column pass does.
//
// Either way the separate launch that moved the whole core through HBM once
// more is gone: 64 signals of 2^20 samples, forward 322 us in three
// launches, 264 in two (294 with ordinary loads of the rows); inverse 321, 260.  HBM bounds the
// kernels.  Row pieces are C/2 elements wide, and the bins' rows start at any
// 8-byte offset, so the forward pieces straddle lines and the store bounds that
// kernel: 512-point lines take tiles of 32 (128-byte pieces; with 16, forward
// 195 us and inverse 142), lines of 1024 fit only 16 (64 bytes: 32 signals of
// 2^22 samples, 399 us forward where the unpaired rows and the pairing took 452).
// The rows' loads are non-temporal (rows_nt) where the core is about as large as
// the 256 MiB last-level cache, so that its lines stay for the bins.
// One workgroup fits a CU, so the kernels are persistent and prefetch the next
// tile like the other 1024-point tiles.
#include "line_device.h"
#include "real.h"
#include "real_pair.h"

namespace dpfft {

// Pass twiddles of these instances: as the persistent line kernels hold them.
template <int L, int C, int MAP, int OMAP, int EPT>
struct PairedTw {
  static constexpr bool DIRECT = pf_direct_tw<L, C, MAP, OMAP, EPT>();
  static constexpr bool FIRST = pf_first_tw<L, C, MAP, OMAP, EPT>();
  static constexpr int NTW = pf_tw_entries<L, C, MAP, OMAP, EPT>();
  static constexpr int N2L = pf_tw2_entries<L, EPT>();
  static constexpr int NLO = 1 << tw2_shift(P2<L>::LG);
  using type = std::conditional_t<DIRECT, TwLdsTable, std::conditional_t<FIRST, TwLdsFirst, TwLds2>>;
  __device__ static void fill(cf *twl, const cf *tw, const cf *tw2, int tid, int nth) {
    for (int i = tid; i < NTW; i += nth) twl[i] = DIRECT ? tw[i] : i < N2L ? tw2[i] : tw[i - N2L];
  }
  __device__ static type make(const cf *twl) {
    if constexpr (DIRECT) {
      return TwLdsTable{twl};
    } else if constexpr (FIRST) {
      return TwLdsFirst{twl + N2L, TwLds2{twl, twl + NLO}};
    } else {
      return TwLds2{twl, twl + NLO};
    }
  }
};

// row (column) of line c of tile t: C/2 from t C/2 on, then their mirrors
template <int C>
__device__ __forceinline__ uint32_t paired_line(uint32_t t, int c, uint32_t n) {
  constexpr uint32_t H = C / 2;
  if (c < (int)H) return t * H + (uint32_t)c;
  return t == 0 && c == (int)H ? n / 2 : n - t * H - ((uint32_t)c - H);
}

// First slot and stride of the persistent walk: every XCD sweeps a contiguous
// slice of each round.
__device__ __forceinline__ uint32_t paired_slot() {
  const uint32_t g = gridDim.x, b = blockIdx.x;
  return g % 8u == 0u ? (b % 8u) * (g / 8u) + b / 8u : b;
}

template <int L, int C, int EPT, int NT>
__global__ void __launch_bounds__(C * (P2<L, EPT>::T))
    k_real_rows(const cf *__restrict__ in, cf *__restrict__ out, RealFourArgs a) {
  using G = P2<L, EPT>;
  constexpr int E = G::E, T = G::T, NTH = C * T, H = C / 2, STEP = NTH / H;
  static_assert(NTH <= 1024 && L % STEP == 0, "whole rounds of pairs");
  using TW = PairedTw<L, C, ELEM_FAST, LINE_FAST, EPT>;
  using LO = Lds<L, C, LINE_FAST, kPadShift>;
  __shared__ __align__(16) cf lds[lds_pairs<L, C, ELEM_FAST, LINE_FAST>()];
  __shared__ cf twl[TW::NTW], whi[L];  // whi: w_N^{n k2}, k2 < L
  const int tid = threadIdx.x;
  TW::fill(twl, a.tw, a.tw2, tid, NTH);
  for (int i = tid; i < L; i += NTH) whi[i] = a.whi[i];
  __syncthreads();
  const typename TW::type tw = TW::make(twl);
  int c, j;
  lane_map<L, EPT, C, ELEM_FAST>(tid, c, j);
  const uint32_t n = a.n, tpb = n / C, nt = a.ntiles, Gd = gridDim.x;
  uint32_t tile = paired_slot();
  if (tile >= nt) return;

  cf v[E], vn[E];
  auto load = [&](uint32_t tl, cf(&x)[E]) {
    const uint32_t bb = tl / tpb, t = tl - bb * tpb;
    const cf *src = in + (int64_t)bb * a.in_b + (int64_t)paired_line<C>(t, c, n) * L + j;
#pragma unroll
    for (int m = 0; m < E; ++m) x[m] = ld_data<NT>(src + T * m);
  };
  load(tile, v);
#pragma unroll
  for (int m = 0; m < E; ++m) pin_regs(v[m]);  // (see k_lines_pf)

  for (; tile < nt; tile += Gd) {
    asm volatile("" : "+v"(c), "+v"(j));
    const uint32_t bb = tile / tpb, t = tile - bb * tpb;
    const int c2 = tid % H, q0 = tid / H;
    const uint32_t k1 = t * H + (uint32_t)c2;
    const cf wl = a.wlo[k1];  // w_N^{k1}
    load(tile + Gd < nt ? tile + Gd : nt - 1, vn);
    all_passes<L, EPT, C, ELEM_FAST>(v, lds, tw, c, j, std::make_integer_sequence<int, G::NP>{});
#pragma unroll
    for (int m = 0; m < E; ++m) lds[LO::idx_off(c, j, T * m)] = v[m];
    __syncthreads();
    cf *dst = out + (int64_t)bb * a.out_b;
    const bool self = t == 0 && c2 == 0;  // rows 0 and n / 2
    const cf wh = a.wlo[n / 2];           // w_N^{n / 2}
    if (self && q0 == 0) {  // k = L / 2 pairs with itself
      const cf zm = lds[LO::idx(0, L / 2)];
      dst[a.L / 2] = make_float2(zm.x, -zm.y);
    }
#pragma unroll
    for (int m = 0; m < L / STEP; ++m) {
      const int p = q0 + STEP * m;
      int ca = c2, cb = c2 + H, pa = p, pb = L - 1 - p;
      uint32_t row = k1;
      cf w0 = wl;
      if (self) {
        // the first half of the pairs are row 0's, the second row n / 2's
        const bool mid = p >= L / 2;
        pa = mid ? p - L / 2 : p;
        pb = mid ? L - 1 - pa : (L - pa) & (L - 1);
        ca = cb = mid ? H : 0;
        row = mid ? n / 2 : 0u;
        w0 = mid ? wh : make_float2(1.0f, 0.0f);
      }
      const cf za = lds[LO::idx(ca, pa)], zb = lds[LO::idx(cb, pb)];
      cf xa, xb;
      real_pair_fwd(za, zb, cmul(whi[pa], w0), xa, xb);
      const uint32_t k = row + n * (uint32_t)pa;
      dst[k] = xa;
      dst[a.L - k] = xb;
    }
    __syncthreads();  // the next tile's passes reuse the buffer
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = vn[m];
  }
}

template <int L, int C, int EPT>
__global__ void __launch_bounds__(C * (P2<L, EPT>::T))
    k_real_cols(const cf *__restrict__ in, cf *__restrict__ out, RealFourArgs a) {
  using G = P2<L, EPT>;
  constexpr int E = G::E, T = G::T, NTH = C * T, H = C / 2;
  static_assert(NTH <= 1024, "a workgroup holds at most 1024 threads");
  using TW = PairedTw<L, C, LINE_FAST, LINE_FAST, EPT>;
  using LI = Lds<L, C, LINE_FAST, kPadShift>;
  __shared__ __align__(16) cf lds[lds_pairs<L, C, LINE_FAST, LINE_FAST>()];
  __shared__ cf twl[TW::NTW], whi[L];  // whi: w_N^{n n1}, n1 < L
  const int tid = threadIdx.x;
  TW::fill(twl, a.tw, a.tw2, tid, NTH);
  for (int i = tid; i < L; i += NTH) whi[i] = a.whi[i];
  __syncthreads();
  const typename TW::type tw = TW::make(twl);
  int c, j;
  lane_map<L, EPT, C, LINE_FAST>(tid, c, j);
  const uint32_t n = a.n, tpb = n / C, nt = a.ntiles, Gd = gridDim.x;
  uint32_t tile = paired_slot();
  if (tile >= nt) return;

  cf v[E], vn[E];
  auto load = [&](uint32_t tl, cf(&x)[E]) {
    const uint32_t bb = tl / tpb, t = tl - bb * tpb;
    const cf *src = in + (int64_t)bb * a.in_b;
    const uint32_t o = paired_line<C>(t, c, n) + (uint32_t)j * n;
#pragma unroll
    for (int m = 0; m < E; ++m) x[m] = ldg<0>(src, o + (uint32_t)(T * m) * n);
  };
  load(tile, v);
#pragma unroll
  for (int m = 0; m < E; ++m) pin_regs(v[m]);  // (see k_lines_pf)

  for (; tile < nt; tile += Gd) {
    asm volatile("" : "+v"(c), "+v"(j));
    const uint32_t bb = tile / tpb, t = tile - bb * tpb;
    const uint32_t n2 = paired_line<C>(t, c, n);
    const uint32_t msk = (1u << a.tw4_shift) - 1u;
    const uint32_t eA = n2 * (uint32_t)j, eB = n2 * (uint32_t)T;
    const cf wl = a.wlo[n2];  // w_N^{n2}
    const cf Ah = a.tw4_hi[eA >> a.tw4_shift], Al = a.tw4_lo[eA & msk];
    const cf Bh = a.tw4_hi[eB >> a.tw4_shift], Bl = a.tw4_lo[eB & msk];
    // bin L of the signal pairs with bin 0 (first tile's line 0)
    const bool self0 = t == 0 && c == 0, selfm = t == 0 && c == H;
    cf xl = make_float2(0.f, 0.f);
    if (self0 && j == 0) xl = in[(int64_t)bb * a.in_b + a.L];
    load(tile + Gd < nt ? tile + Gd : nt - 1, vn);
#pragma unroll
    for (int m = 0; m < E; ++m) lds[LI::idx_off(c, j, T * m)] = v[m];
    __syncthreads();
    const int cb = self0 || selfm ? c : c < H ? c + H : c - H;
#pragma unroll
    for (int m = 0; m < E; ++m) {
      const int p = j + T * m;
      const int pb = self0 ? (L - p) & (L - 1) : L - 1 - p;
      cf xk = v[m], xr = lds[LI::idx(cb, pb)], zk, zr;
      if (m == 0 && self0 && j == 0) {
        xk.y = 0.f;
        xr = make_float2(xl.x, 0.f);
      }
      real_pair_inv(xk, xr, cmul(whi[p], wl), zk, zr);
      v[m] = cswap(zk);
    }
    __syncthreads();  // the pairing reads are done before the passes write LDS
    all_passes<L, EPT, C, LINE_FAST>(v, lds, tw, c, j, std::make_integer_sequence<int, G::NP>{});
    tw4_apply_ab<E>(v, cmul(Ah, Al), cmul(Bh, Bl));
    cf *dst = out + (int64_t)bb * a.out_b;
    const uint32_t o = n2 + (uint32_t)j * n;
#pragma unroll
    for (int m = 0; m < E; ++m) stg<0>(dst, o + (uint32_t)(T * m) * n, v[m]);
#pragma unroll
    for (int m = 0; m < E; ++m) v[m] = vn[m];
  }
}

#define RF(L_, C_, E_)                                                                             \
  RealFourKernel{L_, C_, E_,                                                                     \
                 (const void *)&k_real_rows<L_, C_, E_, 0>, (const void *)&k_real_rows<L_, C_, E_, 1>, \
                 (const void *)&k_real_cols<L_, C_, E_>, C_ * P2<L_, E_>::T,                     \
                 8 * (lds_pairs<L_, C_, ELEM_FAST, LINE_FAST>() + L_ +                           \
                      pf_tw_entries<L_, C_, ELEM_FAST, LINE_FAST, E_>()),                        \
                 8 * (lds_pairs<L_, C_, LINE_FAST, LINE_FAST>() + L_ +                           \
                      pf_tw_entries<L_, C_, LINE_FAST, LINE_FAST, E_>())}
static const RealFourKernel kRealFour[] = {RF(512, 32, 16), RF(1024, 16, 32)};
#undef RF

bool real_four_kernel(int L, RealFourKernel *out) {
  for (const auto &e : kRealFour)
    if (e.L == L) {
      *out = e;
      return true;
    }
  return false;
}

}  // namespace dpfft
