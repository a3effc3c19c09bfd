// Device building blocks of the runtime-radix transforms, shared by the
// batched kernels and the ragged persistent kernel.
#pragma once
#include "fft_common.h"
#include "kernels.h"
#include "mixed.h"

namespace dpfft {

// Address-space-qualified element pointers: the pass functions below are not
// inlined, so their pointer arguments must carry the address space for the
// compiler to emit LDS (ds_*) and global (global_*) instructions rather than
// flat ones.
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) v2f lcf;  // LDS
typedef __attribute__((address_space(1))) v2f gcf;  // global memory

__device__ __forceinline__ lcf *as_lds(cf *p) { return (lcf *)p; }
__device__ __forceinline__ gcf *as_glb(cf *p) { return (gcf *)p; }
__device__ __forceinline__ const gcf *as_glb(const cf *p) { return (const gcf *)p; }

template <class P, class I>
__device__ __forceinline__ cf ldc(P *p, I i) {
  const v2f v = p[i];
  return make_float2(v.x, v.y);
}
template <class P, class I>
__device__ __forceinline__ void stc(P *p, I i, cf y) {
  v2f v;
  v.x = y.x;
  v.y = y.y;
  p[i] = v;
}

// a streamed store (whole lines of data that is read again only much later)
__device__ __forceinline__ void stc_nt(gcf *p, uint32_t i, cf y) {
  v2f v;
  v.x = y.x;
  v.y = y.y;
  __builtin_nontemporal_store(v, p + i);
}

namespace {

__device__ __forceinline__ int midx_elem(int pitch, int c, int pos) {
  return c * pitch + pos + (pos >> 4);
}
__device__ __forceinline__ int midx_line(int C, int c, int pos) {
  const int u = pos * C + c;
  return u + (u >> 4);
}

__device__ __forceinline__ cf tw2_lookup(const lcf *t, int shift, uint32_t e) {
  const cf lo = ldc(t, e & ((1u << shift) - 1u));
  const cf hi = ldc(t, (1u << shift) + (e >> shift));
  return cmul(hi, lo);
}

// Pass twiddles w_L^{e1 r}, r = 1..R-1, into x[1..R-1] (multiplied in).  All are
// looked up: products of a few of them halve the table reads and save time (16 M
// points: 10000 points 7%, 5000 6%, 4000 5%, 2000 4%, 1080 x 1920 images 1%, others
// 0 to 4%) but cost accuracy (5000 = 25 x 20 x 10 points 8%, 3136 = 16 x 14 x 14 8%, 2000
// 4%).
template <int R>
__device__ __forceinline__ void apply_pass_twiddles(cf *x, const lcf *t, int shift, uint32_t e1) {
#pragma unroll
  for (int r = 1; r < R; ++r) x[r] = cmul(x[r], tw2_lookup(t, shift, e1 * (uint32_t)r));
}

// Four-step twiddles w_N^{line (b + r NS)} = A B^r of outputs r = 0..R-1 of
// butterfly b = j + T q: A B^l for l < 4 from A and B, times B^{4 g}, with
// B^4, B^8 and B^16 taken from the two-level table of w_N as well (the error
// of B would grow with the power), so at most three products follow a lookup.
// All but A depend on the line alone: kFourStepVals values per line, looked up
// once per tile by its first threads and kept in LDS, where every lane of the
// line reads the same word.  As per-lane gathers (a dozen cache lines each)
// they cost more than the tile's data loads: 46080 = 192 x 240, 72 M points,
// the column launch 275 us with gathers after the butterflies, 259 with
// gathers issued early, 230 so.
// The values of `C` lines from line0 on at tab[v * C + c]: w_N^{line m}, m =
// ns, 4 ns, 8 ns, 16 ns and T, as far as a line of L outputs needs them (m < L
// keeps line * m below N).
__device__ __forceinline__ void four_step_fill(lcf *tab, const gcf *lo, const gcf *hi, int shift,
                                               int C, uint32_t line0, uint32_t lines, uint32_t L,
                                               uint32_t ns, uint32_t T, int tid, int nth) {
  for (int t = tid; t < kFourStepVals * C; t += nth) {
    const int v = t / C;
    const uint32_t line = line0 + (uint32_t)(t - v * C);
    const uint32_t m = v == 0 ? ns : v == 1 ? 4 * ns : v == 2 ? 8 * ns : v == 3 ? 16 * ns : T;
    if (m >= L || line >= lines) continue;
    const uint32_t e = line * m;
    stc(tab, t, cmul(ldc(hi, e >> shift), ldc(lo, e & ((1u << shift) - 1u))));
  }
}

template <int R, int Q>
struct FourStepTw {
  cf ah[(Q + 1) / 2], al[(Q + 1) / 2];  // table entries of A for even q
  __device__ __forceinline__ void load(const gcf *lo, const gcf *hi, int shift, uint32_t line,
                                       uint32_t j, uint32_t T, uint32_t M) {
#pragma unroll
    for (int q = 0; q < Q; q += 2) {
      const uint32_t b = j + T * (uint32_t)q;
      const uint32_t e = line * (b < M ? b : 0u);
      ah[q / 2] = ldc(hi, e >> shift);
      al[q / 2] = ldc(lo, e & ((1u << shift) - 1u));
    }
  }
  // multiply butterfly q's outputs; tab points at the line's first value
  __device__ __forceinline__ void apply(cf *x, int q, const lcf *tab, int C) const {
    cf a = cmul(ah[q / 2], al[q / 2]);
    if (q & 1) a = cmul(a, ldc(tab, 4 * C));
    cf Al[4] = {a, a, a, a};
    if constexpr (R > 1) {
      const cf b = ldc(tab, 0);
      Al[1] = cmul(a, b);
      if constexpr (R > 2) {
        const cf b2 = cmul(b, b);
        Al[2] = cmul(a, b2);
        if constexpr (R > 3) Al[3] = cmul(a, cmul(b2, b));
      }
    }
    cf p4 = a, p8 = a, p16 = a;
    if constexpr (R > 4) p4 = ldc(tab, C);
    if constexpr (R > 8) p8 = ldc(tab, 2 * C);
    if constexpr (R > 16) p16 = ldc(tab, 3 * C);
#pragma unroll
    for (int l = 0; l < 4 && l < R; ++l) x[l] = cmul(x[l], Al[l]);
#pragma unroll
    for (int g = 1; 4 * g < R; ++g) {
      cf w = g & 1 ? p4 : g & 2 ? p8 : p16;
      if ((g & 1) && (g & 2)) w = cmul(w, p8);
      if ((g & 3) && (g & 4)) w = cmul(w, p16);
#pragma unroll
      for (int l = 0; l < 4; ++l)
        if (4 * g + l < R) x[4 * g + l] = cmul(x[4 * g + l], cmul(Al[l], w));
    }
  }
};

}  // namespace

// One pass.  It is a separate (non-inlined) function per radix so that each
// radix gets its own register allocation; its context travels as plain
// scalars and address-space-qualified pointers.  `tw2` is the two-level
// table of w_L held in LDS.  `sw` is the launch's swap mode.
// The first pass also copies the first `ntw` entries of the global table tw2g
// into tw2 (one per thread): their loads are issued before the tile's data
// loads and their LDS stores after them, so the copy adds no round trip of its
// own (the pass's closing barrier publishes the table to the later passes).
template <int MAP, int OMAP, int TW4, int R>
__device__ __noinline__ void mixed_pass(const gcf *__restrict__ src, gcf *__restrict__ dst,
                                        lcf *lds, lcf *tw2, const gcf *__restrict__ tw2g, int ntw,
                                        const gcf *__restrict__ tw4_lo,
                                        const gcf *__restrict__ tw4_hi, lcf *tw4_tab, int L,
                                        int T, int C, int pitch, int NS, int tw2_shift, int tw4_shift, int c,
                                        int j, bool valid, bool first, bool last, int sw,
                                        int64_t in_e, int64_t out_e, int64_t line, float scale) {
  // The shape arguments arrive in VGPRs (this is a call); they are the same in
  // every lane, so move them to SGPRs: the divisions and branches on them then
  // run once per wave on the scalar unit instead of on the VALU.
  L = __builtin_amdgcn_readfirstlane(L);
  T = __builtin_amdgcn_readfirstlane(T);
  C = __builtin_amdgcn_readfirstlane(C);
  pitch = __builtin_amdgcn_readfirstlane(pitch);
  NS = __builtin_amdgcn_readfirstlane(NS);
  tw2_shift = __builtin_amdgcn_readfirstlane(tw2_shift);
  tw4_shift = __builtin_amdgcn_readfirstlane(tw4_shift);
  first = __builtin_amdgcn_readfirstlane((int)first) != 0;
  last = __builtin_amdgcn_readfirstlane((int)last) != 0;
  sw = __builtin_amdgcn_readfirstlane(sw);
  // element strides and in-line offsets fit 32 bits (checked by the planner:
  // (L - 1) * stride < 2^31), so the per-element index math stays 32-bit
  const uint32_t ie = (uint32_t)__builtin_amdgcn_readfirstlane((int)in_e);
  const uint32_t oe = (uint32_t)__builtin_amdgcn_readfirstlane((int)out_e);
  scale = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(scale)));
  const int M = L / R;
  constexpr int QM = mixed_qmax(R);  // butterflies per thread
  auto li = [&](int m, int pos) {
    return m == ELEM_FAST ? midx_elem(pitch, c, pos) : midx_line(C, c, pos);
  };
  cf v[QM][R];
  bool act[QM];
  int kq[QM];
  // all loads of the pass first (one branch on the source for the whole
  // pass), so every butterfly's data is in flight before the first one is
  // computed
  // k = b mod NS for b = j + T q: one division per pass, then a step of
  // T mod NS (a scalar) and a conditional subtraction per butterfly
  {
    const int k0 = NS > 1 ? j % NS : 0;
    const int tstep = NS > 1 ? T % NS : 0;
    int k = k0;
#pragma unroll
    for (int q = 0; q < QM; ++q) {
      const int b = j + T * q;
      act[q] = valid && b < M;
      kq[q] = k;
      k += tstep;
      if (k >= NS) k -= NS;
    }
  }
  FourStepTw<R, QM> f4;
  if (TW4 && last)
    f4.load(tw4_lo, tw4_hi, tw4_shift, valid ? (uint32_t)line : 0u, (uint32_t)j, (uint32_t)T,
            (uint32_t)M);
  if (first) {
    ntw = __builtin_amdgcn_readfirstlane(ntw);
    const int tid = (int)threadIdx.x;
    cf tv = make_float2(0.0f, 0.0f);
    if (tid < ntw) tv = ldc(tw2g, tid);
#pragma unroll
    for (int q = 0; q < QM; ++q) {
      if (!act[q]) continue;
#pragma unroll
      for (int r = 0; r < R; ++r) v[q][r] = ldc(src, (uint32_t)(j + T * q + r * M) * ie);
    }
    if (tid < ntw) stc(tw2, tid, tv);
  } else {
#pragma unroll
    for (int q = 0; q < QM; ++q) {
      if (!act[q]) continue;
#pragma unroll
      for (int r = 0; r < R; ++r) v[q][r] = ldc(lds, li(MAP, j + T * q + r * M));
    }
  }
#pragma unroll
  for (int q = 0; q < QM; ++q) {
    if (!act[q]) continue;
    if ((sw & 1) && first) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[q][r] = cswap(v[q][r]);
    }
    if (NS > 1) {
      const uint32_t step = (uint32_t)(L / (NS * R));
      apply_pass_twiddles<R>(v[q], tw2, tw2_shift, (uint32_t)kq[q] * step);
    }
    Dft<R>::run(v[q]);
    if (TW4 && last) {
      f4.apply(v[q], q, tw4_tab + c, C);  // the last pass's outputs are k1 = b + r*NS
    }
    if ((sw & 2) && last) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[q][r] = cswap(cscale(v[q][r], scale));
    }
  }
  if (!first) __syncthreads();  // every read of this pass precedes the in-place writes
#pragma unroll
  for (int q = 0; q < QM; ++q) {
    if (!act[q]) continue;
    const int b = j + T * q;
    const int k = kq[q];
    const int base = (b - k) * R + k;
    if (TW4 == TW4_STREAM && last) {
      // the four-step intermediate, streamed: it leaves the L2 to the lines the
      // tile's neighbours read (the four-step signals of the ragged batch: 583
      // us plain, 554 streamed)
#pragma unroll
      for (int r = 0; r < R; ++r) stc_nt(dst, (uint32_t)(base + r * NS) * oe, v[q][r]);
    } else if (last && OMAP == MAP) {
#pragma unroll
      for (int r = 0; r < R; ++r) stc(dst, (uint32_t)(base + r * NS) * oe, v[q][r]);
    } else if (last) {
#pragma unroll
      for (int r = 0; r < R; ++r) stc(lds, li(OMAP, base + r * NS), v[q][r]);
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r) stc(lds, li(MAP, base + r * NS), v[q][r]);
    }
  }
  if (!last || OMAP != MAP) __syncthreads();
}

// The pass of run-time radix R.
template <int MAP, int OMAP, int TW4, class... A>
__device__ __forceinline__ void mixed_pass_any(int R, A... args) {
#define PASS(RR) \
  case RR:       \
    mixed_pass<MAP, OMAP, TW4, RR>(args...); \
    break
  switch (R) {
    PASS(2);
    PASS(3);
    PASS(4);
    PASS(5);
    PASS(6);
    PASS(7);
    PASS(8);
    PASS(9);
    PASS(10);
    PASS(12);
    PASS(14);
    PASS(15);
    PASS(16);
    PASS(18);
    PASS(20);
    PASS(21);
    PASS(24);
    PASS(25);
  }
#undef PASS
}

// One tile (up to C lines of length L) through every pass.  Thread (c, j)
// works on line c; src/dst are its line's base pointers.  With OMAP != MAP the
// last pass leaves the tile in LDS and thread (c2, j2) stores line c2 through
// dst2, coalesced in the output layout.
struct TileLine {
  const cf *src;
  cf *dst;
  int64_t in_e, out_e, line, line0;  // line0: the tile's first line
  int c, j;
  bool valid;
  cf *dst2;      // staged store: output base of line c2
  int c2, j2;
  bool valid2;
};

struct LineShape {
  int L, T, C, pitch, P, tw2_shift;
  uint64_t codes;
  const cf *tw2;  // two-level table of w_L in global memory (copied to LDS per tile)
  const cf *tw4_lo, *tw4_hi;
  int tw4_shift;
  float scale;
  int tw_lds;     // LDS element offset of the copied table (after the tile data)
  int64_t lines;  // four-step: lines of the matrix
};

// entries of the two-level table of w_L: 2^s lo entries and ceil(L / 2^s) hi
__host__ __device__ inline int tw2_entries(int L, int shift) {
  return (1 << shift) + (L + (1 << shift) - 1) / (1 << shift);
}

template <int MAP, int OMAP, int TW4, int SW>
__device__ __forceinline__ void mixed_tile(const LineShape &sh, const TileLine &t, cf *lds,
                                           int nthreads) {
  if (sh.P == 0) {  // length 1: the transform is the identity, up to the swaps and the scale
    if (t.valid && t.j == 0) {
      cf y = t.src[0];
      if (SW & 1) y = cswap(y);
      if (SW & 2) y = cswap(cscale(y, sh.scale));
      t.dst[0] = y;
    }
    return;
  }
  // pass twiddles to LDS: the first pass copies one entry per thread (see
  // mixed_pass), entries past the first nthreads are copied here; the barrier
  // that ends the first pass publishes them before the second pass reads any
  lcf *twl = as_lds(lds) + sh.tw_lds;
  const int ntw = tw2_entries(sh.L, sh.tw2_shift);
  for (int i = threadIdx.x + nthreads; i < ntw; i += nthreads) stc(twl, i, sh.tw2[i]);
  const int ntw0 = ntw < nthreads ? ntw : nthreads;
  if constexpr (TW4) {
    // published by the barrier that ends the first pass (a one-pass line has
    // none, and its own)
    const int RL = (int)((sh.codes >> (5 * (sh.P - 1))) & 31u);
    four_step_fill(twl + ntw, as_glb(sh.tw4_lo), as_glb(sh.tw4_hi), sh.tw4_shift, sh.C,
                   (uint32_t)t.line0, (uint32_t)sh.lines, (uint32_t)sh.L, (uint32_t)(sh.L / RL),
                   (uint32_t)sh.T, (int)threadIdx.x, nthreads);
    if (sh.P == 1) __syncthreads();
  }
  int ns = 1;
  for (int p = 0; p < sh.P; ++p) {
    const bool first = p == 0, last = p == sh.P - 1;
    const int R = (int)((sh.codes >> (5 * p)) & 31u);
    mixed_pass_any<MAP, OMAP, TW4>(R, as_glb(t.src), as_glb(t.dst), as_lds(lds), twl,
                                   as_glb(sh.tw2), ntw0, as_glb(sh.tw4_lo), as_glb(sh.tw4_hi),
                                   twl + ntw, sh.L, sh.T, sh.C, sh.pitch, ns, sh.tw2_shift, sh.tw4_shift, t.c,
                                   t.j, t.valid, first, last, SW, t.in_e, t.out_e, t.line,
                                   sh.scale);
    ns *= R;
  }
  if (OMAP != MAP && t.valid2) {
    for (int i = t.j2; i < sh.L; i += sh.T)
      t.dst2[(int64_t)i * t.out_e] =
          lds[OMAP == ELEM_FAST ? midx_elem(sh.pitch, t.c2, i) : midx_line(sh.C, t.c2, i)];
  }
}

}  // namespace dpfft
