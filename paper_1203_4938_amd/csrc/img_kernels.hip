// Image block compression (section III-B of the paper), five steps:
//   (a) RGB -> luminance Y and chroma Cb, Cr (full-range BT.601 as in JFIF)
//   (b) chroma at a quarter of the pixels (means of 2x2 squares)
//   (c) |grad Y| (central differences, edges replicated) and per 4x4 block
//       its mean (activity), the mean luminance and the 16 deviations
//   (d) k-means codebook of the deviation vectors of blocks with activity
//       >= tau (Lloyd's iteration from the pattern blocks of rank
//       floor(c P / k))
//   (e) per block: code 0 (mean only) or 1 + the nearest codeword.
// The paper runs (a)-(c) and (e) as data-parallel programs and (d) on the
// host; here every step is a kernel, so a batch of images is one sequence of
// launches on one stream with no host round trip.
//
// (a)-(c) are one pass over the pixels (k_img_front): a 64 x 16 pixel tile
// computes Y for itself and a one-pixel halo into LDS, writes Y and the
// quarter-size chroma, then four threads per block reduce its 16 pixels.
// The k-means and the encoding walk the blocks in groups of 1024, one block
// per thread and round, the codebook in LDS; the cluster sums of a group are
// added in block order into per-group partials that k_img_update adds up in a
// fixed order.
#include "fft_common.h"
#include "img.h"

namespace dpfft {

namespace {

__device__ __forceinline__ float luma(float r, float g, float b) {
  return 0.299f * r + 0.587f * g + 0.114f * b;
}
__device__ __forceinline__ float chroma_b(float r, float g, float b) {
  return 128.0f - 0.168736f * r - 0.331264f * g + 0.5f * b;
}
__device__ __forceinline__ float chroma_r(float r, float g, float b) {
  return 128.0f + 0.5f * r - 0.418688f * g - 0.081312f * b;
}

constexpr int HW = kImgTileW + 2, HH = kImgTileH + 2;  // tile with its halo

}  // namespace

// Y of pixel (gy, gx) clamped to the image (the replicated edge).
__device__ __forceinline__ float luma_at(const uint8_t *rgb, int64_t h, int64_t w, int64_t gy,
                                         int64_t gx) {
  gy = gy < 0 ? 0 : (gy >= h ? h - 1 : gy);
  gx = gx < 0 ? 0 : (gx >= w ? w - 1 : gx);
  const uint8_t *p = rgb + (gy * w + gx) * 3;
  return luma((float)p[0], (float)p[1], (float)p[2]);
}

// Thread (row ry, group g) of a tile owns the 4 pixels x0 + 4 g .. + 3 of row
// y0 + ry: their 12 bytes are three aligned 32-bit words (the width is a
// multiple of 4).  It writes their Y, keeps it in LDS with the tile's
// one-pixel halo, and leaves the Cb, Cr sums of its two horizontal pixel
// pairs in LDS for the 2 x 2 means.  Then four threads take each 4 x 4 block,
// one block row each, and add their row sums with lane shuffles.
__global__ void __launch_bounds__(kImgThreads) k_img_front(ImgArgs a) {
  static_assert(kImgTileW == 64 && kImgTileH == 16 && kImgThreads == 256, "tile shape");
  __shared__ float ys[HH * HW];
  __shared__ float2 cpart[kImgTileH][kImgTileW / 2];
  const int64_t img = blockIdx.y;
  const int64_t tiles_x = (a.w + kImgTileW - 1) / kImgTileW;
  const int64_t tx = blockIdx.x % tiles_x, ty = blockIdx.x / tiles_x;
  const int64_t x0 = tx * kImgTileW, y0 = ty * kImgTileH;
  const uint8_t *rgb = a.rgb + img * a.h * a.w * 3;
  float *Y = a.y + img * a.h * a.w;
  const int tid = threadIdx.x;

  // (a) luminance of the tile, (b) chroma sums of horizontal pairs
  {
    const int ry = tid / 16, g = tid % 16;
    const int64_t py = y0 + ry, px = x0 + 4 * g;
    float yv[4];
    if (py < a.h && px < a.w) {
      const uint32_t *p = reinterpret_cast<const uint32_t *>(rgb + (py * a.w + px) * 3);
      const uint32_t d0 = p[0], d1 = p[1], d2 = p[2];
      const float r[4] = {(float)(d0 & 255u), (float)(d0 >> 24), (float)((d1 >> 16) & 255u),
                          (float)((d2 >> 8) & 255u)};
      const float gg[4] = {(float)((d0 >> 8) & 255u), (float)(d1 & 255u), (float)(d1 >> 24),
                           (float)((d2 >> 16) & 255u)};
      const float bb[4] = {(float)((d0 >> 16) & 255u), (float)((d1 >> 8) & 255u), (float)(d2 & 255u),
                           (float)(d2 >> 24)};
      float cb[4], cr[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        yv[i] = luma(r[i], gg[i], bb[i]);
        cb[i] = chroma_b(r[i], gg[i], bb[i]);
        cr[i] = chroma_r(r[i], gg[i], bb[i]);
      }
      *reinterpret_cast<float4 *>(Y + py * a.w + px) = make_float4(yv[0], yv[1], yv[2], yv[3]);
      cpart[ry][2 * g] = make_float2(cb[0] + cb[1], cr[0] + cr[1]);
      cpart[ry][2 * g + 1] = make_float2(cb[2] + cb[3], cr[2] + cr[3]);
    } else {
      // past the image's last row or column: the replicated edge, for the
      // central differences of the blocks along it
#pragma unroll
      for (int i = 0; i < 4; ++i) yv[i] = luma_at(rgb, a.h, a.w, py, px + i);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) ys[(ry + 1) * HW + 4 * g + 1 + i] = yv[i];
  }
  // the halo: rows -1 and 16 of the tile, columns -1 and 64 (corners unused)
  if (tid < 2 * kImgTileW + 2 * kImgTileH) {
    int ly, lx;
    if (tid < 2 * kImgTileW) {
      ly = tid < kImgTileW ? 0 : HH - 1;
      lx = tid % kImgTileW + 1;
    } else {
      const int q = tid - 2 * kImgTileW;
      ly = q % kImgTileH + 1;
      lx = q < kImgTileH ? 0 : HW - 1;
    }
    ys[ly * HW + lx] = luma_at(rgb, a.h, a.w, y0 + ly - 1, x0 + lx - 1);
  }
  __syncthreads();
  // (b) chroma: means of 2 x 2 squares, two per thread of the first 128
  if (tid < kImgTileH / 2 * kImgTileW / 4) {
    const int rp = tid / 16, g = tid % 16;
    const int64_t py = y0 + 2 * rp, px = x0 + 4 * g;
    if (py < a.h && px < a.w) {
      const float2 u0 = cpart[2 * rp][2 * g], l0 = cpart[2 * rp + 1][2 * g];
      const float2 u1 = cpart[2 * rp][2 * g + 1], l1 = cpart[2 * rp + 1][2 * g + 1];
      const int64_t w2 = a.w / 2, o = img * (a.h / 2) * w2 + (py / 2) * w2 + px / 2;
      *reinterpret_cast<float2 *>(a.cb + o) = make_float2(0.25f * (u0.x + l0.x), 0.25f * (u1.x + l1.x));
      *reinterpret_cast<float2 *>(a.cr + o) = make_float2(0.25f * (u0.y + l0.y), 0.25f * (u1.y + l1.y));
    }
  }
  // (c) blocks: four threads per block (lanes 4 q .. 4 q + 3 of one wave)
  {
    const int blk = tid / 4, r = tid % 4;
    const int by = blk / (kImgTileW / 4), bx = blk % (kImgTileW / 4);
    const int ly = 4 * by + r + 1, lx0 = 4 * bx + 1;
    float v[4], s = 0.f, g = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int lx = lx0 + j;
      const float c = ys[ly * HW + lx];
      const float gx = 0.5f * (ys[ly * HW + lx + 1] - ys[ly * HW + lx - 1]);
      const float gyv = 0.5f * (ys[(ly + 1) * HW + lx] - ys[(ly - 1) * HW + lx]);
      g += __builtin_sqrtf(gx * gx + gyv * gyv);
      s += c;
      v[j] = c;
    }
    s += __shfl_xor(s, 1, 64);
    g += __shfl_xor(g, 1, 64);
    s += __shfl_xor(s, 2, 64);
    g += __shfl_xor(g, 2, 64);
    const int64_t gby = y0 / 4 + by, gbx = x0 / 4 + bx, bw = a.w / 4;
    if (gby < a.h / 4 && gbx < bw) {
      const float m = s * (1.0f / 16.0f);
      const int64_t b = img * a.nb + gby * bw + gbx;
      if (r == 0) {
        a.mean[b] = m;
        a.act[b] = g * (1.0f / 16.0f);
      }
      reinterpret_cast<float4 *>(a.dev + 16 * b)[r] = make_float4(v[0] - m, v[1] - m, v[2] - m, v[3] - m);
    }
  }
}

// (d) pattern blocks per group of 256 blocks
__global__ void __launch_bounds__(kImgBlocksPerGroup) k_img_count(ImgArgs a) {
  __shared__ int cnt[kImgBlocksPerGroup / 64];
  const int64_t img = blockIdx.y;
  const int64_t b = (int64_t)blockIdx.x * kImgBlocksPerGroup + threadIdx.x;
  const bool pat = b < a.nb && a.act[img * a.nb + b] >= a.tau;
  const uint64_t m = __ballot(pat);
  if (threadIdx.x % 64 == 0) cnt[threadIdx.x / 64] = __popcll(m);
  __syncthreads();
  if (threadIdx.x == 0) {
    int n = 0;
    for (int w = 0; w < kImgBlocksPerGroup / 64; ++w) n += cnt[w];
    a.wgcount[img * a.groups + blockIdx.x] = n;
  }
}

// Exclusive offsets of the groups' pattern blocks (one workgroup per image,
// sequential over chunks of 256 groups), the pattern count, and a zero
// codebook (codewords with no seed stay zero when no block is a pattern).
__global__ void __launch_bounds__(256) k_img_scan(ImgArgs a) {
  __shared__ int s[256];
  __shared__ int carry;
  const int64_t img = blockIdx.x;
  int32_t *wc = a.wgcount + img * a.groups;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int base = 0; base < a.groups; base += 256) {
    const int i = base + threadIdx.x;
    const int v = i < a.groups ? wc[i] : 0;
    s[threadIdx.x] = v;
    __syncthreads();
    for (int d = 1; d < 256; d *= 2) {  // inclusive scan (Hillis-Steele)
      const int t = threadIdx.x >= d ? s[threadIdx.x - d] : 0;
      __syncthreads();
      s[threadIdx.x] += t;
      __syncthreads();
    }
    if (i < a.groups) wc[i] = carry + s[threadIdx.x] - v;
    __syncthreads();
    if (threadIdx.x == 255) carry += s[255];
    __syncthreads();
  }
  if (threadIdx.x == 0) a.npat[img] = carry;
  for (int i = threadIdx.x; i < a.k * 16; i += 256) a.codebook[img * a.k * 16 + i] = 0.f;
}

// Seeds: codeword c takes the deviation vector of the pattern block of rank
// floor(c P / k); a block of rank r seeds every c with that floor.
__global__ void __launch_bounds__(kImgBlocksPerGroup) k_img_seed(ImgArgs a) {
  __shared__ int cnt[kImgBlocksPerGroup / 64];
  const int64_t img = blockIdx.y;
  const int64_t b = (int64_t)blockIdx.x * kImgBlocksPerGroup + threadIdx.x;
  const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
  const bool pat = b < a.nb && a.act[img * a.nb + b] >= a.tau;
  const uint64_t m = __ballot(pat);
  if (lane == 0) cnt[wave] = __popcll(m);
  __syncthreads();
  if (!pat) return;
  int64_t rank = a.wgcount[img * a.groups + blockIdx.x] + __popcll(m & ((1ull << lane) - 1ull));
  for (int w = 0; w < wave; ++w) rank += cnt[w];
  const int64_t P = a.npat[img];
  const int64_t k = a.k;
  const int64_t c_lo = (rank * k + P - 1) / P, c_hi = ((rank + 1) * k + P - 1) / P;
  const float *src = a.dev + 16 * (img * a.nb + b);
  for (int64_t c = c_lo; c < c_hi && c < k; ++c)
    for (int t = 0; t < 16; ++t) a.codebook[(img * k + c) * 16 + t] = src[t];
}

// Nearest codeword of every pattern block (ties to the lower index).
// The squared distance |v - c|^2 = |v|^2 - 2 (v.c - |c|^2 / 2) is ranked by
// D_c = v.c - h_c with h_c = |c|^2 / 2, the same maximiser as the smallest
// distance in exact arithmetic.
//
// The decision is the one of the FP32 products (exact_codes below:
// v_mfma_f32_16x16x4_f32, 16 codewords x 16 blocks x 4 components each, the
// accumulator started at -h_c, the best kept in index order), but those
// products run on the vector ALU's own pipes: they cost their full time on top
// of the ranking's vector instructions (measured: 16 products 0.87 us, the
// vector instructions 0.34, both 1.31).  So a wave first ranks its 64 blocks
// by BF16 products (v_mfma_f32_32x32x16_bf16, three per tile, a fifth of the
// FP32 products' cycles and mostly beside vector instructions), v and c
// split into hi + lo pieces, and keeps best and
// second best; where the two are further apart than both roundings together
// can move them the FP32 decision is the same, and the groups of 16 blocks
// with a pattern block that is not decided by that margin take the FP32
// products (0.4 to 0.9% of the groups of smooth pictures with noise, k = 16 to
// 256; whole waves of 64, 2 to 3.5% of them: 1296 us for the 1149 of 16 images
// of 2048^2).  The codes are those of the FP32 products bit for bit.
//
// The margin.  BF16 holds 8 significant bits, so |x - hi| and |lo| are at most
// 2^-8 |x|, and lo, rounded to 8 bits itself, leaves |x - hi - lo| <= 2^-17 |x|.
// The products lo c_lo are left out.  Of |v| |c|, which bounds the sum of the
// products' magnitudes, a D so loses up to 2^-16 with lo c_lo and 2^-17 with
// each of the two remainders, 512 u in all (u = 2^-24).  With S = |v| max|c| +
// max|c|^2 / 2 >= |D|, the 51 FP32 sums of the BF16 chain and the 17 of the FP32
// products count 2 u S each, as if they truncated, and the 5 low bits of D that
// hold the codeword's row while ranking 62 u S: 198 u S.  Both D of a decision
// may move by this much.  Values that overflow the pieces fail the comparison
// and take the FP32 products too.
//
// Operand layouts.  32x32x16: lane l supplies A row (l & 31) and B column (l &
// 31) at k = 8 (l >> 5) .. + 7 and holds D column (l & 31), rows 8 (r / 4) + 4 (l
// >> 5) + r % 4, r < 16.  16x16x4: A row and B column (l & 15) at k = l >> 4, D
// column (l & 15), rows 4 (l >> 4) + r, r < 4; step s of the four takes
// component 4 (l >> 4) + s.
//
// A workgroup covers kImgAssignBlocks blocks in rounds of 256 (one per
// thread), the next round's vectors in flight while this one's are ranked; the
// codebook's pieces (padded to whole groups of 32 with codewords that never
// win) and -h_c are staged in LDS once.
// NI > 0: the group's cluster sums (k <= 16 NI).  In each round every pattern
// block takes a rank among its wave's blocks of the same code from the wave's
// own LDS counter (one atomic per block; no other wave touches it, so the
// ranks do not depend on how the waves are scheduled), one wave scans the
// per-wave counts, and the block's number goes to its place in (code, wave,
// rank) order; its vector lies in LDS in block order.  The 16 lanes of group g
// add the vectors of codewords g, g + 16, ... in that order, one component
// each, and keep the running sums of the rounds in registers.  One partial per
// 1024 blocks.
// NI = 0: the codes of every block are written.
// 16 images of 2048^2, k = 64: FP32 products alone, the vectors scattered into
// order and read once more, every (codeword, component) sum a loop of its
// own: 171 us with sums, 125 the codes; 112 and 70 now (50 us is their bytes'
// time: what is left is vector instructions, half of them the ranking's, and
// the four barriers of a round).
typedef float img_f4 __attribute__((ext_vector_type(4)));
typedef float img_f16 __attribute__((ext_vector_type(16)));
typedef __bf16 img_b8 __attribute__((ext_vector_type(8)));

// LDS words of the assignment: pieces of the padded codebook, -h_c, max h_c;
// with sums also the round's vectors and a zero one, the per-wave counts,
// per-wave offsets, the run offsets and the block order (two bytes each, runs
// padded to 4).
struct AssignLds {
  int k4, hneg, hmax, blk, wcnt, woff, off, idx, nidx, total;
  __host__ __device__ AssignLds(int k, bool sums) {
    const int kp = (k + 31) & ~31;
    k4 = (k + 3) & ~3;
    nidx = (kImgThreads + 3 * (k < kImgThreads ? k : kImgThreads) + 3) & ~3;
    hneg = kp * 16;
    hmax = hneg + kp;
    blk = hmax + 4;
    wcnt = blk + (sums ? 16 * (kImgThreads + 1) : 0);
    woff = wcnt + (sums ? 4 * k4 : 0);
    off = woff + (sums ? 4 * k4 : 0);
    idx = off + (sums ? k4 + 4 : 0);
    total = idx + (sums ? nidx / 2 : 0);
  }
};

constexpr float kImgNever = -3.4e38f;  // below every codeword's D

// hi and lo BF16 pieces of eight components
__device__ __forceinline__ void bf16_pieces(float4 p, float4 q, img_b8 &hi, img_b8 &lo) {
  const float x[8] = {p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w};
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    hi[i] = (__bf16)x[i];
    lo[i] = (__bf16)(x[i] - (float)hi[i]);
  }
}
__device__ __forceinline__ float max3f(float a, float b, float c) {
  float d;
  asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
__device__ __forceinline__ float med3f(float a, float b, float c) {
  float d;
  asm("v_med3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
__device__ __forceinline__ float max2f(float a, float b) {
  float d;
  asm("v_max_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}
__device__ __forceinline__ float min2f(float a, float b) {
  float d;
  asm("v_min_f32 %0, %1, %2" : "=v"(d) : "v"(a), "v"(b));
  return d;
}

// Best codeword of the lane's own block (16 g4 + col of the wave's 64, whose
// first is `dev`, `nblk` of them in the image) by the FP32 products, 16 blocks
// at a time: few registers, as it runs seldom.  Only for the groups of 16 with
// a block marked in `which` (uniform over the wave); 0 for the others.
__device__ __forceinline__ int exact_codes(const float *gcb, const float *hneg, int k, int kp,
                                           const float *dev, int64_t nblk, uint64_t which) {
  const int lane = threadIdx.x & 63, col = lane & 15, g4 = lane >> 4;
  int best = 0;
#pragma unroll 1
  for (int nt = 0; nt < 4; ++nt) {
    if (!((which >> (16 * nt)) & 0xffffu)) continue;
    const float4 v = 16 * nt + col < nblk
                         ? reinterpret_cast<const float4 *>(dev)[4 * (16 * nt + col) + g4]
                         : make_float4(0.f, 0.f, 0.f, 0.f);
    float bv = kImgNever;
    int bi = 0;
#pragma unroll 1
    for (int m0 = 0; m0 < kp; m0 += 16) {
      float4 va = make_float4(0.f, 0.f, 0.f, 0.f);
      if (m0 + col < k) {
        const float *c = gcb + 16 * (m0 + col) + 4 * g4;
        va = make_float4(c[0], c[1], c[2], c[3]);
      }
      img_f4 d = *reinterpret_cast<const img_f4 *>(hneg + m0 + 4 * g4);
      d = __builtin_amdgcn_mfma_f32_16x16x4f32(va.x, v.x, d, 0, 0, 0);
      d = __builtin_amdgcn_mfma_f32_16x16x4f32(va.y, v.y, d, 0, 0, 0);
      d = __builtin_amdgcn_mfma_f32_16x16x4f32(va.z, v.z, d, 0, 0, 0);
      d = __builtin_amdgcn_mfma_f32_16x16x4f32(va.w, v.w, d, 0, 0, 0);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const bool more = d[r] > bv;
        bv = more ? d[r] : bv;
        bi = more ? m0 + 4 * g4 + r : bi;
      }
    }
    // the four lanes of a column (g4 = 0..3) hold interleaved rows: combine
#pragma unroll
    for (int x = 16; x <= 32; x *= 2) {
      const float ov = __shfl_xor(bv, x, 64);
      const int oi = __shfl_xor(bi, x, 64);
      const bool take = ov > bv || (ov == bv && oi < bi);
      bv = take ? ov : bv;
      bi = take ? oi : bi;
    }
    best = nt == g4 ? bi : best;
  }
  return best;
}

template <int NI>
__global__ void __launch_bounds__(kImgThreads, NI > 8 ? 3 : 4)
    k_img_assign(ImgArgs a) {
  static_assert(kImgThreads == 256 && kImgAssignBlocks % kImgThreads == 0,
                "four waves of blocks, whole rounds");
  constexpr bool ACC = NI > 0;
  extern __shared__ __align__(16) float img_lds[];
  const int k = a.k, kp = (k + 31) & ~31;
  const AssignLds ly(k, ACC);
  img_b8 *cpc = reinterpret_cast<img_b8 *>(img_lds);  // [codeword][component half][hi, lo]
  float *hneg = img_lds + ly.hneg, *hmax = img_lds + ly.hmax, *blk = img_lds + ly.blk;
  int *wcnt = (int *)(img_lds + ly.wcnt), *woff = (int *)(img_lds + ly.woff);
  int *off = (int *)(img_lds + ly.off);
  uint16_t *idx = (uint16_t *)(img_lds + ly.idx);
  const uint32_t grp = a.back ? gridDim.x - 1 - blockIdx.x : blockIdx.x;
  const int64_t img = a.back ? gridDim.y - 1 - blockIdx.y : blockIdx.y;
  const int tid = threadIdx.x;
  const float *gcb = a.codebook + img * (int64_t)k * 16;
  const int64_t base = (int64_t)grp * kImgAssignBlocks;

  // a round's vectors: block 32 nt + col of the wave's 64, components 8 hl ..
  // 8 hl + 7 (col = lane & 31, hl = lane >> 5); and the activity of the lane's
  // own block
  float4 vb[2][2];
  float act = 0.f;
  auto load = [&](int64_t r0, int id) {
    const int wave = __builtin_amdgcn_readfirstlane(id >> 6), lane = id & 63;
    const int col = lane & 31, hl = lane >> 5;
    const int64_t b0 = r0 + 64 * wave;
    const float4 *src = reinterpret_cast<const float4 *>(a.dev + 16 * (img * a.nb + b0));
    if (r0 + kImgThreads <= a.nb) {  // uniform over the workgroup
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int e = 0; e < 2; ++e) vb[nt][e] = src[4 * (32 * nt + col) + 2 * hl + e];
      act = a.act[img * a.nb + b0 + lane];
    } else {
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int e = 0; e < 2; ++e)
          vb[nt][e] = b0 + 32 * nt + col < a.nb ? src[4 * (32 * nt + col) + 2 * hl + e]
                                                : make_float4(0.f, 0.f, 0.f, 0.f);
      act = b0 + lane < a.nb ? a.act[img * a.nb + b0 + lane] : 0.f;
    }
  };
  load(base, tid);

  for (int i = tid; i < kp * 2; i += kImgThreads) {
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = i < k * 2 ? gcb[8 * i + e] : 0.f;
    bf16_pieces(make_float4(x[0], x[1], x[2], x[3]), make_float4(x[4], x[5], x[6], x[7]),
                cpc[2 * i], cpc[2 * i + 1]);
  }
  {
    float h = 0.f;  // thread c: codeword c (k <= 256)
    if (tid < k) {
#pragma unroll
      for (int t = 0; t < 16; ++t) h = __builtin_fmaf(gcb[16 * tid + t], gcb[16 * tid + t], h);
      h *= 0.5f;
    }
    if (tid < kp) hneg[tid] = tid < k ? -h : kImgNever;
    // the wave's largest h; a NaN must not get lost in a maximum
    float m = h == h ? h : __builtin_inff();
#pragma unroll
    for (int x = 1; x < 64; x *= 2) m = fmaxf(m, __shfl_xor(m, x, 64));
    if ((tid & 63) == 0) hmax[tid >> 6] = m;
  }
  if constexpr (ACC) {
    for (int i = tid; i < 4 * ly.k4; i += kImgThreads) wcnt[i] = 0;
    if (tid < 16) blk[16 * kImgThreads + tid] = 0.f;
  }
  __syncthreads();

  // margin per |v|, and alone: 2 (512 u |v| cmax + 198 u (|v| cmax + h)), rounded up
  const float hm = fmaxf(fmaxf(hmax[0], hmax[1]), fmaxf(hmax[2], hmax[3]));
  constexpr uint32_t kRowBits = 31u;
  constexpr float ulp = 1.0f / 16777216.0f, ev = 2.02f * 710.0f * ulp, eh = 2.02f * 198.0f * ulp;
  // (cmax from h, whose squares underflow below 1e-18: what that hides is added)
  const float mv = ev * 1.001f * (__builtin_sqrtf(2.0f * hm) + 1e-18f), mh = eh * hm + 1e-30f;

  float gs[ACC ? NI : 1];  // running sums of codewords (tid >> 4) + 16 i, component tid & 15
  int gn[ACC ? NI : 1];    // their counts
#pragma unroll
  for (int i = 0; i < (ACC ? NI : 1); ++i) gs[i] = 0.f, gn[i] = 0;
  bool fp32_only = false;  // (uniform over the wave)

  for (int rd = 0; rd < kImgAssignBlocks / kImgThreads; ++rd) {
    const int64_t r0 = base + (int64_t)rd * kImgThreads;  // the round's first block
    if (r0 >= a.nb) break;                                // uniform over the workgroup
    // Keep the compiler from hoisting a round's addresses out of the loop: held
    // through all of it they spill.
    int id = tid;
    asm volatile("" : "+v"(id));
    const int wave = __builtin_amdgcn_readfirstlane(id >> 6), lane = id & 63;
    const int col = lane & 31, hl = lane >> 5;
    const int64_t b = r0 + id;
    const bool in = b < a.nb;
    const bool pat = in && act >= a.tau;
    float4 *bw = reinterpret_cast<float4 *>(blk + 16 * 64 * wave);  // the wave's vectors
    if constexpr (ACC) {
      // the previous round's sums have been read off blk, idx and the counts
      if (rd > 0) {
        __syncthreads();
        for (int i = lane; i < ly.k4; i += 64) wcnt[wave * ly.k4 + i] = 0;
      }
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
#pragma unroll
        for (int e = 0; e < 2; ++e) bw[4 * (32 * nt + col) + 2 * hl + e] = vb[nt][e];
    }
    img_b8 vh[2], vl[2];
    float need;  // margin of the lane's own block (nt = hl; its other half is in lane ^ 32)
    {
      float n2[2];  // the lane's share of |v|^2
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        const float4 p = vb[nt][0], q = vb[nt][1];
        bf16_pieces(p, q, vh[nt], vl[nt]);
        n2[nt] = p.x * p.x + p.y * p.y + p.z * p.z + p.w * p.w + q.x * q.x + q.y * q.y +
                 q.z * q.z + q.w * q.w;
      }
      need =
          mv * __builtin_sqrtf((hl ? n2[1] : n2[0]) + __shfl_xor(hl ? n2[0] : n2[1], 32, 64)) + mh;
    }
    // the next round's vectors take this one's registers
    if (rd + 1 < kImgAssignBlocks / kImgThreads && r0 + kImgThreads < a.nb) load(r0 + kImgThreads, id);
    int best = 0;
    bool open = true;  // not decided by the BF16 products
    if (!fp32_only) {
      float bv[2], sv[2];  // best and second D
      int gr[2];           // the best one's group of 32 codewords
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) bv[nt] = sv[nt] = kImgNever, gr[nt] = 0;
      for (int m0 = 0; m0 < kp; m0 += 32) {
        const img_b8 ch = cpc[2 * (2 * (m0 + col) + hl)], cl = cpc[2 * (2 * (m0 + col) + hl) + 1];
        img_f16 init;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const img_f4 h4 = *reinterpret_cast<const img_f4 *>(hneg + m0 + 8 * q + 4 * hl);
#pragma unroll
          for (int r = 0; r < 4; ++r) init[4 * q + r] = h4[r];
        }
        img_f16 d[2];
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
          d[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch, vh[nt], init, 0, 0, 0);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
          d[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cl, vh[nt], d[nt], 0, 0, 0);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
          d[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch, vl[nt], d[nt], 0, 0, 0);
#pragma unroll
        for (int nt = 0; nt < 2; ++nt) {
          const float was = bv[nt];
#pragma unroll
          for (int r = 0; r < 16; r += 2) {
            // the row within the group, but for bit 2 (hl), in the low bits
            const float x0 = __uint_as_float((__float_as_uint(d[nt][r]) & ~kRowBits) |
                                             (uint32_t)(8 * (r / 4) + r % 4));
            const float x1 = __uint_as_float((__float_as_uint(d[nt][r + 1]) & ~kRowBits) |
                                             (uint32_t)(8 * (r / 4) + r % 4 + 1));
            sv[nt] = max2f(sv[nt], med3f(bv[nt], x0, x1));
            bv[nt] = max3f(bv[nt], x0, x1);
          }
          gr[nt] = bv[nt] > was ? m0 : gr[nt];
        }
      }
      // lanes l and l ^ 32 hold the two halves of a column's rows: each ends
      // with block 32 hl + col, its own
      int code[2];
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
        code[nt] = gr[nt] + 4 * hl + (int)(__float_as_uint(bv[nt]) & kRowBits);
      const float kb = hl ? bv[1] : bv[0], ks = hl ? sv[1] : sv[0];
      const float ob = __shfl_xor(hl ? bv[0] : bv[1], 32, 64);
      const float os = __shfl_xor(hl ? sv[0] : sv[1], 32, 64);
      const int oc = __shfl_xor(hl ? code[0] : code[1], 32, 64);
      best = ob > kb ? oc : hl ? code[1] : code[0];
      const float second = max3f(min2f(kb, ob), ks, os), first = max2f(kb, ob);
      // (an S too large for the pieces, infinite or NaN, leaves the block open)
      open = pat && !(first - second > need && need < 1e30f);
    }
    const uint64_t undecided = __ballot(open);
    if (undecided) {
      // many at once (equal codewords, say): the wave stays with FP32
      if (__popcll(undecided) > 16) fp32_only = true;
      const int64_t b0 = r0 + 64 * wave;
      const int exact = exact_codes(gcb, hneg, k, kp, a.dev + 16 * (img * a.nb + b0), a.nb - b0,
                                    undecided);
      best = open ? exact : best;
    }
    if constexpr (ACC) {
      const int rank = pat ? atomicAdd(&wcnt[wave * ly.k4 + best], 1) : 0;
      __syncthreads();
      if (wave == (rd & 3)) {
        // exclusive scan of the k <= 256 counts, rounded up to 4, by one wave,
        // four codes per lane
        const int c0 = 4 * lane;
        int run = 0, wc[4][4], loc[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int4 n4 = c0 < ly.k4 ? *reinterpret_cast<const int4 *>(wcnt + w * ly.k4 + c0)
                                     : make_int4(0, 0, 0, 0);
          wc[w][0] = n4.x, wc[w][1] = n4.y, wc[w][2] = n4.z, wc[w][3] = n4.w;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          loc[q] = run;
          run += (wc[0][q] + wc[1][q] + wc[2][q] + wc[3][q] + 3) & ~3;
        }
        int incl = run;
#pragma unroll
        for (int d = 1; d < 64; d *= 2) {
          const int o = __shfl_up(incl, d, 64);
          if (lane >= d) incl += o;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) loc[q] += incl - run;
        if (c0 < ly.k4) {
          *reinterpret_cast<int4 *>(off + c0) = make_int4(loc[0], loc[1], loc[2], loc[3]);
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            *reinterpret_cast<int4 *>(woff + w * ly.k4 + c0) =
                make_int4(loc[0], loc[1], loc[2], loc[3]);
#pragma unroll
            for (int q = 0; q < 4; ++q) loc[q] += wc[w][q];
          }
        }
      } else {
        // the other waves point every place of the order at the zero vector
        const int w = (wave - (rd & 3)) & 3;  // 1..3
        for (int i = 64 * (w - 1) + lane; i < ly.nidx / 2; i += 192)
          reinterpret_cast<uint32_t *>(idx)[i] = kImgThreads | (kImgThreads << 16);
      }
      __syncthreads();
      if (pat) idx[woff[wave * ly.k4 + best] + rank] = (uint16_t)id;
      __syncthreads();
      const int g = id >> 4, t = id & 15;
      const float *bt = blk + t;
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int c = g + 16 * i;
        if (c < k) {
          const int n = wcnt[c] + wcnt[ly.k4 + c] + wcnt[2 * ly.k4 + c] + wcnt[3 * ly.k4 + c];
          const int q0 = off[c];
          float sum = 0.f;
          // (adding the zero vector of a run's padding changes no sum)
          for (int q = q0; q < q0 + n; q += 4) {
            const uint2 e = *reinterpret_cast<const uint2 *>(idx + q);
            const float v0 = bt[16 * (e.x & 0xffffu)], v1 = bt[16 * (e.x >> 16)];
            const float v2 = bt[16 * (e.y & 0xffffu)], v3 = bt[16 * (e.y >> 16)];
            sum += v0;
            sum += v1;
            sum += v2;
            sum += v3;
          }
          gs[i] += sum;
          gn[i] += n;
        }
      }
    } else {
      if (in) a.code[img * a.nb + b] = pat ? best + 1 : 0;
    }
  }
  if constexpr (ACC) {
    const int g = tid >> 4, t = tid & 15;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = g + 16 * i;
      if (c < k) {
        float *part = a.part + ((img * k + c) * a.agroups + grp) * 17;
        part[t] = gs[i];
        if (t == 0) part[16] = (float)gn[i];
      }
    }
  }
}

// Dynamic LDS of k_img_assign for k codewords.
size_t img_assign_lds_bytes(int k, bool accumulate) {
  return sizeof(float) * (size_t)AssignLds(k, accumulate).total;
}

// New codewords: one workgroup per (codeword blockIdx.x, image blockIdx.y).
// Thread i adds the partials of groups i, i + 256, ... in order, then the 256
// thread sums are added in a fixed tree (two steps through LDS, the rest inside
// a wave), so the result does not depend on scheduling; a codeword without
// blocks keeps its value.  The partials of a codeword lie back to back (68
// bytes per group): 11 us for 16 images, k = 64, with the groups' partials in
// (group, codeword) order and every step of the tree through LDS;
// 7 us now.
__global__ void __launch_bounds__(256) k_img_update(ImgArgs a) {
  __shared__ float red[17][256];
  const int64_t img = blockIdx.y;
  const int c = blockIdx.x, tid = threadIdx.x;
  const float *part = a.part + (img * a.k + c) * (int64_t)a.agroups * 17;
  float s[17];
#pragma unroll
  for (int t = 0; t < 17; ++t) s[t] = 0.f;
  for (int g = tid; g < a.agroups; g += 256) {
    const float *p = part + g * 17;
#pragma unroll
    for (int t = 0; t < 17; ++t) s[t] += p[t];
  }
#pragma unroll
  for (int t = 0; t < 17; ++t) red[t][tid] = s[t];
  __syncthreads();
  if (tid < 128) {
#pragma unroll
    for (int t = 0; t < 17; ++t) red[t][tid] += red[t][tid + 128];
  }
  __syncthreads();
  if (tid >= 64) return;
#pragma unroll
  for (int t = 0; t < 17; ++t) {
    s[t] = red[t][tid] + red[t][tid + 64];
#pragma unroll
    for (int st = 32; st > 0; st >>= 1) s[t] += __shfl_down(s[t], st, 64);
  }
  if (tid == 0 && s[16] > 0.f) {
#pragma unroll
    for (int t = 0; t < 16; ++t) a.codebook[(img * a.k + c) * 16 + t] = s[t] / s[16];
  }
}

const void *img_kernel_front() { return (const void *)&k_img_front; }
const void *img_kernel_count() { return (const void *)&k_img_count; }
const void *img_kernel_scan() { return (const void *)&k_img_scan; }
const void *img_kernel_seed() { return (const void *)&k_img_seed; }
const void *img_kernel_assign(bool accumulate, int k) {
  // sums of up to 4, 8 or 16 codewords per 16-lane group in registers
  return !accumulate ? (const void *)&k_img_assign<0>
         : k <= 64   ? (const void *)&k_img_assign<4>
         : k <= 128  ? (const void *)&k_img_assign<8>
                     : (const void *)&k_img_assign<16>;
}
const void *img_kernel_update() { return (const void *)&k_img_update; }

}  // namespace dpfft
