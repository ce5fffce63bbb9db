// Bloom (lens glare, Section 3.4.3): a point spread function approximated by small-support
// filters on the mipmaps of the final image, before tone mapping.
//
//   P_0 = I;  P_k = 2x2 box average of P_{k-1} (ceil(n/2) per axis, clamped source indices)
//   U_K = w_K P_K;  U_k = w_k P_k + up(U_{k+1});  O = w_0 I + up(U_1)
//
// up() doubles the resolution bilinearly: fine pixel x reads the coarse grid at x/2 - 1/4,
// i.e. coarse pixels (x-1)>>1 and (x+1)>>1 with weights 3/4, 1/4 (or 1/4, 3/4), clamped to
// the edge.  With weights summing to 1 an interior impulse keeps its flux.
//
// Three launches:
//   k_bloom_down  one workgroup per 64x64 image tile builds the tile's levels 1..6 in LDS
//                 (a level-k pixel depends on a 2^k x 2^k block of the image, inside one
//                 tile) and writes them (HBM-bound: reads the image once);
//   k_bloom_tail  one workgroup builds the coarse levels 7..K and their U chain, which are
//                 small (at most 120 x 68 pixels at 7680 x 4320), only when K > 7 (for
//                 K = 7 the output pass forms the U_7 values it needs from level 6);
//   k_bloom_up    one workgroup per 64x64 or 32x32 output tile (launch_bloom_up says which)
//                 runs the U chain for levels 6..1 over the tile plus the one-pixel halo each
//                 bilinear doubling needs, in LDS, then writes O (HBM-bound: reads the image
//                 once more, writes O), or O's display encoding (below) in place of O.
//
// Display encoding (the tone mapping that follows the glare pass; the paper prints no
// operator, so this is one reading): per colour channel c, x = exposure * c, y = 1 - exp(-x)
// (0 for x <= 0 or NaN), v = the sRGB transfer function of y (IEC 61966-2-1), 8-bit code
// floor(255 v + 1/2); alpha 255; bytes R, G, B, A.  k_tonemap applies it to a whole image.
#include "bh_dev.h"

namespace bh {

constexpr int kBloomTileLevels = 6;  // levels built inside a 64 x 64 tile

__device__ __forceinline__ float4 f4_fma(float a, float4 x, float4 y) {
  return make_float4(fmaf(a, x.x, y.x), fmaf(a, x.y, y.y), fmaf(a, x.z, y.z), fmaf(a, x.w, y.w));
}

__device__ __forceinline__ float4 box4(float4 a, float4 b, float4 c, float4 d) {
  return make_float4(0.25f * ((a.x + b.x) + (c.x + d.x)), 0.25f * ((a.y + b.y) + (c.y + d.y)),
                     0.25f * ((a.z + b.z) + (c.z + d.z)), 0.25f * ((a.w + b.w) + (c.w + d.w)));
}

// bilinear blend of the four coarse neighbours of a fine pixel (fx, fy: weights of the
// second column / row, 1/4 or 3/4): two rows across, then the rows
__device__ __forceinline__ float4 across(float4 v0, float4 v1, float fx) {
  const float gx = 1.0f - fx;
  return make_float4(gx * v0.x + fx * v1.x, gx * v0.y + fx * v1.y, gx * v0.z + fx * v1.z,
                     gx * v0.w + fx * v1.w);
}
__device__ __forceinline__ float4 down(float4 a, float4 b, float fy) { return across(a, b, fy); }
__device__ __forceinline__ float4 blend(float4 v00, float4 v10, float4 v01, float4 v11, float fx,
                                        float fy) {
  return down(across(v00, v10, fx), across(v01, v11, fx), fy);
}

// ---- display encoding ------------------------------------------------------------------------

// 8-bit code of one colour channel.  1 - exp(-x) loses ~1e-7 absolute to cancellation, which
// the linear sRGB segment (3295 codes per unit) would turn into 4e-4 codes, so below x = 1/16
// it comes from its Taylor series to x^5 (truncation below 1e-9 relative).  With hardware
// exp2 and log2 (about 1 ulp each) the value whose floor is the code stays within 2e-4 of its
// exact value.
__device__ __forceinline__ uint32_t display_code(float c, float exposure) {
  const float x = exposure * c;
  if (!(x > 0.0f)) return 0u;
  const float series =
      x * fmaf(-x, fmaf(-x, fmaf(-x, fmaf(-x, 1.0f / 120.0f, 1.0f / 24.0f), 1.0f / 6.0f), 0.5f),
               1.0f);
  const float y = x < 0.0625f ? series
                              : 1.0f - __builtin_amdgcn_exp2f(x * -1.44269504088896341f);
  const float v = y <= 0.0031308f
                      ? 12.92f * y
                      : fmaf(1.055f,
                             __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(y) * (1.0f / 2.4f)),
                             -0.055f);
  return min((uint32_t)fmaf(255.0f, v, 0.5f), 255u);  // v >= 0: truncation is the floor
}

__device__ __forceinline__ uint32_t display_pixel(float4 c, float exposure) {
  return display_code(c.x, exposure) | (display_code(c.y, exposure) << 8) |
         (display_code(c.z, exposure) << 16) | 0xff000000u;
}

__global__ void __launch_bounds__(256)
    k_tonemap(const float4* __restrict__ in, uint32_t* __restrict__ out, int64_t n,
              float exposure) {
  // two pixels per thread, one grid apart (both loads in flight before either encoding);
  // the launch has ceil(n / 512) workgroups, so i0 + step covers the rest of the image
  const int64_t step = (int64_t)gridDim.x * 256;
  const int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x, i1 = i0 + step;
  const float4 a = i0 < n ? in[i0] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  const float4 b = i1 < n ? in[i1] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  if (i0 < n) store_stream(&out[i0], display_pixel(a, exposure));
  if (i1 < n) store_stream(&out[i1], display_pixel(b, exposure));
}

// ---- level building inside one 64 x 64 tile --------------------------------------------------

// LDS holds level k of the tile at local index l for every l in [0, 64 / 2^k), also beyond
// the level's last pixel: an entry past it holds the last pixel's value (its index clamped),
// so the next level's 2x2 averages need no clamping of their own.
constexpr int kDownThreads = 512;

__global__ void __launch_bounds__(kDownThreads)
    k_bloom_down(const float4* __restrict__ img, float4* __restrict__ P, BloomDev B) {
  __shared__ float4 s1[32 * 32];
  __shared__ float4 s2[16 * 16];
  const int tx = blockIdx.x % B.tiles_x, ty = blockIdx.x / B.tiles_x;
  const int m = min(B.levels, kBloomTileLevels);
  const int t = threadIdx.x;
  float4* cur = s1;
  float4* nxt = s2;
  // level 1 from the image, every load in flight before the first average
  {
    constexpr int kEach = 32 * 32 / kDownThreads;
    const int n1x = B.w[1], n1y = B.h[1];
    const int lx = t & 31, gx = tx * 32 + lx, cx = min(gx, n1x - 1);
    const int x0 = 2 * cx, x1 = min(x0 + 1, B.w[0] - 1);
    float4 v[kEach][4];
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
      const int cy = min(ty * 32 + (t >> 5) + j * (kDownThreads / 32), n1y - 1);
      const float4* r0 = img + (size_t)(2 * cy) * B.w[0];
      const float4* r1 = img + (size_t)min(2 * cy + 1, B.h[0] - 1) * B.w[0];
      v[j][0] = r0[x0];
      v[j][1] = r0[x1];
      v[j][2] = r1[x0];
      v[j][3] = r1[x1];
    }
#pragma unroll
    for (int j = 0; j < kEach; ++j) {
      const int ly = (t >> 5) + j * (kDownThreads / 32), gy = ty * 32 + ly;
      const float4 p = box4(v[j][0], v[j][1], v[j][2], v[j][3]);
      cur[ly * 32 + lx] = p;
      if (gx < n1x && gy < n1y) P[B.off[1] + (size_t)gy * n1x + gx] = p;
    }
  }
  __syncthreads();
  // levels 2 .. m from the previous level in LDS
  for (int k = 2; k <= m; ++k) {
    const int lside = 6 - k, side = 1 << lside, pside = side * 2;
    const int nx = B.w[k], ny = B.h[k];
    const int sx = tx * side, sy = ty * side;  // the tile's first level-k pixel
    for (int l = t; l < side * side; l += kDownThreads) {
      const int lx = l & (side - 1), ly = l >> lside;
      const int cx = min(sx + lx, nx - 1) - sx, cy = min(sy + ly, ny - 1) - sy;
      const float4 v = box4(cur[(2 * cy) * pside + 2 * cx], cur[(2 * cy) * pside + 2 * cx + 1],
                            cur[(2 * cy + 1) * pside + 2 * cx],
                            cur[(2 * cy + 1) * pside + 2 * cx + 1]);
      nxt[l] = v;
      if (sx + lx < nx && sy + ly < ny) P[B.off[k] + (size_t)(sy + ly) * nx + sx + lx] = v;
    }
    __syncthreads();
    float4* sw = cur;
    cur = nxt;
    nxt = sw;
  }
}

// levels 7 .. K and U_K .. U_7, one workgroup, a barrier between levels.  LDS: the levels live
// in shared memory (U_k overwrites P_k in place) and only U_7, which the output tiles read, goes
// to global memory; used when levels 7 .. K hold at most kBloomTailLds pixels (7680 x 4320
// needs 2685).  Otherwise the levels are kept in global memory.
constexpr int kBloomTailLds = 3072;

template <bool LDS>
__global__ void __launch_bounds__(256)
    k_bloom_tail(float4* __restrict__ P, float4* __restrict__ U, BloomDev B) {
  __shared__ float4 sl[LDS ? kBloomTailLds : 1];
  const int t = threadIdx.x;
  const int64_t base = B.off[kBloomTileLevels + 1];
  for (int k = kBloomTileLevels + 1; k <= B.levels; ++k) {
    const int nx = B.w[k], ny = B.h[k], px = B.w[k - 1], py = B.h[k - 1];
    for (int l = t; l < nx * ny; l += 256) {
      const int x = l % nx, y = l / nx;
      const int x0 = 2 * x, y0 = 2 * y, x1 = min(x0 + 1, px - 1), y1 = min(y0 + 1, py - 1);
      float4 v;
      if (!LDS || k == kBloomTileLevels + 1) {
        const float4* src = P + B.off[k - 1];
        v = box4(src[(size_t)y0 * px + x0], src[(size_t)y0 * px + x1],
                 src[(size_t)y1 * px + x0], src[(size_t)y1 * px + x1]);
      } else {
        const float4* src = sl + (B.off[k - 1] - base);
        v = box4(src[y0 * px + x0], src[y0 * px + x1], src[y1 * px + x0], src[y1 * px + x1]);
      }
      if (LDS)
        sl[B.off[k] - base + l] = v;
      else
        P[B.off[k] + l] = v;
    }
    __syncthreads();
  }
  for (int k = B.levels; k > kBloomTileLevels; --k) {
    const int nx = B.w[k], ny = B.h[k];
    const float wk = B.wt[k];
    for (int l = t; l < nx * ny; l += 256) {
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (k < B.levels) {
        const int x = l % nx, y = l / nx, cx = B.w[k + 1], cy = B.h[k + 1];
        const int xa = max((x - 1) >> 1, 0), xb = min((x + 1) >> 1, cx - 1);
        const int ya = max((y - 1) >> 1, 0), yb = min((y + 1) >> 1, cy - 1);
        const float4* c = LDS ? sl + (B.off[k + 1] - base) : U + B.off[k + 1];
        v = blend(c[ya * cx + xa], c[ya * cx + xb], c[yb * cx + xa], c[yb * cx + xb],
                  (x & 1) ? 0.25f : 0.75f, (y & 1) ? 0.25f : 0.75f);
      }
      const float4 u = f4_fma(wk, LDS ? sl[B.off[k] - base + l] : P[B.off[k] + l], v);
      if (LDS) {
        sl[B.off[k] - base + l] = u;
        if (k == kBloomTileLevels + 1) U[B.off[k] + l] = u;
      } else {
        U[B.off[k] + l] = u;
      }
    }
    __syncthreads();
  }
}

// ---- the U chain and the output, per T x T output tile ------------------------------------------
//
// A 64 x 64 tile reads level-1 pixels 32 t - 1 .. 32 t + 32 (34 per axis), level-2 pixels 18 per
// axis, then 10, 6, 4 and 3 at level 6.  Levels 2 .. 6 together are 485 pixels, so each thread
// owns at most one of them (and its share of level 1): its P value is loaded first, together with
// the thread's image pixels, and the chain of levels then waits on LDS only.  A wave computes
// only the levels it owns elements of, and two output rows at a time come from the same three
// rows of U_1.  With every level's elements spread over all threads and one output row at a
// time, the display form issued 829 vector instructions a wave for 4 pixels a lane: 18.4 us at
// 1920 x 1080, now 16.2 (whole pass 26.5 -> 23.7; linear 3839 x 2158 93.7 -> 86.2).  At 1920 x
// 1080 every workgroup is resident at once, so the phases (the image's loads, the chain, the
// encoding) add up instead of overlapping.
struct Region {
  int lox, hix, loy, hiy;
};

// Shape of the output pass: T x T tiles of TH threads.  side(k): the most pixels an axis that a
// tile reads of level k, which is also that level's LDS row stride (T / 2^k + 2, at least 3).
template <int T_, int TH_>
struct UpShape {
  static constexpr int T = T_, TH = TH_;
  static constexpr int side(int k) { return T / (1 << k) + 2 < 3 ? 3 : T / (1 << k) + 2; }
  // first thread that owns an element of level k >= 2
  static constexpr int first(int k) {
    int n = 0;
    for (int j = 2; j < k; ++j) n += side(j) * side(j);
    return n;
  }
  static constexpr int kRest = first(kBloomTileLevels + 1);
  static_assert(kRest <= TH, "one element of levels 2 .. 6 a thread");
  static_assert(TH % T == 0 && T % (2 * (TH / T)) == 0, "whole row pairs per pass");
};

template <class S>
struct UpLds {
  float4 l1[S::side(1) * S::side(1)];
  float4 rest[S::kRest];  // levels 2 .. 6, level k from S::first(k)
  float4 u7[16];          // the level-7 neighbourhood of level 6's region (row stride 4)
};

// the thread's element of level K (>= 2): true when it owns one inside the region
template <class S, int K>
__device__ __forceinline__ bool up_element(const Region& R, int* r, int* c) {
  constexpr int N = S::side(K);
  const int e = (int)threadIdx.x - S::first(K);
  if (e < 0 || e >= N * N) return false;
  *r = e / N;
  *c = e - *r * N;
  return *c <= R.hix - R.lox && *r <= R.hiy - R.loy;
}

template <class S, int K>
__device__ __forceinline__ void load_p(const BloomDev& B, const float4* __restrict__ P,
                                       const Region& R, float4* p) {
  int r, c;
  if (up_element<S, K>(R, &r, &c))
    *p = P[B.off[K] + (size_t)(R.loy + r) * B.w[K] + R.lox + c];
}

// U_7 = w_7 P_7 at level-7 pixel (x, y) of a pyramid of exactly 7 levels, from level 6: the
// operations of the tail kernel, in its order, so the values are the same bits
__device__ __forceinline__ float4 u7_from_p6(const BloomDev& B, const float4* __restrict__ P,
                                             int x, int y) {
  constexpr int K = kBloomTileLevels + 1;
  const int px = B.w[K - 1], py = B.h[K - 1];
  const int x0 = 2 * x, y0 = 2 * y, x1 = min(x0 + 1, px - 1), y1 = min(y0 + 1, py - 1);
  const float4* src = P + B.off[K - 1];
  const float4 p = box4(src[(size_t)y0 * px + x0], src[(size_t)y0 * px + x1],
                        src[(size_t)y1 * px + x0], src[(size_t)y1 * px + x1]);
  return f4_fma(B.wt[K], p, make_float4(0.f, 0.f, 0.f, 0.f));
}

// The level-7 neighbourhood of a tile's level-6 region R: at most 3 x 3 pixels
__device__ __forceinline__ Region coarse_region(const BloomDev& B, const Region& R) {
  constexpr int K = kBloomTileLevels + 1;
  return Region{max((R.lox - 1) >> 1, 0), min((R.hix + 1) >> 1, B.w[K] - 1),
                max((R.loy - 1) >> 1, 0), min((R.hiy + 1) >> 1, B.h[K] - 1)};
}

// U_7 over the region C, one value per thread, into LDS `su7` (row stride 4): with exactly 7
// levels formed from level 6, with more from the global U array the tail kernel wrote
__device__ __forceinline__ void fill_u7(const BloomDev& B, const float4* __restrict__ P,
                                        const float4* __restrict__ U, const Region& C,
                                        float4* su7) {
  constexpr int K = kBloomTileLevels + 1;
  const int x = threadIdx.x & 3, y = threadIdx.x >> 2;
  if (x > C.hix - C.lox || y > C.hiy - C.loy) return;
  su7[threadIdx.x] = B.levels == K
                         ? u7_from_p6(B, P, C.lox + x, C.loy + y)
                         : U[B.off[K] + (size_t)(C.loy + y) * B.w[K] + C.lox + x];
}

// U_K = w_K P_K + up(U_{K+1}) at element (r, c) of level K's region R; `src` holds U_{K+1} over
// the region Rs (row stride SS), absent for K = levels
template <int K, int SS>
__device__ __forceinline__ float4 u_value(const BloomDev& B, float4 p, const Region& R, int r,
                                          int c, const float4* src, const Region& Rs) {
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (K < B.levels) {
    const int x = R.lox + c, y = R.loy + r, cnx = B.w[K + 1], cny = B.h[K + 1];
    const int xa = max((x - 1) >> 1, 0) - Rs.lox, xb = min((x + 1) >> 1, cnx - 1) - Rs.lox;
    const int ya = (max((y - 1) >> 1, 0) - Rs.loy) * SS;
    const int yb = (min((y + 1) >> 1, cny - 1) - Rs.loy) * SS;
    v = blend(src[ya + xa], src[ya + xb], src[yb + xa], src[yb + xb], (x & 1) ? 0.25f : 0.75f,
              (y & 1) ? 0.25f : 0.75f);
  }
  return f4_fma(B.wt[K], p, v);
}

// level K = 6 .. 2 of the chain: the threads that own an element write U_K
template <class S, int K>
__device__ __forceinline__ void u_level(const BloomDev& B, const float4& p, const Region& R,
                                        const Region& Rs, UpLds<S>& L) {
  int r, c;
  if (!up_element<S, K>(R, &r, &c)) return;
  if constexpr (K == kBloomTileLevels)
    L.rest[threadIdx.x] = u_value<K, 4>(B, p, R, r, c, L.u7, Rs);
  else
    L.rest[threadIdx.x] =
        u_value<K, S::side(K + 1)>(B, p, R, r, c, L.rest + S::first(K + 1), Rs);
}

// DISPLAY: `out` receives the display encoding of O (uint32 per pixel), else O (float4)
template <class S, bool DISPLAY>
__global__ void __launch_bounds__(S::TH)
    k_bloom_up(const float4* __restrict__ img, void* __restrict__ out,
               const float4* __restrict__ P, const float4* __restrict__ U, BloomDev B,
               float exposure) {
  constexpr int T = S::T, TH = S::TH, S1 = S::side(1), N1 = (S1 * S1 + TH - 1) / TH;
  __shared__ UpLds<S> L;
  const int ntx = (B.w[0] + T - 1) / T;
  const int tx = blockIdx.x % ntx, ty = blockIdx.x / ntx;
  const int m = min(B.levels, kBloomTileLevels);
  // regions of levels 0 .. 6
  Region R[kBloomTileLevels + 1];
  R[0].lox = tx * T;
  R[0].hix = min(R[0].lox + T - 1, B.w[0] - 1);
  R[0].loy = ty * T;
  R[0].hiy = min(R[0].loy + T - 1, B.h[0] - 1);
#pragma unroll
  for (int k = 1; k <= kBloomTileLevels; ++k) {
    const int nx = B.w[min(k, B.levels)], ny = B.h[min(k, B.levels)];
    R[k].lox = max((R[k - 1].lox - 1) >> 1, 0);
    R[k].hix = min((R[k - 1].hix + 1) >> 1, nx - 1);
    R[k].loy = max((R[k - 1].loy - 1) >> 1, 0);
    R[k].hiy = min((R[k - 1].hiy + 1) >> 1, ny - 1);
  }
  // P of the chain, in flight at once (levels beyond m are not loaded)
  float4 pk, p1[N1];
  if (m >= 6) load_p<S, 6>(B, P, R[6], &pk);
  if (m >= 5) load_p<S, 5>(B, P, R[5], &pk);
  if (m >= 4) load_p<S, 4>(B, P, R[4], &pk);
  if (m >= 3) load_p<S, 3>(B, P, R[3], &pk);
  if (m >= 2) load_p<S, 2>(B, P, R[2], &pk);
  if (m >= 1) {
#pragma unroll
    for (int j = 0; j < N1; ++j) {
      const int l = threadIdx.x + TH * j, r = l / S1, c = l - r * S1;
      if (c <= R[1].hix - R[1].lox && r <= R[1].hiy - R[1].loy)
        p1[j] = P[B.off[1] + (size_t)(R[1].loy + r) * B.w[1] + R[1].lox + c];
    }
  }
  const Region C7 = coarse_region(B, R[6]);
  if (B.levels > kBloomTileLevels && threadIdx.x < 16) fill_u7(B, P, U, C7, L.u7);
  // this thread's image pixels (column x, row pairs y0 + kStep j), in flight during the chain;
  // positions past the image's edge load the edge pixel, unused
  constexpr int kStep = 2 * (TH / T), kIt = T / kStep;
  const int x = R[0].lox + (int)(threadIdx.x % T);
  const int y0 = R[0].loy + 2 * (int)(threadIdx.x / T);
  float4 im[kIt][2];
#pragma unroll
  for (int j = 0; j < kIt; ++j)
#pragma unroll
    for (int q = 0; q < 2; ++q)
      im[j][q] = img[(size_t)min(y0 + kStep * j + q, R[0].hiy) * B.w[0] + min(x, R[0].hix)];
  // U_k, k = m .. 1 (m is the same for the whole launch, so the barriers are uniform)
  if (B.levels > kBloomTileLevels) __syncthreads();
  if (m >= 6) { u_level<S, 6>(B, pk, R[6], C7, L); __syncthreads(); }
  if (m >= 5) { u_level<S, 5>(B, pk, R[5], R[6], L); __syncthreads(); }
  if (m >= 4) { u_level<S, 4>(B, pk, R[4], R[5], L); __syncthreads(); }
  if (m >= 3) { u_level<S, 3>(B, pk, R[3], R[4], L); __syncthreads(); }
  if (m >= 2) { u_level<S, 2>(B, pk, R[2], R[3], L); __syncthreads(); }
  if (m >= 1) {
#pragma unroll
    for (int j = 0; j < N1; ++j) {
      const int l = threadIdx.x + TH * j, r = l / S1, c = l - r * S1;
      if (c <= R[1].hix - R[1].lox && r <= R[1].hiy - R[1].loy)
        L.l1[l] = u_value<1, S::side(2)>(B, p1[j], R[1], r, c, L.rest, R[2]);
    }
    __syncthreads();
  }
  // O = w_0 I + up(U_1): rows 2i and 2i + 1 blend rows i - 1, i and i, i + 1 of U_1
  if (x > R[0].hix) return;
  const float w0 = B.wt[0];
  const int cnx = B.w[1], cny = B.h[1];
  const int xa = max((x - 1) >> 1, 0) - R[1].lox, xb = min((x + 1) >> 1, cnx - 1) - R[1].lox;
  const float fx = (x & 1) ? 0.25f : 0.75f;
#pragma unroll
  for (int j = 0; j < kIt; ++j) {
    const int y = y0 + kStep * j, i = y >> 1;
    if (y > R[0].hiy) break;
    float4 h[3];  // rows i - 1, i, i + 1 of U_1 at column x
    if (B.levels >= 1) {
      const int row[3] = {max(i - 1, 0), min(i, cny - 1), min(i + 1, cny - 1)};
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const float4* s = L.l1 + (row[q] - R[1].loy) * S1;
        h[q] = across(s[xa], s[xb], fx);
      }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (q && y + 1 > R[0].hiy) break;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      if (B.levels >= 1) v = down(h[q], h[q + 1], q ? 0.25f : 0.75f);
      const float4 o = f4_fma(w0, im[j][q], v);
      const size_t at = (size_t)(y + q) * B.w[0] + x;
      if constexpr (DISPLAY)
        store_stream(&static_cast<uint32_t*>(out)[at], display_pixel(o, exposure));
      else
        store_stream(&static_cast<float4*>(out)[at], o);
    }
  }
}

hipError_t launch_tonemap(const float4* in, uint32_t* out, int64_t n, float exposure,
                          hipStream_t s) {
  hipLaunchKernelGGL(k_tonemap, dim3((unsigned)((n + 511) / 512)), dim3(256), 0, s, in, out, n,
                     exposure);
  return hipGetLastError();
}

template <int T, int TH, bool DISPLAY>
static void up(const float4* in, void* out, const float4* P, const float4* U, const BloomDev& B,
               float exposure, hipStream_t s) {
  const int tiles = ((B.w[0] + T - 1) / T) * ((B.h[0] + T - 1) / T);
  hipLaunchKernelGGL((k_bloom_up<UpShape<T, TH>, DISPLAY>), dim3(tiles), dim3(TH), 0, s, in, out,
                     P, U, B, exposure);
}

// Output tiles.  64 x 64 tiles read the least around each tile, but a small image has too few of
// them to fill the chip: below kUpFewTiles (about 960 x 540) 32 x 32 tiles of 8 waves (640 x 360
// display: 11.4 against 13.3 us; 1280 x 720: 17.4 against 14.7).  64 x 64 tiles of 8 waves reside
// four on a CU and overlap their phases; with the encoding's arithmetic 16 waves a tile are
// quicker while the image is one round of them, two on a CU (kUpRoundTiles).  Display, us, 16
// waves and 8: 1920 x 1080 (510 tiles) 23.9 and 24.4, 1600 x 900 19.6 and 20.6; 1920 x 1200 (570)
// 30.1 and 29.0, 2560 x 1440 40.2 and 39.6, 3840 x 2160 73.4 and 70.4, 3839 x 2158 77.2 and 75.1,
// 7680 x 4320 281 and 276.  Linear: 1920 x 1080 21.6 and 21.3, 1920 x 1200 27.6 and 25.2, 3839 x
// 2158 86.1 and 86.2, 5120 x 2880 148 and 141.  (32 x 32 tiles of 4 waves: 3839 x 2158 display
// 78.8, 5120 x 2880 125 against 120.)
constexpr int kUpFewTiles = 128, kUpRoundTiles = 512;

static hipError_t launch_bloom_up(const float4* in, void* out, const float4* P, const float4* U,
                                  const BloomDev& B, bool display, float exposure,
                                  hipStream_t s) {
  const int tiles = B.tiles_x * B.tiles_y;
  if (tiles < kUpFewTiles) {
    display ? up<32, 512, true>(in, out, P, U, B, exposure, s)
            : up<32, 512, false>(in, out, P, U, B, exposure, s);
  } else if (display) {
    tiles > kUpRoundTiles ? up<64, 512, true>(in, out, P, U, B, exposure, s)
                          : up<64, 1024, true>(in, out, P, U, B, exposure, s);
  } else {
    up<64, 512, false>(in, out, P, U, B, exposure, s);
  }
  return hipGetLastError();
}

// display: write the display encoding of O (exposure) to `out` (uint32 per pixel), else O
hipError_t launch_bloom(const float4* in, void* out, float4* P, float4* U, const BloomDev& B,
                        bool display, float exposure, hipStream_t s) {
  const int tiles = B.tiles_x * B.tiles_y;
  if (B.levels >= 1) {
    hipLaunchKernelGGL(k_bloom_down, dim3(tiles), dim3(kDownThreads), 0, s, in, P, B);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  // with exactly 7 levels the output pass computes the few U_7 values it needs itself
  if (B.levels > kBloomTileLevels + 1) {
    const int64_t tail = B.off[B.levels] + (int64_t)B.w[B.levels] * B.h[B.levels] -
                         B.off[kBloomTileLevels + 1];
    if (tail <= kBloomTailLds)
      hipLaunchKernelGGL(k_bloom_tail<true>, dim3(1), dim3(256), 0, s, P, U, B);
    else
      hipLaunchKernelGGL(k_bloom_tail<false>, dim3(1), dim3(256), 0, s, P, U, B);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return launch_bloom_up(in, out, P, U, B, display, exposure, s);
}

}  // namespace bh
