// Star cube map (Section 3.3.2 "Emitted light").  Each texel of every mip level holds the
// intensity sum of the stars inside it, their intensity-weighted mean temperature and
// their intensity-weighted mean position inside the texel; mips combine the four children
// with the same rule (sum of intensities, intensity-weighted averages).  Stars that land in
// the same level-0 texel are merged by the same rule, in star-index order, so the build is
// deterministic whatever order the atomics run in.
// Face of a direction d: k = argmax |d_k| (ties to the lowest index), face 2k + (d_k < 0),
// U = d_{(k+1)%3} / |d_k|, V = d_{(k+2)%3} / |d_k| in [-1, 1].
// Stored texels: FP16 (I / scale_L, T / 1024, p_u, p_v) with a per-level power-of-two
// scale chosen from the level's largest intensity, or FP32 (I, T, p_u, p_v).
//
// Band-colour maps (light of any colour, Section 3.4.2): each texel holds the band sums
// (R, G, B) of its stars and their position inside the texel weighted by S = R + G + B; mips
// combine the four children by the same rule.  Stored texels: FP16 (R / scale_L, G / scale_L,
// B / scale_L, p_u, p_v, 0, 0, 0) with the per-level power of two of the (I, T) format chosen
// from the level's largest band value, or the same eight values in FP32.
//
// Build.  The level-0 map is cut into square tiles (star_tile_log) and the stars are sorted into
// bins of one or more tiles (count, scan, scatter).  One workgroup then owns a tile: it picks its
// stars from the bin, lists them per texel in LDS (or sorts them, where they are many), merges
// them, and forms every mip level that fits inside the tile, so no level ever goes through
// memory.  The FP16 scales need each level's maximum first: a first pass over the tiles only
// finds the maxima and the tiles' topmost texels, from which k_star_tail forms the remaining
// levels; a second pass merges again (the stars are few against the texels) and writes the
// stored texels and the occupancy bits, each byte once.
// 10^6 stars on 6 x 2048^2: 351 us of kernels (count 19, scatter 41, tiles 119 and 152, tail 13),
// where linking the stars through a texel-sized head array and passing every level through
// FP32 texels in memory took 1550 us, 60 launches and 0.9 GB of scratch.  The map's own 277 MB
// are 45 us; the tile passes wait on their chains of LDS and FP64 latency (a wave lives for 13
// us and issues 450 vector instructions; LDS fits three workgroups a CU).
#include <algorithm>

#include "bh_dev.h"

namespace bh {

struct __align__(8) Half4 {
  _Float16 x, y, z, w;
};
struct __align__(16) Half4x2 {
  Half4 a, b;
};
struct __align__(16) Half8 {
  _Float16 v[8];
};

static inline unsigned blocks_for(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

__global__ void k_fill_int(int* p, int64_t n, int v) {
  int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t < n) p[t] = v;
}

// ---- where a star lands -------------------------------------------------------------------

struct Place {
  bool lit;            // emits and has a direction
  int face, ix, iy;    // level-0 texel
  float pu, pv;        // position inside it
};

template <bool BANDS>
__device__ __forceinline__ Place place_star(const float* __restrict__ dirs,
                                            const float* __restrict__ inten, int64_t s, int n0) {
  const float d0 = dirs[3 * s], d1 = dirs[3 * s + 1], d2 = dirs[3 * s + 2];
  bool lit;
  if constexpr (BANDS) {
    // S > 0 exactly when a band is positive
    lit = inten[3 * s] > 0.0f || inten[3 * s + 1] > 0.0f || inten[3 * s + 2] > 0.0f;
  } else {
    lit = inten[s] > 0.0f;
  }
  const float a0 = fabsf(d0), a1 = fabsf(d1), a2 = fabsf(d2);
  int k = 0;
  float m = a0;
  if (a1 > m) { k = 1; m = a1; }
  if (a2 > m) { k = 2; m = a2; }
  Place p;
  p.lit = lit && m > 0.0f;
  const float dk = k == 0 ? d0 : (k == 1 ? d1 : d2);
  const float da = k == 0 ? d1 : (k == 1 ? d2 : d0);
  const float db = k == 0 ? d2 : (k == 1 ? d0 : d1);
  p.face = 2 * k + (dk < 0.0f);
  const float U = da / m, V = db / m;
  const float gx = 0.5f * (U + 1.0f) * (float)n0, gy = 0.5f * (V + 1.0f) * (float)n0;
  p.ix = min(max((int)floorf(gx), 0), n0 - 1);
  p.iy = min(max((int)floorf(gy), 0), n0 - 1);
  p.pu = gx - (float)p.ix;
  p.pv = gy - (float)p.iy;
  return p;
}

// bin of a star, and its texel inside the bin (column low, row high)
__device__ __forceinline__ int bin_of(const Place& p, int n0, int bl) {
  const int nb = n0 >> bl;
  return (p.face * nb + (p.iy >> bl)) * nb + (p.ix >> bl);
}
__device__ __forceinline__ uint32_t bin_texel(const Place& p, int bl) {
  const int mask = (1 << bl) - 1;
  return (uint32_t)(p.ix & mask) | ((uint32_t)(p.iy & mask) << 16);
}

// ---- content hash and bin counts ------------------------------------------------------------

// Content hash of a star field, the key under which its maps are shared: every star
// contributes a 64-bit mix of its index and the bit patterns of its values, and the
// contributions are summed (addition commutes, so the result does not depend on the order
// the atomics run in).  The mix is the splitmix64 finaliser.  A band field starts from a
// different seed, so it never shares a key with an (I, T) field.
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

template <bool BANDS>
__device__ __forceinline__ uint64_t star_hash(const float* __restrict__ dirs,
                                              const float* __restrict__ inten,
                                              const float* __restrict__ temp, int64_t s) {
  uint64_t h = mix64((uint64_t)s + (BANDS ? 0x632be59bd9b4e019ull : 0x9e3779b97f4a7c15ull));
  h = mix64(h ^ __float_as_uint(dirs[3 * s]));
  h = mix64(h ^ ((uint64_t)__float_as_uint(dirs[3 * s + 1]) << 32));
  h = mix64(h ^ __float_as_uint(dirs[3 * s + 2]));
  if constexpr (BANDS) {
    h = mix64(h ^ ((uint64_t)__float_as_uint(inten[3 * s]) << 32));
    h = mix64(h ^ __float_as_uint(inten[3 * s + 1]));
    h = mix64(h ^ ((uint64_t)__float_as_uint(inten[3 * s + 2]) << 32));
  } else {
    h = mix64(h ^ ((uint64_t)__float_as_uint(inten[s]) << 32));
    h = mix64(h ^ __float_as_uint(temp[s]));
  }
  return h;
}

// The sorting kernels keep their counts in LDS and add them to the bins' with one global
// atomic per bin and workgroup.  Large workgroups (8192 stars) and at most
// kMaxBins bins keep those few: 10^6 stars straight onto the 6144 tiles of 6 x 2048^2
// were 10^6 scattered device atomics, 65 us a pass; onto the 96 of 6 x 256^2, 10^4 queued on
// each counter.
constexpr int kSortThreads = 1024, kSortPer = 8, kSortStars = kSortThreads * kSortPer;
constexpr int kMaxBins = 1536;

// Hash of the field, stars per bin and whether a band value is negative, infinite or NaN, which
// fails the whole build (unless `count` and `bad` are null).  One 64-bit atomic per workgroup:
// one per wave queued 15 600 of them on the same address, 192 us for 10^6 stars.  Each thread takes
// `per` stars, fewer in a small field, so that it spreads over the chip.
template <bool BANDS>
__global__ void __launch_bounds__(kSortThreads)
    k_star_count(const float* __restrict__ dirs, const float* __restrict__ inten,
                 const float* __restrict__ temp, int64_t n, int per, int n0, int bl, int bins,
                 unsigned long long* __restrict__ acc, int* __restrict__ bad,
                 int* __restrict__ count) {
  __shared__ int hist[kMaxBins];
  __shared__ unsigned long long wsum[kSortThreads / 64];
  if (count)
    for (int b = threadIdx.x; b < bins; b += kSortThreads) hist[b] = 0;
  __syncthreads();
  const int64_t first = (int64_t)blockIdx.x * kSortThreads * per + threadIdx.x;
  uint64_t h = 0;
  bool any_bad = false;
#pragma unroll 4
  for (int q = 0; q < per; ++q) {
    const int64_t s = first + q * kSortThreads;
    if (s >= n) continue;
    h += star_hash<BANDS>(dirs, inten, temp, s);
    if constexpr (BANDS) {
      const float r = inten[3 * s], g = inten[3 * s + 1], b = inten[3 * s + 2];
      any_bad = any_bad || !(r >= 0.0f && g >= 0.0f && b >= 0.0f) || isinf(r) || isinf(g) ||
                isinf(b);
    }
    if (!count) continue;
    const Place p = place_star<BANDS>(dirs, inten, s, n0);
    if (p.lit) atomicAdd(&hist[bin_of(p, n0, bl)], 1);
  }
  if (any_bad && bad) atomicOr(bad, 1);
  for (int o = 32; o > 0; o >>= 1) h += __shfl_xor(h, o);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = h;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    for (int w = 0; w < kSortThreads / 64; ++w) t += wsum[w];
    atomicAdd(acc, t);
  }
  if (count)
    for (int b = threadIdx.x; b < bins; b += kSortThreads)
      if (hist[b]) atomicAdd(&count[b], hist[b]);
}

// start[b] = stars in the bins before b (start[bins] = all); `count` becomes the scatter's
// cursors, the same values.  One workgroup, at most 2 bins a thread.
__global__ void __launch_bounds__(1024)
    k_star_scan(int* __restrict__ count, int* __restrict__ start, int bins) {
  __shared__ int part[1024];
  const int t = threadIdx.x, b = 2 * t;
  const int c0 = b < bins ? count[b] : 0, c1 = b + 1 < bins ? count[b + 1] : 0;
  part[t] = c0 + c1;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int v = t >= o ? part[t - o] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  const int at = part[t] - c0 - c1;
  if (b < bins) start[b] = count[b] = at;
  if (b + 1 < bins) start[b + 1] = count[b + 1] = at + c0;
  if (t == 1023) start[bins] = part[1023];
}

// ---- texels -----------------------------------------------------------------------------------

// (I, T, p_u, p_v) or (R, G, B, p_u, p_v); all zero when nothing lands in the texel
template <bool BANDS>
struct Master {
  static constexpr int kN = BANDS ? 5 : 4;
  float v[kN];
};

template <bool BANDS>
__device__ __forceinline__ Master<BANDS> no_star() {
  Master<BANDS> m;
#pragma unroll
  for (int q = 0; q < Master<BANDS>::kN; ++q) m.v[q] = 0.0f;
  return m;
}

// the level's maximum is taken over this
template <bool BANDS>
__device__ __forceinline__ float brightest(const Master<BANDS>& m) {
  return BANDS ? fmaxf(m.v[0], fmaxf(m.v[1], m.v[2])) : m.v[0];
}

// Quotients by one divisor d > 0: a reciprocal by Newton's iteration, then each quotient
// corrected once by its own remainder, which rounds as the division itself does (Markstein; the
// stored texels are the division's bit for bit).  Divisors that could overflow or vanish on the
// way take the plain division.  An infinite numerator (a temperature can be infinite) has no
// remainder: of_any returns it as it is.
struct Divider {
  double d, r;
  bool plain;
  __device__ __forceinline__ explicit Divider(double x) : d(x) {
    plain = !(x > 0x1p-500 && x < 0x1p500);
    r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    r = fma(fma(-x, r, 1.0), r, r);
  }
  __device__ __forceinline__ float operator()(double n) const {
    if (plain) return (float)(n / d);
    const double q = n * r;
    return (float)fma(fma(-d, q, n), r, q);
  }
  __device__ __forceinline__ float of_any(double n) const {
    return !plain && isinf(n) ? (float)n : (*this)(n);
  }
};

// Running sums of a texel in FP64, in the order the stars or children are added
template <bool BANDS>
struct Sums {
  double s[Master<BANDS>::kN] = {};
  __device__ __forceinline__ void add(const Master<BANDS>& m, double u, double v) {
    if constexpr (BANDS) {
      const double S = (double)m.v[0] + (double)m.v[1] + (double)m.v[2];
      s[0] += m.v[0];
      s[1] += m.v[1];
      s[2] += m.v[2];
      s[3] += S * u;
      s[4] += S * v;
    } else {
      const double I = m.v[0];
      s[0] += I;
      s[1] += I * (double)m.v[1];
      s[2] += I * u;
      s[3] += I * v;
    }
  }
  __device__ __forceinline__ Master<BANDS> texel() const {
    Master<BANDS> m = no_star<BANDS>();
    if constexpr (BANDS) {
      const double S = s[0] + s[1] + s[2];
      if (S > 0.0) {
        const Divider over(S);
        m.v[0] = (float)s[0];
        m.v[1] = (float)s[1];
        m.v[2] = (float)s[2];
        m.v[3] = over(s[3]);
        m.v[4] = over(s[4]);
      }
    } else if (s[0] > 0.0) {
      const Divider over(s[0]);
      m.v[0] = (float)s[0];
      m.v[1] = over.of_any(s[1]);
      m.v[2] = over(s[2]);
      m.v[3] = over(s[3]);
    }
    return m;
  }
};

// value and position of star s
template <bool BANDS>
__device__ __forceinline__ Master<BANDS> star_value(const StarBuild& B, int64_t s,
                                                    const Place& p) {
  Master<BANDS> m;
  if constexpr (BANDS) {
    m.v[0] = B.inten[3 * s];
    m.v[1] = B.inten[3 * s + 1];
    m.v[2] = B.inten[3 * s + 2];
    m.v[3] = p.pu;
    m.v[4] = p.pv;
  } else {
    m.v[0] = B.inten[s];
    m.v[1] = B.temp[s];
    m.v[2] = p.pu;
    m.v[3] = p.pv;
  }
  return m;
}

// Star values in bin order (4 floats a star, or 4 and then, after all of them, 1): the tiles
// read their stars in a row instead of gathering three cache lines for each.
template <bool BANDS>
__device__ __forceinline__ void put_value(const StarBuild& B, int64_t at, const Master<BANDS>& m) {
  B.val[at] = make_float4(m.v[0], m.v[1], m.v[2], m.v[3]);
  if constexpr (BANDS) ((float*)(B.val + B.n))[at] = m.v[4];
}

// value of the star at slot `at` of the bin order
template <bool BANDS>
__device__ __forceinline__ Master<BANDS> value_at(const StarBuild& B, int64_t at) {
  if (!B.val) {
    const int64_t s = B.order[at];
    return star_value<BANDS>(B, s, place_star<BANDS>(B.dirs, B.inten, s, B.n0));
  }
  const float4 v = B.val[at];
  Master<BANDS> m;
  m.v[0] = v.x;
  m.v[1] = v.y;
  m.v[2] = v.z;
  m.v[3] = v.w;
  if constexpr (BANDS) m.v[4] = ((const float*)(B.val + B.n))[at];
  return m;
}

// star indices, texels and values in bin order (any order inside a bin: the merge sorts)
template <bool BANDS>
__global__ void __launch_bounds__(kSortThreads)
    k_star_scatter(StarBuild B, int* __restrict__ cursor) {
  __shared__ int hist[kMaxBins];
  const int64_t first = (int64_t)blockIdx.x * kSortStars + threadIdx.x;
  for (int b = threadIdx.x; b < B.bins; b += kSortThreads) hist[b] = 0;
  __syncthreads();
  int bin[kSortPer], rank[kSortPer];
  uint32_t texel[kSortPer];
  Master<BANDS> m[kSortPer];
#pragma unroll
  for (int q = 0; q < kSortPer; ++q) {
    const int64_t s = first + q * kSortThreads;
    bin[q] = -1;
    if (s >= B.n) continue;
    const Place p = place_star<BANDS>(B.dirs, B.inten, s, B.n0);
    if (!p.lit) continue;
    bin[q] = bin_of(p, B.n0, B.bl);
    texel[q] = bin_texel(p, B.bl);
    m[q] = star_value<BANDS>(B, s, p);
    rank[q] = atomicAdd(&hist[bin[q]], 1);
  }
  __syncthreads();
  for (int b = threadIdx.x; b < B.bins; b += kSortThreads) {
    const int c = hist[b];
    if (c) hist[b] = atomicAdd(&cursor[b], c);
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kSortPer; ++q) {
    if (bin[q] < 0) continue;
    const int at = hist[bin[q]] + rank[q];
    B.order[at] = (int)(first + q * kSortThreads);
    if (B.where) B.where[at] = texel[q];
    if (B.val) put_value<BANDS>(B, at, m[q]);
  }
}

// parent texel from children (0,0), (1,0), (0,1), (1,1)
template <bool BANDS, class Child>
__device__ __forceinline__ Master<BANDS> parent_texel(Child child) {
  constexpr int P = Master<BANDS>::kN - 2;  // p_u, p_v
  Sums<BANDS> t;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const Master<BANDS> m = child(c);
    bool lit;
    if constexpr (BANDS)
      lit = (double)m.v[0] + (double)m.v[1] + (double)m.v[2] > 0.0;
    else
      lit = m.v[0] > 0.0f;
    if (lit) t.add(m, 0.5 * ((c & 1) + (double)m.v[P]), 0.5 * ((c >> 1) + (double)m.v[P + 1]));
  }
  return t.texel();
}

// per-level scale: power of two so that the largest intensity maps to about 2^14
__device__ __forceinline__ float level_scale(const unsigned* __restrict__ maxbits, int l,
                                             int fp16) {
  if (!fp16) return 1.0f;
  const float mx = __uint_as_float(maxbits[l]);
  return mx > 0.0f ? exp2f(ceilf(log2f(mx)) - 14.0f) : 1.0f;
}

__device__ __forceinline__ Half4 half_texel(const Master<false>& m, float inv) {
  Half4 h;
  h.x = (_Float16)(m.v[0] * inv);
  h.y = (_Float16)(m.v[1] * (1.0f / 1024.0f));
  h.z = (_Float16)m.v[2];
  h.w = (_Float16)m.v[3];
  return h;
}

// stores texel t; true when it is occupied (a stored intensity or band is positive)
template <bool BANDS>
__device__ __forceinline__ bool store_texel(void* out, int64_t t, const Master<BANDS>& m,
                                            float inv, int fp16) {
  if constexpr (BANDS) {
    if (fp16) {
      Half8 h;
      h.v[0] = (_Float16)(m.v[0] * inv);
      h.v[1] = (_Float16)(m.v[1] * inv);
      h.v[2] = (_Float16)(m.v[2] * inv);
      h.v[3] = (_Float16)m.v[3];
      h.v[4] = (_Float16)m.v[4];
      h.v[5] = h.v[6] = h.v[7] = (_Float16)0.0f;
      ((Half8*)out)[t] = h;
      return (float)h.v[0] > 0.0f || (float)h.v[1] > 0.0f || (float)h.v[2] > 0.0f;
    }
    ((float4*)out)[2 * t] = make_float4(m.v[0], m.v[1], m.v[2], m.v[3]);
    ((float4*)out)[2 * t + 1] = make_float4(m.v[4], 0.f, 0.f, 0.f);
    return m.v[0] > 0.0f || m.v[1] > 0.0f || m.v[2] > 0.0f;
  } else {
    if (fp16) {
      const Half4 h = half_texel(m, inv);
      ((Half4*)out)[t] = h;
      return (float)h.x > 0.0f;
    }
    ((float4*)out)[t] = make_float4(m.v[0], m.v[1], m.v[2], m.v[3]);
    return m.v[0] > 0.0f;
  }
}

// two texels of a row, t even: bit 0 and bit 1 of the result say which are occupied
template <bool BANDS>
__device__ __forceinline__ unsigned store_pair(void* out, int64_t t, const Master<BANDS>& a,
                                               const Master<BANDS>& b, float inv, int fp16) {
  if constexpr (!BANDS) {
    if (fp16) {
      const Half4x2 h = {half_texel(a, inv), half_texel(b, inv)};
      *(Half4x2*)((Half4*)out + t) = h;
      return ((float)h.a.x > 0.0f ? 1u : 0u) | ((float)h.b.x > 0.0f ? 2u : 0u);
    }
  }
  return (store_texel<BANDS>(out, t, a, inv, fp16) ? 1u : 0u) |
         (store_texel<BANDS>(out, t + 1, b, inv, fp16) ? 2u : 0u);
}

// ---- tiles ------------------------------------------------------------------------------------

// Occupancy bits of one level: one bit per texel (stored intensity > 0), each texel row
// padded to whole 32-bit words plus one guard word, so a footprint row of at most 9
// texels is read from two consecutive words of its row that never leave the row's storage.
// Every row is stored paired with the next row of its face (the last row with an empty
// one), the two rows' words interleaved: word wi of the pair starting at row R = face nl + y
// is at 2 (R wpr + wi) for row y and 2 (R wpr + wi) + 1 for row y + 1, so one 16-byte load
// returns two consecutive words of two consecutive rows, from any starting row.
// Bits of row y of `face` at word wi of level `occ`; the whole array is zero before.  `whole`:
// this call holds all of the word's bits, otherwise they are added to what is there.
__device__ __forceinline__ void put_occupancy(uint32_t* occ, int nl, int face, int y, int wi,
                                              uint32_t bits, bool whole) {
  if (!bits) return;
  const int wpr = ((nl + 31) >> 5) + 1;
  const int64_t R = (int64_t)face * nl + y;
  uint32_t* first = occ + 2 * (R * wpr + wi);                // with the next row
  uint32_t* second = occ + 2 * ((R - 1) * wpr + wi) + 1;     // with the row before
  if (whole) {
    *first = bits;
    if (y > 0) *second = bits;
  } else {
    atomicOr(first, bits);
    if (y > 0) atomicOr(second, bits);
  }
}

constexpr int kMaxTileLog = 6, kTileThreads = 512;
constexpr int kMipTexels = 1365;    // levels 1 .. 6 of a 64 x 64 tile
constexpr int kTileMaxima = 8;      // per tile: the maxima of levels 0 .. 6
// Stars of a tile kept in LDS.  While they all fit (10^6 stars on 6 x 2048^2 are 163 per tile),
// levels 0 and 1 are formed from lists: one lane per star merges the texels whose list it
// heads, then one lane per parent that has a child.  Every texel of the tile in turn ran the
// FP64 merge for the few lanes of each wave that had anything (230 us a pass, of issue alone).
constexpr int kStash = 512;
// Tiles with more stars, or with more than kListed a texel (a merge from a list looks through it
// once for each of its stars), sort them first, through memory: counts per texel and their
// prefix sums in LDS, a scatter of the star indices, and each star's rank among the indices of its
// texel, one lane per star.  The second pass over the tiles counts again and finds the order in
// memory.  Then a texel's sum is one walk, in LDS where the values fit.  All kernels for 10^6
// stars, where every texel looked through a list in memory once for each of its stars, and now:
// 6 x 32^2 229 and 0.88 ms, 64^2 19.5 and 0.40; 256^2 593 and 195 us, 512^2 235 and 175, 1024^2
// 239 and 232; on 2048^2 with half of the stars in a cluster of 0.02 rad 46 and 3.1 ms (one CU's
// work, almost all of it); 10^7 stars on 4096^2, where the denser third of the tiles just passes
// kStash, 2.45 and 2.55 ms.
constexpr int kListed = 8;

// PACK: write the tile's stored texels and occupancy bits; otherwise only its levels' maxima
// and its topmost texel (level tl) for the tail.  LDS fits three workgroups a CU (two with bands).
template <bool BANDS, bool PACK>
__global__ void __launch_bounds__(kTileThreads, BANDS ? 4 : 6) k_star_tiles(StarBuild B) {
  using M = Master<BANDS>;
  constexpr int P = M::kN - 2;
  __shared__ int head[1 << (2 * kMaxTileLog)];
  __shared__ M mip[kMipTexels];
  // kStash stars with their indices, links and texels, and their parents; or, when the tile's stars
  // are sorted, the values of as many as fit
  constexpr int kEach = sizeof(M) + 2 * sizeof(int) + 2 * sizeof(short);
  constexpr int kStaged = kStash * kEach / sizeof(M);
  __shared__ __align__(16) char stars[kStash * kEach];
  M* const stash = (M*)stars;
  int* const stash_id = (int*)(stash + kStash);
  int* const stash_next = stash_id + kStash;
  short* const stash_at = (short*)(stash_next + kStash);
  short* const parents = stash_at + kStash;
  __shared__ unsigned seen[32];           // parents already listed
  __shared__ int own, listed;             // stars of this tile, parents with a child
  __shared__ int part[kTileThreads / 64];
  __shared__ unsigned word[2 * 64 + 64];  // PACK: occupancy words of levels 0 .. 6
  __shared__ unsigned top[kTileMaxima];
  const int t = threadIdx.x, tl = B.tl, T = 1 << tl, n0 = B.n0;
  const int lnt = B.levels - 1 - tl, nt = 1 << lnt;  // tiles of a face edge
  if (PACK && (int)blockIdx.x >= B.tiles) {  // the tail's levels, one thread per texel
    const int64_t q = (int64_t)(blockIdx.x - B.tiles) * kTileThreads + t;
    const int64_t k = q + (B.off[tl + 1] - B.off[tl]);  // in B.tail
    if (q >= B.tail_texels) return;
    int l = tl + 1;
    while (l + 1 < B.levels && k >= (int64_t)(B.off[l + 1] - B.off[tl])) ++l;
    const int nl = n0 >> l, ll = B.levels - 1 - l;
    const int e = (int)(k - (B.off[l] - B.off[tl]));
    const int x = e & (nl - 1), y = (e >> ll) & (nl - 1), face = e >> (2 * ll);
    const M m = ((const M*)B.tail)[k];
    if (store_texel<BANDS>(B.out, (int64_t)B.off[l] + e, m,
                           1.0f / level_scale(B.maxbits, l, B.fp16), B.fp16))
      put_occupancy(B.occ + B.ooff[l], nl, face, y, x >> 5, 1u << (x & 31), false);
    return;
  }
  const int tile = blockIdx.x, face = tile >> (2 * lnt);
  const int ty = (tile >> lnt) & (nt - 1), tx = tile & (nt - 1);
  // the tile's bin, and the tile's first texel inside it
  const int bl = B.bl, nb = n0 >> bl, sub = bl - tl;
  const int bin = (face * nb + (ty >> sub)) * nb + (tx >> sub);
  const int base = B.start[bin], cnt = B.start[bin + 1] - base;
  const int bx = (tx & ((1 << sub) - 1)) << tl, by = (ty & ((1 << sub) - 1)) << tl;
  if (PACK) {
    if (tile == 0 && t < B.levels) B.scale[t] = level_scale(B.maxbits, t, B.fp16);
  }
  for (int q = t; q < T * T; q += kTileThreads) head[q] = -1;
  if (PACK)
    for (int q = t; q < 192; q += kTileThreads) word[q] = 0u;
  else if (t < kTileMaxima)
    top[t] = 0u;
  for (int q = t; q < T * T / 4; q += kTileThreads) mip[q] = no_star<BANDS>();
  if (t < 32) seen[t] = 0u;
  if (t == 0) own = listed = 0;
  __syncthreads();
  // calls f(slot in the bin, texel of this tile) for the tile's stars, others(star's tile) for the
  // bin's other stars
  constexpr int kScan = 4;  // loads in flight: a bin holds several tiles' stars
  const auto scan_bin = [&](auto f, auto others) {
    for (int q0 = t; q0 < cnt; q0 += kScan * kTileThreads) {
      uint32_t w[kScan];
#pragma unroll
      for (int k = 0; k < kScan; ++k) {
        const int q = base + min(q0 + k * kTileThreads, cnt - 1);
        w[k] = B.where ? B.where[q]
                       : bin_texel(place_star<BANDS>(B.dirs, B.inten, B.order[q], n0), bl);
      }
#pragma unroll
      for (int k = 0; k < kScan; ++k) {
        const int q = q0 + k * kTileThreads;
        const int x = (int)(w[k] & 0xffffu), y = (int)(w[k] >> 16), lx = x - bx, ly = y - by;
        if (q >= cnt) continue;
        if ((unsigned)lx < (unsigned)T && (unsigned)ly < (unsigned)T)
          f(q, ly * T + lx);
        else
          others(((y >> tl) << sub) + (x >> tl));
      }
    }
  };
  const int most = min(kStash, kListed * T * T);  // more stars are sorted
  if (sub == 0 && cnt > most) {  // a bin of one tile
    if (t == 0) own = cnt;
  } else {
    // pick the tile's stars from the bin and list the first kStash per texel
    scan_bin(
        [&](int q, int at) {
          const int i = atomicAdd(&own, 1);
          if (i >= kStash) return;
          stash[i] = value_at<BANDS>(B, base + q);
          stash_id[i] = B.order[base + q];
          stash_at[i] = (short)at;
          stash_next[i] = atomicExch(&head[at], i);
        },
        [](int) {});
  }
  __syncthreads();
  if (own == 0) {  // uniform
    const M zero = no_star<BANDS>();
    if (PACK) {
      for (int l = 0; l <= tl; ++l) {
        const int s = T >> l, nl = n0 >> l;
        const int64_t at = (int64_t)B.off[l] + ((int64_t)face * nl + ty * s) * nl + tx * s;
        if (s > 1) {
          for (int q = t; q < s * s / 2; q += kTileThreads)
            store_pair<BANDS>(B.out,
                              at + (int64_t)(q >> (tl - l - 1)) * nl + 2 * (q & (s / 2 - 1)),
                              zero, zero, 1.0f, B.fp16);
        } else if (t == 0) {
          store_texel<BANDS>(B.out, at, zero, 1.0f, B.fp16);
        }
      }
    } else {
      if (t < kTileMaxima) B.tilemax[(size_t)tile * kTileMaxima + t] = 0.0f;
      if (t == 0) ((M*)B.tail)[tile] = zero;
    }
    return;
  }
  const int mine = own;
  // Sorts the tile's stars; returns where they are.
  const auto sort_tile = [&] {
    __syncthreads();
    for (int q = t; q < T * T; q += kTileThreads) head[q] = 0;
    if (t < kTileThreads / 64) part[t] = 0;
    __syncthreads();
    // stars per texel, and the stars of the bin's tiles before this one
    const int number = ((ty & ((1 << sub) - 1)) << sub) + (tx & ((1 << sub) - 1));
    int before = 0;
    scan_bin([&](int, int at) { atomicAdd(&head[at], 1); },
             [&](int tile) { before += tile < number ? 1 : 0; });
    if (before) atomicAdd(&part[0], before);
    __syncthreads();
    const int first = base + part[0];
    __syncthreads();
    // prefix sums over runs of texels: starts (ends where the order is known already)
    const int per = max(1, T * T / kTileThreads), k0 = t * per;
    int sum = 0;
    for (int k = 0; k < per; ++k)
      if (k0 + k < T * T) sum += head[k0 + k];
    int upto = sum;
    for (int o = 1; o < 64; o <<= 1) {
      const int v = __shfl_up(upto, o);
      if ((t & 63) >= o) upto += v;
    }
    if ((t & 63) == 63) part[t >> 6] = upto;
    __syncthreads();
    for (int w = 0; w < t >> 6; ++w) upto += part[w];
    int at = upto - sum;
    for (int k = 0; k < per; ++k)
      if (k0 + k < T * T) {
        const int c = head[k0 + k];
        head[k0 + k] = PACK ? at + c : at;
        at += c;
      }
    __syncthreads();
    int* sorted = B.sorted + first;
    if (PACK) return sorted;
    int* ids = B.list + first;
    int* slots = B.val ? B.slots + first : nullptr;
    scan_bin(
        [&](int q, int at) {
          const int p = atomicAdd(&head[at], 1);
          ids[p] = B.order[base + q];
          if (slots) slots[p] = q;
        },
        [](int) {});
    __syncthreads();
    for (int p = t; p < mine; p += kTileThreads) {
      const int id = ids[p];
      int lo = 0, hi = T * T - 1;  // the first texel that ends past p
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (head[mid] > p)
          hi = mid;
        else
          lo = mid + 1;
      }
      const int a = lo ? head[lo - 1] : 0, b = head[lo];
      int rank = 0;
#pragma unroll 8
      for (int j = a; j < b; ++j) rank += ids[j] < id ? 1 : 0;
      sorted[a + rank] = slots ? slots[p] : id;
    }
    __syncthreads();
    return sorted;
  };
  // level-0 texel from its list: its stars in increasing star index
  const auto merge = [&](int h) {
    if (h < 0) return no_star<BANDS>();
    Sums<BANDS> sum;
    int last = -1;
    for (;;) {
      int best = 0x7fffffff, at = -1;
      for (int e = h; e >= 0; e = stash_next[e]) {
        const int id = stash_id[e];
        if (id > last && id < best) {
          best = id;
          at = e;
        }
      }
      if (at < 0) break;
      const M m = stash[at];
      sum.add(m, (double)m.v[P], (double)m.v[P + 1]);
      last = best;
    }
    return sum.texel();
  };
  const bool dense = mine > most;
  const int* sorted = nullptr;
  const auto star = [&](int e) {
    if (B.val) return value_at<BANDS>(B, base + e);
    return star_value<BANDS>(B, e, place_star<BANDS>(B.dirs, B.inten, e, n0));
  };
  const bool staged = dense && mine <= kStaged;
  if (dense) {
    sorted = sort_tile();
    if (staged) {
      for (int p = t; p < mine; p += kTileThreads) stash[p] = star(sorted[p]);
      __syncthreads();
    }
  }
  // level-0 texel from the sorted stars
  const auto merge_sorted = [&](int at) {
    constexpr int kAhead = 4;  // stars whose values are in flight
    Sums<BANDS> sum;
    int j = at ? head[at - 1] : 0;
    const int end = head[at];
    if (staged) {
      for (; j < end; ++j) {
        const M m = stash[j];
        sum.add(m, (double)m.v[P], (double)m.v[P + 1]);
      }
      return sum.texel();
    }
    for (; j + kAhead <= end; j += kAhead) {
      M m[kAhead];
#pragma unroll
      for (int k = 0; k < kAhead; ++k) m[k] = star(sorted[j + k]);
#pragma unroll
      for (int k = 0; k < kAhead; ++k) sum.add(m[k], (double)m[k].v[P], (double)m[k].v[P + 1]);
    }
    for (; j < end; ++j) {
      const M m = star(sorted[j]);
      sum.add(m, (double)m.v[P], (double)m.v[P + 1]);
    }
    return sum.texel();
  };
  const auto texel_at = [&](int l, int lx, int ly) {
    const int nl = n0 >> l, s = T >> l;
    return (int64_t)B.off[l] + ((int64_t)face * nl + ty * s + ly) * nl + tx * s + lx;
  };
  // first occupancy word of level l in `word`: T >> l rows of max(1, (T >> l) / 32) words
  const auto word_base = [&](int l) {
    int w = 0;
    for (int k = 0; k < l; ++k) w += (T >> k) * max(1, (T >> k) >> 5);
    return w;
  };
  // stores texels (x, y), (x + 1, y) of level l, x even, and their occupancy bits
  const auto put_pair = [&](int l, int wb, int x, int y, const M& c0, const M& c1, float inv) {
    const unsigned o = store_pair<BANDS>(B.out, texel_at(l, x, y), c0, c1, inv, B.fp16);
    if (o) atomicOr(&word[wb + y * max(1, (T >> l) >> 5) + (x >> 5)], o << (x & 31));
  };
  if (tl == 0) {  // a 1 x 1 face: its texel is also the topmost
    if (t == 0) {
      const M m = dense ? merge_sorted(0) : merge(head[0]);
      if (PACK) {
        if (store_texel<BANDS>(B.out, texel_at(0, 0, 0), m,
                               1.0f / level_scale(B.maxbits, 0, B.fp16), B.fp16))
          put_occupancy(B.occ + B.ooff[0], n0, face, 0, 0, 1u, false);
      } else {
        B.tilemax[(size_t)tile * kTileMaxima] = brightest(m);
        ((M*)B.tail)[tile] = m;
      }
    }
    return;
  }
  // levels 0 and 1
  float max0 = 0.0f, max1 = 0.0f;
  const int half = T >> 1;
  const float inv0 = PACK ? 1.0f / level_scale(B.maxbits, 0, B.fp16) : 1.0f;
  if (!dense) {
    for (int i = t; i < mine; i += kTileThreads) {
      const int at = stash_at[i];
      if (head[at] != i) continue;
      const M m = merge(i);  // the list's other stars are read here only
      stash[i] = m;
      max0 = fmaxf(max0, brightest(m));
      const int q = (at >> (tl + 1)) * half + ((at & (T - 1)) >> 1);
      const unsigned bit = 1u << (q & 31);
      if (!(atomicOr(&seen[q >> 5], bit) & bit)) parents[atomicAdd(&listed, 1)] = (short)q;
    }
    __syncthreads();
    const auto texel0 = [&](int h) { return h < 0 ? no_star<BANDS>() : stash[h]; };
    for (int a = t; a < listed; a += kTileThreads) {
      const int q = parents[a], at = 2 * (q >> (tl - 1)) * T + 2 * (q & (half - 1));
      const M m = parent_texel<BANDS>(
          [&](int k) { return texel0(head[at + (k >> 1) * T + (k & 1)]); });
      mip[q] = m;
      max1 = fmaxf(max1, brightest(m));
    }
    if (PACK) {
      for (int q = t; q < T * half; q += kTileThreads) {
        const int x = 2 * (q & (half - 1)), y = q >> (tl - 1);
        const int2 h = *(const int2*)&head[y * T + x];
        put_pair(0, 0, x, y, texel0(h.x), texel0(h.y), inv0);
      }
    }
  } else if (4 * mine < T * T) {
    // few stars a texel: a lane per parent
    for (int p = t; p < half * half; p += kTileThreads) {
      const int x = 2 * (p & (half - 1)), y = 2 * (p >> (tl - 1));
      M c[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        c[k] = merge_sorted((y + (k >> 1)) * T + x + (k & 1));
        max0 = fmaxf(max0, brightest(c[k]));
      }
      const M m = parent_texel<BANDS>([&](int k) { return c[k]; });
      mip[p] = m;
      max1 = fmaxf(max1, brightest(m));
      if (PACK) {
        put_pair(0, 0, x, y, c[0], c[1], inv0);
        put_pair(0, 0, x, y + 1, c[2], c[3], inv0);
      }
    }
  } else {
    // a lane per texel, the four children of a parent side by side
    for (int q = t; q < T * T; q += kTileThreads) {
      const int p = q >> 2, x = 2 * (p & (half - 1)) + (q & 1);
      const int y = 2 * (p >> (tl - 1)) + ((q >> 1) & 1);
      const M own_texel = merge_sorted(y * T + x);
      max0 = fmaxf(max0, brightest(own_texel));
      const auto child = [&](int k) {
        M m;
#pragma unroll
        for (int i = 0; i < M::kN; ++i) m.v[i] = __shfl(own_texel.v[i], (t & 60) + k);
        return m;
      };
      const M c1 = child(1), c3 = child(3);
      const M m = parent_texel<BANDS>(
          [&](int k) { return k == 1 ? c1 : (k == 3 ? c3 : child(k)); });
      if ((q & 3) == 0) {
        mip[p] = m;
        max1 = fmaxf(max1, brightest(m));
      }
      if (PACK && !(q & 1)) put_pair(0, 0, x, y, own_texel, (q & 2) ? c3 : c1, inv0);
    }
  }
  if (!PACK) {
    for (int o = 32; o > 0; o >>= 1) {
      max0 = fmaxf(max0, __shfl_xor(max0, o));
      max1 = fmaxf(max1, __shfl_xor(max1, o));
    }
    if ((t & 63) == 0) {
      atomicMax(&top[0], __float_as_uint(max0));  // values >= 0: their bits order as they do
      atomicMax(&top[1], __float_as_uint(max1));
    }
  }
  __syncthreads();
  if (PACK) {
    const float inv1 = 1.0f / level_scale(B.maxbits, 1, B.fp16);
    const int wb = word_base(1);
    if (half > 1) {
      for (int q = t; q < half * half / 2; q += kTileThreads)
        put_pair(1, wb, 2 * q & (half - 1), 2 * q >> (tl - 1), mip[2 * q], mip[2 * q + 1], inv1);
    } else if (t == 0 && store_texel<BANDS>(B.out, texel_at(1, 0, 0), mip[0], inv1, B.fp16)) {
      word[wb] = 1u;
    }
  }
  // levels 2 .. tl
  const M* prev = mip;
  for (int l = 2; l <= tl; ++l) {
    const int s = T >> l, ps = 2 * s;
    M* cur = const_cast<M*>(prev) + ps * ps;
    const float inv = PACK ? 1.0f / level_scale(B.maxbits, l, B.fp16) : 1.0f;
    const int wb = PACK ? word_base(l) : 0;
    for (int q = t; q < s * s; q += kTileThreads) {
      const int x = q & (s - 1), y = q >> (tl - l);
      const M m = parent_texel<BANDS>(
          [&](int k) { return prev[(2 * y + (k >> 1)) * ps + 2 * x + (k & 1)]; });
      cur[q] = m;
      if (PACK) {
        if (store_texel<BANDS>(B.out, texel_at(l, x, y), m, inv, B.fp16))
          atomicOr(&word[wb + y], 1u << x);  // s <= 16: one word per row
      } else {
        atomicMax(&top[l], __float_as_uint(brightest(m)));
      }
    }
    __syncthreads();
    prev = cur;
  }
  if (!PACK) {
    if (t < kTileMaxima) B.tilemax[(size_t)tile * kTileMaxima + t] = __uint_as_float(top[t]);
    if (t == 0) ((M*)B.tail)[tile] = *prev;
    return;
  }
  // occupancy words: whole ones of levels at least 32 texels wide, else shared with neighbours
  for (int l = 0, wb = 0; l <= tl; ++l) {
    const int s = T >> l, wp = max(1, s >> 5);
    for (int q = t; q < s * wp; q += kTileThreads) {
      const int y = wp == 2 ? q >> 1 : q, gx = tx * s + (wp == 2 ? 32 * (q & 1) : 0);
      put_occupancy(B.occ + B.ooff[l], n0 >> l, face, ty * s + y, gx >> 5,
                    word[wb + q] << (gx & 31), s >= 32);
    }
    wb += s * wp;
  }
}

// The levels above the tiles' topmost, one workgroup per face, and every level's maximum.
template <bool BANDS>
__global__ void __launch_bounds__(kTileThreads) k_star_tail(StarBuild B) {
  using M = Master<BANDS>;
  __shared__ unsigned top[16];
  const int t = threadIdx.x, face = blockIdx.x, tl = B.tl, nt = B.n0 >> tl;
  if (t < 16) top[t] = 0u;
  if (face == 0 && t < B.levels) {
    B.level_off_dev[t] = B.off[t];
    B.occ_off_dev[t] = B.ooff[t];
  }
  __syncthreads();
  float mx[kTileMaxima] = {};
  for (int q = t; q < nt * nt; q += kTileThreads) {
    const float4* r = (const float4*)(B.tilemax + (size_t)(face * nt * nt + q) * kTileMaxima);
    const float4 a = r[0], b = r[1];
    mx[0] = fmaxf(mx[0], a.x);
    mx[1] = fmaxf(mx[1], a.y);
    mx[2] = fmaxf(mx[2], a.z);
    mx[3] = fmaxf(mx[3], a.w);
    mx[4] = fmaxf(mx[4], b.x);
    mx[5] = fmaxf(mx[5], b.y);
    mx[6] = fmaxf(mx[6], b.z);
  }
#pragma unroll
  for (int l = 0; l < 7; ++l) {
    for (int o = 32; o > 0; o >>= 1) mx[l] = fmaxf(mx[l], __shfl_xor(mx[l], o));
    if (l <= tl && (t & 63) == 0) atomicMax(&top[l], __float_as_uint(mx[l]));
  }
  M* tail = (M*)B.tail;
  for (int l = tl + 1; l < B.levels; ++l) {
    const int nl = B.n0 >> l, np = 2 * nl;
    const M* prev = tail + (B.off[l - 1] - B.off[tl]) + (int64_t)face * np * np;
    M* cur = tail + (B.off[l] - B.off[tl]) + (int64_t)face * nl * nl;
    float v = 0.0f;
    for (int q = t; q < nl * nl; q += kTileThreads) {
      const int x = q & (nl - 1), y = q >> (B.levels - 1 - l);
      const M m = parent_texel<BANDS>(
          [&](int k) { return prev[(2 * y + (k >> 1)) * np + 2 * x + (k & 1)]; });
      cur[q] = m;
      v = fmaxf(v, brightest(m));
    }
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
    if ((t & 63) == 0) atomicMax(&top[l], __float_as_uint(v));
    __syncthreads();
  }
  __syncthreads();
  if (t < B.levels && top[t]) atomicMax(B.maxbits + t, top[t]);
}

// ---- host-side launchers ------------------------------------------------------------------------

// Tiles of 64 texels an edge from 1024 texels a face, else 32: a map of few tiles needs the
// smaller ones to spread over the chip (6 x 256^2: 384 workgroups instead of 96).  Smaller still
// while they hold more than four times kStash on average, which too few workgroups would sort,
// down to bins of four tiles, each of which looks through its bin.  Splitting further costs more
// rounds of workgroups than it saves: past 2 kStash, 3 10^6 stars on 6 x 1024^2 571 against 433
// us; past kStash / 2, 10^6 on 256^2 349 against 226.
int star_tile_log(int n0, int64_t n) {
  int lg = 0;
  while ((2 << lg) <= n0) ++lg;
  int tl = n0 >= 1024 ? kMaxTileLog : std::min(lg, kMaxTileLog - 1);
  const auto tiles = [&](int l) { return (int64_t)6 * (n0 >> l) * (n0 >> l); };
  while (tl > 0 && n > 4 * kStash * tiles(tl) && tiles(tl - 1) <= 4 * kMaxBins) --tl;
  return tl;
}

size_t star_tail_texel_bytes(int bands) {
  return bands ? sizeof(Master<true>) : sizeof(Master<false>);
}
size_t star_tile_max_bytes() { return kTileMaxima * sizeof(float); }

// Bins: one tile each while there are at most kMaxBins of them, else squares of tiles.
int star_bin_log(int n0, int64_t n) {
  int bl = star_tile_log(n0, n);
  while (6 * (n0 >> bl) * (n0 >> bl) > kMaxBins) ++bl;
  return bl;
}

// hash (*acc), *bad and the stars per bin (`bad`, `count`: or null); all zero before
hipError_t launch_star_count(const float* dirs, const float* inten, const float* temp, int64_t n,
                             int n0, int bands, unsigned long long* acc, int* bad, int* count,
                             hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int bl = star_bin_log(n0, n), nb = n0 >> bl;
  const int per = (int)std::min<int64_t>(n / (256 * kSortThreads) + 1, kSortPer);
  const dim3 grid(blocks_for(n, kSortThreads * per));
  if (bands)
    hipLaunchKernelGGL(k_star_count<true>, grid, dim3(kSortThreads), 0, s, dirs, inten, temp, n,
                       per, n0, bl, 6 * nb * nb, acc, bad, count);
  else
    hipLaunchKernelGGL(k_star_count<false>, grid, dim3(kSortThreads), 0, s, dirs, inten, temp, n,
                       per, n0, bl, 6 * nb * nb, acc, bad, count);
  return hipGetLastError();
}

template <bool BANDS>
static hipError_t build(const StarBuild& B, int* count, int64_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_fill_int, dim3(blocks_for(B.occ_words, 256)), dim3(256), 0, s,
                     (int*)B.occ, B.occ_words, 0);
  hipLaunchKernelGGL(k_star_scan, dim3(1), dim3(1024), 0, s, count, B.start, B.bins);
  if (n > 0)
    hipLaunchKernelGGL(k_star_scatter<BANDS>, dim3(blocks_for(n, kSortStars)), dim3(kSortThreads),
                       0, s, B, count);
  hipLaunchKernelGGL((k_star_tiles<BANDS, false>), dim3(B.tiles), dim3(kTileThreads), 0, s, B);
  hipLaunchKernelGGL(k_star_tail<BANDS>, dim3(6), dim3(kTileThreads), 0, s, B);
  hipLaunchKernelGGL((k_star_tiles<BANDS, true>),
                     dim3(B.tiles + blocks_for(B.tail_texels, kTileThreads)), dim3(kTileThreads),
                     0, s, B);
  return hipGetLastError();
}

// Every level, its scale and its occupancy bits, from the bin counts of launch_star_count.
hipError_t launch_star_build(const StarBuild& B, int* count, int64_t n, int bands,
                             hipStream_t s) {
  return bands ? build<true>(B, count, n, s) : build<false>(B, count, n, s);
}

// ---- reading a map back ---------------------------------------------------------------------

__global__ void k_star_unpack(const void* __restrict__ in, int64_t count, float scale, int fp16,
                              float4* __restrict__ out) {
  int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= count) return;
  if (fp16) {
    Half4 h = ((const Half4*)in)[t];
    out[t] = make_float4((float)h.x * scale, (float)h.y * 1024.0f, (float)h.z, (float)h.w);
  } else {
    out[t] = ((const float4*)in)[t];
  }
}

// stored texels back to (R, G, B, p_u) (p_v, 0, 0, 0) records in the caller's units
__global__ void k_star_unpack_bands(const void* __restrict__ in, int64_t count, float scale,
                                    int fp16, float4* __restrict__ out) {
  int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (t >= count) return;
  if (fp16) {
    const Half8 h = ((const Half8*)in)[t];
    out[2 * t] = make_float4((float)h.v[0] * scale, (float)h.v[1] * scale,
                             (float)h.v[2] * scale, (float)h.v[3]);
    out[2 * t + 1] = make_float4((float)h.v[4], 0.f, 0.f, 0.f);
  } else {
    out[2 * t] = ((const float4*)in)[2 * t];
    out[2 * t + 1] = ((const float4*)in)[2 * t + 1];
  }
}

hipError_t launch_star_unpack_bands(const void* in, int64_t count, float scale, int fp16,
                                    float4* out, hipStream_t s) {
  hipLaunchKernelGGL(k_star_unpack_bands, dim3(blocks_for(count, 256)), dim3(256), 0, s, in,
                     count, scale, fp16, out);
  return hipGetLastError();
}

hipError_t launch_fill_int(int* p, int64_t n, int v, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_int, dim3(blocks_for(n, 256)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_star_unpack(const void* in, int64_t count, float scale, int fp16, float4* out,
                              hipStream_t s) {
  hipLaunchKernelGGL(k_star_unpack, dim3(blocks_for(count, 256)), dim3(256), 0, s, in, count,
                     scale, fp16, out);
  return hipGetLastError();
}

}  // namespace bh
