// Per-pixel beam tracer (Sections 3.2-3.4) for gfx950.
//
// Thread layout: one wavefront covers an 8x8 pixel block; lane l handles quad l >> 2 of
// the block (4x4 quads) and pixel (l & 1, (l >> 1) & 1) inside the quad, so the 2x2 quad
// partners needed for screen-space derivatives are lanes l^1 (same row) and l^2 (same
// column) and are read with DPP quad permutations.  A workgroup tile is TW x TH pixels made of
// 8x8 blocks; each wave walks PPT blocks.  Pixels outside the image are computed (their
// rays are valid) but not stored, so every quad is complete.
//
// Steps per pixel:
//   beam init   camera direction n_C -> aberration into the static frame (eq. d) ->
//               coordinate direction d (e_r has length sqrt(1-u), eq. staticbasis) ->
//               ray plane e_x', e_y', e_z', angle delta, disc angle alpha (eqs. raybasis,
//               alpha)
//   TraceRay    Algorithm 1 with bilinear fetches of D(e,u), D(e,u_a) and U(e,phi)
//   disc        T' from the temperature law, Doppler factor g(k,l)/g(k',l') with the
//               Keplerian k' (eq. k_prime), band radiances of a blackbody at D T'
//               (Section 3.4.2), front-to-back composite
//   stars       fine quad differences of d' and of q, face Jacobian, mip
//               level such that the extended footprint spans at most 9x9 texels,
//               tent-weighted gather f(w) f(h), lensing factor Omega/Omega', one Doppler
//               shift per pixel.
#include <type_traits>

#include "bh_dev.h"

#include "bh_probes.h"

namespace bh {

struct __align__(8) Half4r {
  _Float16 x, y, z, w;
};
struct __align__(16) Half8r {
  _Float16 v[8];
};
struct __align__(8) OccPair {  // two words of two consecutive occupancy rows (stars.hip)
  uint32_t a0, a1, b0, b1;      // row r word k, row r + 1 word k, row r word k + 1, row r + 1 word k + 1
};

// Stored texels are (I, T, p_u, p_v); the FP16 format keeps I / scale_L and T / 1024, and
// the caller applies both factors once to the footprint sums.  Band-colour maps store
// (R, G, B, p_u, p_v, 0, 0, 0), FP16 bands divided by scale_L.
enum { kTexIT16 = 0, kTexIT32 = 1, kTexBand16 = 2, kTexBand32 = 3 };

// Footprint of one pixel on one star-map level: texel columns x0 .. x0 + 8 and rows
// y0 .. y0 + ny at most, read from the occupancy bits into one 81-bit mask (bit 9 r + c for
// row y0 + r, column x0 + c; rows 0-6 in `lo`, rows 7-8 in `hi`), then one pass over the set
// bits.  A single loop over occupied texels keeps the lanes of a wave in step far better
// than a loop per row.  Adds the tent-weighted sums of I and I T, in stored units, to A, B
// (FMT kTexIT16, kTexIT32), or of R, G, B to A, B, C (kTexBand16, kTexBand32).
struct Footprint {
  uint32_t texel0;       // texel index of (x0, y0)
  const uint32_t* occ;   // occupancy word of (x0, y0) in the row pair starting at y0
  int nL, wpr4, sh, ny;  // wpr4: occupancy words from one row pair to the pair two rows down
  uint32_t span;         // bit mask of the footprint's columns, shifted to bit 0
  // screen-space coordinates (w, h) of a star at (c + p_u, r + p_v) texels from the
  // footprint's corner: w = W0 + Wc (c + p_u) + Wr (r + p_v), h = H0 + Hc (..) + Hr (..)
  float W0, Wc, Wr, H0, Hc, Hr;
  float one;             // 1, not known to the compiler: p_u + c stays one mixed-precision FMA
};

// Buffers of the measurement variant (COUNT): one bit per star-map texel the footprints
// visit, and the total of the bytes every pixel requests through the caches (table and band
// table fetches, occupancy words, texels, level records, image and AOV stores).
struct CountBufs {
  uint32_t* touched;
  unsigned long long* l2_bytes;
};

template <int FMT, bool COUNT, bool PAIR = true>
__device__ __forceinline__ void gather(const void* tex, const Footprint& F, const CountBufs* cnt,
                                       uint32_t& req, float& A, float& B, float& C) {
  uint32_t w0 = 0, w1 = 0, hi = 0;  // lo = w0 + 2^32 w1
  // Every row's two occupancy words are loaded before any is used, so a lane waits once for
  // its rows instead of once per row.  Rows come in pairs (r, r + 1), one 16-byte load each
  // (the occupancy layout of stars.hip); pairs past the footprint load nothing, and the
  // second row of the last pair is dropped when it lies past the footprint.
  uint32_t ra[10], rb[10];
#pragma unroll
  for (int p = 0; p < 5; ++p) {
    ra[2 * p] = rb[2 * p] = ra[2 * p + 1] = rb[2 * p + 1] = 0u;
    if (2 * p <= F.ny) {
      const OccPair q = *(const OccPair*)(F.occ + (uint32_t)p * (uint32_t)F.wpr4);
      ra[2 * p] = q.a0;
      ra[2 * p + 1] = q.a1;
      rb[2 * p] = q.b0;
      rb[2 * p + 1] = q.b1;
    }
  }
  if (COUNT) req += 16 * (F.ny / 2 + 1);  // one 16-byte load per row pair
#pragma unroll
  for (int r = 0; r < 9; ++r) {
    // the row's 9 columns from bit x0 & 31 of two consecutive words (a funnel shift)
    uint32_t b = __builtin_amdgcn_alignbit(rb[r], ra[r], (uint32_t)F.sh) & F.span;
    if ((r & 1) && r > F.ny) b = 0u;
    if (r < 3) {
      w0 |= b << (9 * r);
    } else if (r == 3) {
      w0 |= b << 27;
      w1 |= b >> 5;
    } else if (r < 7) {
      w1 |= b << (9 * r - 32);
    } else {
      hi |= b << (9 * (r - 7));
    }
  }
  uint64_t lo = (uint64_t)w0 | ((uint64_t)w1 << 32);
  // texels from the footprint's corner: row r, column c lies r nL + c = idx + r (nL - 9)
  // texels on (nL - 9 >= -8: a signed 24-bit product)
  const Half4r* tex16 = (const Half4r*)tex + F.texel0;
  const float4* tex32 = (const float4*)tex + F.texel0;
  const Half8r* texb16 = (const Half8r*)tex + F.texel0;
  const float4* texb32 = (const float4*)tex + 2 * (size_t)F.texel0;
  const int nLm9 = F.nL - 9;
  // the texel of mask bit idx (row r, column c lies r nL + c = idx + r (nL - 9) texels from
  // the footprint's corner)
  auto at = [&](int idx) {
    const int r = (idx * 57) >> 9;  // idx / 9 for idx < 81
    return (uint32_t)(__mul24(r, nLm9) + idx);
  };
  struct Tx {  // one stored texel of any format
    Half4r h4;
    Half8r h8;
    float4 f0, f1;
  };
  auto load = [&](uint32_t t) {
    Tx x;
    if constexpr (FMT == kTexIT16) x.h4 = tex16[t];
    if constexpr (FMT == kTexIT32) x.f0 = tex32[t];
    if constexpr (FMT == kTexBand16) x.h8 = texb16[t];
    if constexpr (FMT == kTexBand32) {
      x.f0 = texb32[2 * t];
      x.f1 = texb32[2 * t + 1];
    }
    return x;
  };
  // tent weight f(w) f(h) of the star of texel x at bit idx, 0 unless `use`, then the sums
  auto weigh = [&](const Tx& x, int idx, bool use) {
    const int r = (idx * 57) >> 9, c = idx - 9 * r;
    const float fc = (float)c, fr = (float)r;
    float a, b;
    if constexpr (FMT == kTexIT16) {
      // half operands go straight into mixed-precision multiply-adds
      a = fmaf((float)x.h4.z, F.one, fc);
      b = fmaf((float)x.h4.w, F.one, fr);
    } else if constexpr (FMT == kTexIT32) {
      a = fc + x.f0.z;
      b = fr + x.f0.w;
    } else if constexpr (FMT == kTexBand16) {
      a = fmaf((float)x.h8.v[3], F.one, fc);
      b = fmaf((float)x.h8.v[4], F.one, fr);
    } else {
      a = fc + x.f0.w;
      b = fr + x.f1.x;
    }
    const float w = fmaf(F.Wc, a, fmaf(F.Wr, b, F.W0));
    const float h = fmaf(F.Hc, a, fmaf(F.Hr, b, F.H0));
    float wt = __builtin_amdgcn_fmed3f(1.0f - fabsf(w), 0.0f, 1.0f) *
               __builtin_amdgcn_fmed3f(1.0f - fabsf(h), 0.0f, 1.0f);  // max(1 - |x|, 0)
    wt = use ? wt : 0.0f;
    if constexpr (FMT == kTexIT16) {
      const float wi = fmaf(wt, (float)x.h4.x, 0.0f);
      A += wi;
      B = fmaf(wi, (float)x.h4.y, B);
    } else if constexpr (FMT == kTexIT32) {
      const float wi = wt * x.f0.x;
      A += wi;
      B = fmaf(wi, x.f0.y, B);
    } else if constexpr (FMT == kTexBand16) {
      A = fmaf(wt, (float)x.h8.v[0], A);
      B = fmaf(wt, (float)x.h8.v[1], B);
      C = fmaf(wt, (float)x.h8.v[2], C);
    } else {
      A = fmaf(wt, x.f0.x, A);
      B = fmaf(wt, x.f0.y, B);
      C = fmaf(wt, x.f0.z, C);
    }
  };
  // Two taps per iteration, both texel loads in flight before either is weighed, so a lane
  // waits on its scattered loads half as often.  With one tap left the second repeats the
  // first texel with weight 0 and adds nothing: the sums take the taps in bit order.  Only
  // the bit indices stay live across the loads (row and column are recomputed after).
  auto two_taps = [&](int i0, int i1, bool two) {
    if (COUNT) {
      for (int k = 0; k < 2; ++k) {
        if (k == 1 && !two) break;
        const uint32_t ta = F.texel0 + at(k == 0 ? i0 : i1);
        atomicOr(&cnt->touched[ta >> 5], 1u << (ta & 31));
        req += FMT == kTexIT16 ? 8 : (FMT == kTexBand32 ? 32 : 16);
      }
    }
    const Tx x0 = load(at(i0)), x1 = load(at(i1));
    weigh(x0, i0, true);
    weigh(x1, i1, two);
  };
  if constexpr (PAIR) {
    while (lo) {
      const int i0 = __builtin_ctzll(lo);
      lo &= lo - 1u;
      const bool two = lo != 0;
      const int i1 = two ? __builtin_ctzll(lo) : i0;
      lo &= lo - 1u;  // 0 stays 0
      two_taps(i0, i1, two);
    }
    while (hi) {
      const int i0 = 63 + __builtin_ctz(hi);
      hi &= hi - 1u;
      const bool two = hi != 0;
      const int i1 = two ? 63 + __builtin_ctz(hi) : i0;
      hi &= hi - 1u;
      two_taps(i0, i1, two);
    }
  } else {
    // band texels are twice as wide: one tap per iteration keeps the band kernels' register
    // budget (two in flight spilled 19 registers at 8 waves per SIMD, and gave nothing at 5: the
    // 1080p any-colour frame 109.3 us with, 108.7 without), and the kernel for band star maps
    // without area maps takes (I, T) maps one tap at a time too (PAIR)
    auto one_tap = [&](int i) {
      if (COUNT) {
        const uint32_t ta = F.texel0 + at(i);
        atomicOr(&cnt->touched[ta >> 5], 1u << (ta & 31));
        req += FMT == kTexBand32 ? 32 : 16;
      }
      weigh(load(at(i)), i, true);
    };
    while (lo) {
      const int i = __builtin_ctzll(lo);
      lo &= lo - 1u;
      one_tap(i);
    }
    while (hi) {
      const int i = 63 + __builtin_ctz(hi);
      hi &= hi - 1u;
      one_tap(i);
    }
  }
}

struct TraceOut {
  float e;             // the beam's invariant e = sqrt(e^2)
  float dprime;        // escape angle (valid if !captured)
  float ucr[2];
  float tret[2];       // retarded times of the crossings (TIMED only)
  int mcr[2];          // crossing k lies at beam-plane angle alpha + mcr[k] pi (TIMED only)
  int ncross;
  unsigned bits;
  uint32_t req;        // bytes the table fetches request (read by the measurement variant only)
};

// singular part of the coordinate time along a ray: t = tau + S(u) + const
__device__ __forceinline__ float time_singular(float u) {
  return __log2f(fdiv(u, 1.0f - u)) * 0.693147180559945309f - fdiv(1.0f, u);
}

// Algorithm 1, TraceRay, in FP32.  Returns crossings in order along the beam.  TIMED also
// returns each crossing's retarded time (the coordinate time the light takes from it to
// the camera): s (t_0 - t) for crossing 0 and 2 t_a - t - t_1 for crossing 1, with
// t = tau + S(u) and tau = (e tau from the time channels) / e.  `hide`: a first crossing hides
// whatever lies behind it, so a second one is not looked for.
template <bool TIMED>
__device__ __forceinline__ TraceOut trace_ray(const TablesDev& T, float u, float delta,
                                             float alpha, float cotd, float u_ic, float u_oc,
                                             bool hide = false) {
  TraceOut o;
  o.ncross = 0;
  o.ucr[0] = o.ucr[1] = 0.0f;
  o.tret[0] = o.tret[1] = 0.0f;
  o.mcr[0] = o.mcr[1] = 0;
  o.bits = 0;
  o.dprime = 0.0f;
  o.req = 0;
  float udot = -u * cotd;
  float e2 = udot * udot + u * u * (1.0f - u);
  float e = fsqrt(e2);
  o.e = e;
  if (e2 < kMu && u > 2.0f / 3.0f) {
    o.bits = BH_CAPTURED_BIT;
    return o;
  }
  const bool in = udot >= 0.0f;  // towards the hole: s = 1, else s = -1
  const float s = in ? 1.0f : -1.0f;
  bool bound = e2 < kMu;
  float ua = bound ? apsis_f(e2) : 0.0f;
  const TablePoint pd = point_D(T, bound, e2, u, ua, udot);
  float Da;
  float Dl = fetch_D(T, T.D, pd, &Da);
  const float phia = bound ? Da + 0.5f * kPi : __builtin_inff();
  o.req += 24;  // a bilinear fetch reads two pairs of adjacent floats, the apsis one
  float ie = 0.0f, t_cam = 0.0f, t_a = 0.0f;
  if (TIMED) {
    ie = fdiv(1.0f, e);
    float ta;
    t_cam = fetch_D(T, T.Dt, pd, &ta) * ie + time_singular(u);
    if (bound) t_a = ta * ie + time_singular(ua);
  }
  float phi = Dl + (in ? kPi - delta : delta) + s * alpha;
  float m0 = floorf(phi * (1.0f / kPi));
  float phi0 = phi - kPi * m0;
  const PointU cu = columns_U(T, e2, e);
  const TablePoint p0 = point_U(T, cu, phi0);
  float u0 = bilinear(T.U, p0, T.u_ne);
  o.req += 16;
  if (phi0 < phia && u_oc <= u0 && u0 <= u_ic && (in ? u0 > u : u0 < u)) {
    o.ucr[0] = u0;
    o.ncross = 1;
    o.bits |= BH_CROSS0_BIT;
    if (TIMED) {
      o.tret[0] = s * (bilinear(T.Ut, p0, T.u_ne) * ie + time_singular(u0) - t_cam);
      o.mcr[0] = (int)m0;
    }
  }
  if (bound && in && !(hide && o.ncross != 0)) {
    phi = 2.0f * phia - phi;
    float m1 = floorf(phi * (1.0f / kPi));
    float phi1 = phi - kPi * m1;
    const TablePoint p1 = point_U(T, cu, phi1);
    float u1 = bilinear(T.U, p1, T.u_ne);
    o.req += 16;
    if (phi1 < phia && u_oc <= u1 && u1 <= u_ic) {
      float t1 = 0.0f;
      if (TIMED)
        t1 = 2.0f * t_a - t_cam - (bilinear(T.Ut, p1, T.u_ne) * ie + time_singular(u1));
      // static indices only: a dynamically indexed array would be placed in LDS
      if (o.ncross == 0) {
        o.ucr[0] = u1;
        o.tret[0] = t1;
        o.mcr[0] = (int)m1;
      } else {
        o.ucr[1] = u1;
        o.tret[1] = t1;
        o.mcr[1] = (int)m1;
      }
      o.ncross += 1;
      o.bits |= BH_CROSS1_BIT;
    }
  }
  if (udot > 0.0f) {
    if (bound) {
      Dl = 2.0f * Da - Dl;
    } else {
      o.bits |= BH_CAPTURED_BIT;
      return o;
    }
  }
  o.dprime = delta + Dl;
  return o;
}

// ---- ray marching in place of TraceRay: the ablation of Section 5 (method M3, Table 1)
// Classic fourth-order Runge-Kutta on (u, w = du/dphi), w' = 3/2 u^2 - u (eq. rayequation),
// with the constant step h = 2 pi / N and at most N steps.  Inside a step u is the cubic
// Hermite interpolant of the two end states; in t = s / h, with the slopes scaled by h,
// p(t) = ((c3 t + c2) t + a) t + p0.  Its first root places the escape (Newton from the
// secant), its value at alpha + m pi a disc crossing.  h < pi (N >= 3): a step passes at
// most one disc-plane angle.  A beam still travelling after N steps is drawn as captured.
__device__ __forceinline__ float march_acc(float u) { return u * fmaf(1.5f, u, -1.0f); }

__device__ __forceinline__ TraceOut march_ray(float u, float alpha, float cotd, float u_ic,
                                              float u_oc, int nsteps, float h) {
  TraceOut o;
  o.ncross = 0;
  o.ucr[0] = o.ucr[1] = 0.0f;
  o.tret[0] = o.tret[1] = 0.0f;
  o.mcr[0] = o.mcr[1] = 0;
  o.bits = 0;
  o.dprime = 0.0f;
  o.req = 0;
  float w = -u * cotd;
  o.e = fsqrt(w * w + u * u * (1.0f - u));
  if (fabsf(cotd) >= 1e6f) {
    // within 1e-6 of the radius: the beam moves along r only (a step in phi cannot follow
    // it); outward it escapes undeflected at delta' = delta ~ 1 / cot(delta), inward it falls
    if (cotd > 0.0f)
      o.dprime = fdiv(1.0f, cotd);
    else
      o.bits = BH_CAPTURED_BIT;
    return o;
  }
  const bool inward = w > 0.0f;  // an apsis (largest u) can lie ahead
  const float hh = 0.5f * h, h6 = h * (1.0f / 6.0f), ih = fdiv(1.0f, h);
  float phid = alpha > 0.0f ? alpha : alpha + kPi;  // next disc-plane angle ahead
  for (int n = 0; n < nsteps; ++n) {
    const float a1 = march_acc(u);
    const float u2 = fmaf(hh, w, u), w2 = fmaf(hh, a1, w), a2 = march_acc(u2);
    const float u3 = fmaf(hh, w2, u), w3 = fmaf(hh, a2, w), a3 = march_acc(u3);
    const float u4 = fmaf(h, w3, u), w4 = fmaf(h, a3, w), a4 = march_acc(u4);
    const float un = fmaf(h6, fmaf(2.0f, w2 + w3, w + w4), u);
    const float wn = fmaf(h6, fmaf(2.0f, a2 + a3, a1 + a4), w);
    const float phi = (float)n * h;
    const bool esc = un < 0.0f;
    const float td = (phid - phi) * ih;
    if (esc || td <= 1.0f) {
      const float A = h * w, B = h * wn;
      const float c3 = 2.0f * (u - un) + A + B, c2 = 3.0f * (un - u) - 2.0f * A - B;
      float tend = 1.0f;
      if (esc) {
        float t = fdiv(u, u - un);
#pragma unroll
        for (int it = 0; it < 3; ++it) {
          float p = fmaf(fmaf(fmaf(c3, t, c2), t, A), t, u);
          float dp = fmaf(fmaf(3.0f * c3, t, 2.0f * c2), t, A);
          t = clampf(t - fdiv(p, dp), 0.0f, 1.0f);
        }
        tend = t;
      }
      if (td <= tend) {
        const float ud = fmaf(fmaf(fmaf(c3, td, c2), td, A), td, u);
        if (ud >= u_oc && ud <= u_ic) {
          const float slope = fmaf(fmaf(3.0f * c3, td, 2.0f * c2), td, A);
          o.bits |= inward && slope < 0.0f ? BH_CROSS1_BIT : BH_CROSS0_BIT;
          if (o.ncross == 0) o.ucr[0] = ud;
          else o.ucr[1] = ud;
          o.ncross = min(o.ncross + 1, 2);
        }
        phid += kPi;
      }
      if (esc) {
        o.dprime = fmaf(tend, h, phi);
        return o;
      }
    }
    u = un;
    w = wn;
    if (u >= 1.0f) {
      o.bits |= BH_CAPTURED_BIT;
      return o;
    }
  }
  o.bits |= BH_CAPTURED_BIT | BH_UNFINISHED_BIT;
  return o;
}

__device__ __forceinline__ float disc_temperature(const ViewDev& v, float u) {
  if (v.T_law == 1) {
    float f = u * u * u * (1.0f - fsqrt(3.0f * u));
    return f > 0.0f ? v.T0 * fsqrt(fsqrt(f * v.T_norm)) : 0.0f;
  }
  return v.T0 * __builtin_amdgcn_exp2f(-v.T_exp * __log2f(3.0f * u));
}

// Partner of this lane inside its quad (DPP quad permutation, all lanes active): MASK 1
// swaps lanes 0<->1, 2<->3 (row partner), MASK 2 swaps 0<->2, 1<->3 (column partner).
template <int MASK>
__device__ __forceinline__ float quad_partner(float x) {
  constexpr int ctrl = MASK == 1 ? 0xB1 : 0x4E;  // quad_perm [1,0,3,2] / [2,3,0,1]
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), ctrl, 0xF, 0xF, true));
}

// (value at the quad partner) - (value here): the forward difference along the row
// (MASK 1) or column (MASK 2) on lanes at the quad's low side and its negative on the
// others.  Every use below is invariant under flipping the sign of all row (or all
// column) differences of a lane: footprint extents and the tent weights take |.|, and
// the solid angles are norms of cross products; IEEE negation is exact, so the results
// equal those of the forward differences bit for bit.
template <int MASK>
__device__ __forceinline__ float quad_diff(float x) {
  return quad_partner<MASK>(x) - x;
}

// atan2 over the whole circle, from the half-plane version
__device__ __forceinline__ float fatan2_any(float y, float x) {
  float r = fatan2_pos(fabsf(y), x);
  return y < 0.0f ? -r : r;
}

// Density of the procedural disc particles (Appendix B) at the hit point (ht, hr, hphi):
// particle j's point a = (hphi - phi_j(ht)) mod 2 pi, phi_j(t) = omega_j t + phi0_j, has
// u_a = u1 + (u2 - u1) sin^2(c_j (a + phi_j(ht))); d^2 = (a/pi - 1)^2 + (hr - 1/u_a)^2 and
// the particle adds (1 - d^2)^2 inside d < 1.  Particle records (two float4 each):
// (u1, u2 - u1, c, omega), (phi0, r_peri - 1, r_apo + 1, 0), sorted by r_peri - 1; the
// radial bounds skip particles that cannot reach d < 1.
__device__ __forceinline__ float disc_density(const ViewDev& v, float ht, float hr, float hphi) {
  const float k2Pi = 2.0f * kPi;
  float rho = 0.0f;
  // particles are sorted by the inner end of their radial reach; no particle before
  // pstart[bin of hr] reaches out to hr.  The wave starts at the smallest such index over
  // its active lanes and stops at the first particle whose reach starts beyond the largest
  // hr of its active lanes (an LDS minimum and maximum in the wave's own slots: one wave's
  // LDS operations complete in order), so the loop and its exit are wave-uniform and the
  // records are scalar loads; each lane tests its own hr against the particle's reach.
  __shared__ int wave_start[16], wave_hmax[16];
  int j0 = 0;
  float hmax = 0.0f;
  if (v.nparts > 0) {
    int* slot = &wave_start[threadIdx.x >> 6];
    int* hslot = &wave_hmax[threadIdx.x >> 6];
    *slot = v.nparts;
    *hslot = 0;
    atomicMin(slot, v.pstart[(int)fminf(hr * v.pscale, (float)v.pbins)]);
    atomicMax(hslot, __float_as_int(hr));  // hr > 0: its bit patterns order as its values
    j0 = __builtin_amdgcn_readfirstlane(*(volatile int*)slot);
    hmax = __int_as_float(__builtin_amdgcn_readfirstlane(*(volatile int*)hslot));
  }
  for (int j = j0; j < v.nparts; ++j) {
    const float4 p0 = v.parts[2 * j], p1 = v.parts[2 * j + 1];
    if (hmax < p1.y) break;  // this and every later particle starts beyond every lane's hr
    if (hr >= p1.y && hr <= p1.z) {
      float ph = fmaf(p0.w, ht, p1.x);
      float a = hphi - ph;
      a -= k2Pi * floorf(a * (1.0f / k2Pi));
      // sin^2 x = (1 - cos 2x) / 2, with the hardware cosine (argument in turns: 2x / 2 pi)
      const float c2 = __builtin_amdgcn_cosf(p0.z * (a + ph) * (1.0f / kPi));
      float ua = fmaf(p0.y, fmaf(-0.5f, c2, 0.5f), p0.x);
      float dr = hr - fdiv(1.0f, ua);
      float da = a * (1.0f / kPi) - 1.0f;
      float d2 = da * da + dr * dr;
      if (d2 < 1.0f) rho += (1.0f - d2) * (1.0f - d2);
    }
  }
  return rho;
}

// ---- area sources (Section 3.3.2 "Emitted light": nebulae and galaxies in a cube map) ----
// The paper reads them with the texture unit's anisotropic filtering over the beam's
// footprint; this is that filter written out.  The footprint is the parallelogram of
// directions d' + w d_w d' + h d_h d', |w|, |h| <= 1/2 (the pixel's box); its two axes are
// measured in level-0 texels on the face of d' (face Jacobian, Euclidean length); an
// N_maj x N_min grid of probes sits at the cell centres of the parallelogram, spaced no
// closer than half a level-0 texel: with s = max(l_min / 2, 1/2), N_maj = clamp(ceil(l_maj /
// s), 1, 16) along the longer axis and N_min = clamp(ceil(l_min / s), 1, 2) across it (so
// N_maj = ceil(2 l_maj / l_min) by 2 once l_min >= 1); every probe reads level
// lambda = log2(max(l_maj / N_maj, l_min / N_min)) - 1 trilinearly; the result is the probes'
// mean of (I, I T), or of (R, G, B) on a band map.  Each probe takes the face of its own
// direction, so footprints cross cube edges; bilinear coordinates are clamped to the face's
// outermost texel centres.

// texel types of the two map formats: (I, I T), and (R, G, B, 0) for band maps
template <bool BANDS> struct AreaTexel { using type = float2; };
template <> struct AreaTexel<true> { using type = float4; };

// One level of the map as a probe reads it
struct AreaLevel {
  uint32_t first;        // its texel 0
  int nL, last;          // last = max(nL - 2, 0)
  float half, off, top;  // nL / 2, nL / 2 - 1/2, nL - 1
};
__device__ __forceinline__ AreaLevel area_level(const AreaDev& M, int L) {
  AreaLevel a;
  a.nL = M.n0 >> L;
  a.last = max(a.nL - 2, 0);
  a.first = 8u * ((uint32_t)M.n0 * (uint32_t)M.n0 - (uint32_t)a.nL * (uint32_t)a.nL);
  const float fn = (float)a.nL;
  a.half = 0.5f * fn;
  a.off = fmaf(0.5f, fn, -0.5f);
  a.top = fn - 1.0f;
  return a;
}

// The 2 x 2 texels of a level around face coordinates (U, V) of `face`, and the position between
// them.  On the level of one texel a face the read starts at that texel, but three texels before
// the map's end at the latest, and area_add picks the face's own.
template <bool BANDS>
struct AreaQuad {
  typename AreaTexel<BANDS>::type a, b, c, e;
  float fx, fy;
};
template <bool BANDS>
__device__ __forceinline__ AreaQuad<BANDS> area_read(const AreaDev& M, const AreaLevel& A,
                                                     int face, float U, float V) {
  const float x = clampf(fmaf(A.half, U, A.off), 0.0f, A.top);
  const float y = clampf(fmaf(A.half, V, A.off), 0.0f, A.top);
  const int i0 = min((int)x, A.last), j0 = min((int)y, A.last);
  AreaQuad<BANDS> q;
  q.fx = x - (float)i0;
  q.fy = y - (float)j0;
  // face nL + j0 and nL have 24 bits at most; a map has 2 GiB at most (n0 <= 4096), so the offset
  // stays in 32 bits beside the map's address
  const uint32_t nL = (uint32_t)A.nL;
  const uint32_t first = __umul24(__umul24((uint32_t)face, nL) + (uint32_t)j0, nL) +
                         (A.first + (uint32_t)i0);
  const uint32_t end = 8u * (uint32_t)M.n0 * (uint32_t)M.n0 - 2u;
  using Tx = typename AreaTexel<BANDS>::type;
  const uint32_t at = min(first, end - 3u) * (uint32_t)sizeof(Tx);
  const Tx* r0 = (const Tx*)((const char*)M.tex + at);
  const Tx* r1 = (const Tx*)((const char*)M.tex + (at + nL * (uint32_t)sizeof(Tx)));
  q.a = r0[0];
  q.b = r0[1];
  q.c = r1[0];
  q.e = r1[1];
  return q;
}
// s += weight * (the bilinear value of q)
template <bool BANDS>
__device__ __forceinline__ void area_add(const AreaQuad<BANDS>& q, float weight, int nL,
                                         int face, float3& s) {
  if (nL == 1) {
    auto own = [&](float a, float b, float e) { return face < 4 ? a : (face == 4 ? b : e); };
    s.x = fmaf(weight, own(q.a.x, q.b.x, q.e.x), s.x);
    s.y = fmaf(weight, own(q.a.y, q.b.y, q.e.y), s.y);
    if constexpr (BANDS) s.z = fmaf(weight, own(q.a.z, q.b.z, q.e.z), s.z);
    return;
  }
  const float y1 = q.fy * weight, y0 = weight - y1;
  const float wb = q.fx * y0, we = q.fx * y1, wa = y0 - wb, wc = y1 - we;
  s.x = fmaf(we, q.e.x, fmaf(wc, q.c.x, fmaf(wb, q.b.x, fmaf(wa, q.a.x, s.x))));
  s.y = fmaf(we, q.e.y, fmaf(wc, q.c.y, fmaf(wb, q.b.y, fmaf(wa, q.a.y, s.y))));
  if constexpr (BANDS)
    s.z = fmaf(we, q.e.z, fmaf(wc, q.c.z, fmaf(wb, q.b.z, fmaf(wa, q.a.z, s.z))));
}

// The footprint of d' on the face of its centre, shared by the star gather and the area filter:
// the axes d_w d', d_h d' in the face's component order and their face-coordinate changes
// (J00, J10) and (J01, J11).
struct FaceFootprint {
  FaceOf c;
  float im, sg, U, V;              // 1 / |d'_k|, sign of d'_k, face coordinates of d'
  float wk, wa, wb, hk, ha, hb;
  float J00, J01, J10, J11;
};

__device__ __forceinline__ FaceFootprint face_footprint(float d0, float d1, float d2, float w0,
                                                        float w1, float w2, float h0, float h1,
                                                        float h2) {
  FaceFootprint f;
  f.c = face_of(d0, d1, d2);
  const int k = f.c.k;
  f.wk = k == 0 ? w0 : (k == 1 ? w1 : w2);
  f.wa = k == 0 ? w1 : (k == 1 ? w2 : w0);
  f.wb = k == 0 ? w2 : (k == 1 ? w0 : w1);
  f.hk = k == 0 ? h0 : (k == 1 ? h1 : h2);
  f.ha = k == 0 ? h1 : (k == 1 ? h2 : h0);
  f.hb = k == 0 ? h2 : (k == 1 ? h0 : h1);
  f.sg = f.c.pk < 0.0f ? -1.0f : 1.0f;
  f.im = fdiv(1.0f, f.c.m);
  f.U = f.c.pa * f.im;
  f.V = f.c.pb * f.im;
  f.J00 = (f.wa - f.U * f.sg * f.wk) * f.im;
  f.J01 = (f.ha - f.U * f.sg * f.hk) * f.im;
  f.J10 = (f.wb - f.V * f.sg * f.wk) * f.im;
  f.J11 = (f.hb - f.V * f.sg * f.hk) * f.im;
  return f;
}

// mean (I, I T) of the map over the footprint f of d', or mean (R, G, B) of a band map (BANDS,
// into A, B, C).  PAIR: two probes per iteration also where two levels are read.
template <bool BANDS, bool PAIR>
__device__ __forceinline__ void area_filter(const AreaDev& M, const FaceFootprint& f, float& A,
                                            float& B, float& Cc) {
  const float half_n0 = 0.5f * (float)M.n0;
  // axis lengths in level-0 texels
  const float la = half_n0 * fsqrt(f.J00 * f.J00 + f.J10 * f.J10);
  const float lb = half_n0 * fsqrt(f.J01 * f.J01 + f.J11 * f.J11);
  const bool swap = lb > la;
  const float lmaj = swap ? lb : la, lmin = swap ? la : lb;
  const float spc = fmaxf(0.5f * lmin, 0.5f), ispc = fdiv(1.0f, spc);
  const int nmaj = (int)clampf(ceilf(lmaj * ispc), 1.0f, 16.0f);
  const int nmin = lmin * ispc > 1.0f ? 2 : 1;
  float3 sum = make_float3(0.0f, 0.0f, 0.0f);
  const AreaLevel l0 = area_level(M, 0);
  // A footprint within half a texel takes one probe, at d' itself and on level 0 (its spacing is
  // at most half a texel): no corners, levels or probe loop.  Most of a frame magnifies the map;
  // a wave of such pixels skips the rest.
  if (nmaj == 1 && nmin == 1) {
    area_add<BANDS>(area_read<BANDS>(M, l0, f.c.face, f.U, f.V), 1.0f, l0.nL, f.c.face, sum);
  } else {
    const float fmaj = (float)nmaj, fmin = (float)nmin;
    const float sp = fmaxf(fdiv(lmaj, fmaj), fdiv(lmin, fmin));
    float lam = sp > 0.0f ? __log2f(sp) - 1.0f : 0.0f;
    lam = clampf(lam, 0.0f, (float)(M.levels - 1));
    // The directions on one face form a convex set of (w, h) (an intersection of half-planes),
    // so when the parallelogram's four corners lie on the face of d', every probe does too and
    // needs no face lookup.  The corners lie on it when |p_k| - |p_a| and |p_k| - |p_b| stay
    // positive there: four linear functions of (w, h), least at the corner where both axes lower
    // them.
    auto least = [&](float p, float wp, float hp) {
      return fmaf(f.sg, f.c.pk, p) -
             0.5f * (fabsf(fmaf(f.sg, f.wk, wp)) + fabsf(fmaf(f.sg, f.hk, hp)));
    };
    AreaProbes P;
    P.k = f.c.k;
    P.face = f.c.face;
    P.one_face = fminf(fminf(least(f.c.pa, f.wa, f.ha), least(-f.c.pa, -f.wa, -f.ha)),
                       fminf(least(f.c.pb, f.wb, f.hb), least(-f.c.pb, -f.wb, -f.hb))) > 0.0f;
    P.pk = f.c.pk;
    P.pa = f.c.pa;
    P.pb = f.c.pb;
    P.jk = swap ? f.hk : f.wk;
    P.ja = swap ? f.ha : f.wa;
    P.jb = swap ? f.hb : f.wb;
    P.nk = swap ? f.wk : f.hk;
    P.na = swap ? f.wa : f.ha;
    P.nb = swap ? f.wb : f.hb;
    P.n = nmaj * nmin;
    P.minor = nmin;
    P.inv = fdiv(1.0f, fmaj);
    const float in = P.inv * (nmin == 1 ? 1.0f : 0.5f);  // weight of a probe
    // A probe is one wait for its scattered texels, and the waves of the photon ring (0.4% of a
    // 1600 x 900 frame's take 32 probes on two levels) end last, on an idle chip: 13 of 44 us went
    // to footprints of more than 4 major probes.  So two probes' texels are in flight at a time.
    // Level 0 alone, for every lane here (97% of the waves under a map of 512 x 512 texels): its
    // record is the wave's.
    if (__ballot(lam > 0.0f) == 0ull) {
      for (int t = 0; t < P.n; t += 2) {
        const AreaAt p0 = area_at(P, t), p1 = area_at(P, min(t + 1, P.n - 1));
        const AreaQuad<BANDS> q0 = area_read<BANDS>(M, l0, p0.face, p0.u, p0.v);
        const AreaQuad<BANDS> q1 = area_read<BANDS>(M, l0, p1.face, p1.u, p1.v);
        area_add<BANDS>(q0, in, l0.nL, p0.face, sum);
        if (t + 1 < P.n) area_add<BANDS>(q1, in, l0.nL, p1.face, sum);
      }
    } else {
      const int La = (int)lam, Lb = min(La + 1, M.levels - 1);
      const float fr = lam - (float)La;
      const bool two = fr > 0.0f && Lb != La;  // the second level has weight
      const float in1 = two ? fr * in : 0.0f, in0 = in - in1;
      const AreaLevel la_ = area_level(M, La), lb_ = area_level(M, Lb);
      // In the kernels with band code a second probe has no registers: it spilled 11 of them and
      // cost the 1080p any-colour frame 109.6 -> 111.3 us; without it the odd-sized nebula frame
      // takes 44.8 us for 39.8.
      constexpr int kProbes = PAIR ? 2 : 1;
      for (int t = 0; t < P.n; t += kProbes) {
        AreaQuad<BANDS> q0[kProbes], q1[kProbes];
        int face[kProbes];
#pragma unroll
        for (int i = 0; i < kProbes; ++i) {
          const AreaAt p = area_at(P, min(t + i, P.n - 1));
          face[i] = p.face;
          q0[i] = area_read<BANDS>(M, la_, p.face, p.u, p.v);
          q1[i] = area_read<BANDS>(M, lb_, p.face, p.u, p.v);
        }
#pragma unroll
        for (int i = 0; i < kProbes; ++i) {
          if (i > 0 && t + i >= P.n) break;
          area_add<BANDS>(q0[i], in0, la_.nL, face[i], sum);
          if (two) area_add<BANDS>(q1[i], in1, lb_.nL, face[i], sum);
        }
      }
    }
  }
  A = sum.x;
  B = sum.y;
  Cc = sum.z;
}

// C_b(r, g, D) from the colour-shift table (Section 3.4.2; cshift.hip): log2 values read
// trilinearly, linearly in r and g and, between the two D nodes around D, linearly in 1 / D;
// r, g and log2 D clamped to the node range
__device__ __forceinline__ float3 lerp3(float f, float3 a, float3 b) {
  return make_float3(fmaf(f, b.x - a.x, a.x), fmaf(f, b.y - a.y, a.y), fmaf(f, b.z - a.z, a.z));
}
struct ShiftPlane {  // the D nodes around a pixel's D, the same for its stars and its sky
  int k0;
  float fz;
};
__device__ __forceinline__ ShiftPlane cshift_plane(float D) {
  constexpr float step = 6.0f / (float)(kCshiftN - 1);
  const float Dc = clampf(D, 0.125f, 8.0f);
  const int k0 = min((int)((__log2f(Dc) + 3.0f) * (1.0f / step)), kCshiftN - 2);
  // hardware 2^x: the arguments, and the table's log2 C >= -100, keep the results normal
  const float inv0 = __builtin_amdgcn_exp2f(3.0f - (float)k0 * step);
  const float inv1 = __builtin_amdgcn_exp2f(3.0f - (float)(k0 + 1) * step);
  return ShiftPlane{k0, clampf(fdiv(fdiv(1.0f, Dc) - inv0, inv1 - inv0), 0.0f, 1.0f)};
}

__device__ __forceinline__ float3 cshift_lookup(const float4* __restrict__ tab, float r, float g,
                                                const ShiftPlane& D) {
  constexpr float top = (float)(kCshiftN - 1);
  const float x = clampf(r * top, 0.0f, top), y = clampf(g * top, 0.0f, top);
  const int i0 = min((int)x, kCshiftN - 2), j0 = min((int)y, kCshiftN - 2);
  const float fx = x - (float)i0, fy = y - (float)j0, fz = D.fz;
  const int k0 = D.k0;
  const float4* p = tab + ((uint32_t)k0 * kCshiftN + (uint32_t)i0) * kCshiftN + (uint32_t)j0;
  constexpr uint32_t sk = kCshiftN * kCshiftN, si = kCshiftN;
  const float4 c000 = p[0], c010 = p[1], c100 = p[si], c110 = p[si + 1];
  const float4 c001 = p[sk], c011 = p[sk + 1], c101 = p[sk + si], c111 = p[sk + si + 1];
  auto between = [&](const float4& a, const float4& b) {  // in D
    return lerp3(fz, make_float3(a.x, a.y, a.z), make_float3(b.x, b.y, b.z));
  };
  const float3 e = lerp3(fx, lerp3(fy, between(c000, c001), between(c010, c011)),
                         lerp3(fy, between(c100, c101), between(c110, c111)));
  return make_float3(__builtin_amdgcn_exp2f(e.x), __builtin_amdgcn_exp2f(e.y),
                     __builtin_amdgcn_exp2f(e.z));
}

// The view record of a kernel that takes it as its first argument (launch_plain checks that it
// does), to be read again from the argument segment where it is used: fields kept since the
// kernel's start would hold scalar registers across the whole trace (8 to 28 of them spilled into
// vector registers, and two of those to memory; without: 1080p frame 29.0 -> 28.0 us, 8K 324 ->
// 307, animated 52.5 -> 49.4).
__device__ __forceinline__ const ViewDev& reread(const ViewDev&) {
  typedef const __attribute__((address_space(4))) ViewDev* Args;
  Args p = (Args)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const ViewDev*)p;
}

// One pixel; every lane of the wave must call this together (quad exchanges).
// COUNT: also mark every star-map texel the footprint visits and add up the bytes the pixel
// requests (measurement only, see CountBufs).  ANIM: views may have a particle disc
// (retarded times).
// MARCH: ray marching (march_ray) in place of TraceRay; no tables are read.
// LATE: the view is the kernel's first argument (reread).
template <bool COUNT, bool ANIM = false, bool MARCH = false, int AREA = 0, bool LATE = false>
__device__ __forceinline__ void render_pixel(const ViewDev& v0, const TablesDev& T,
                                             const LutDev& L, int px, int py,
                                             const CountBufs* cnt) {
  const ViewDev& v = v0;

  // ---- beam initialisation (Section 3.2)
  float qw = (float)px + 0.5f - v.half_w;
  float qh = v.half_h - (float)py - 0.5f;
  float inq = __builtin_amdgcn_rsqf(qw * qw + qh * qh + v.f * v.f);  // argument >= f^2 > 0
  float q0 = qw * inq, q1 = qh * inq, q2 = -v.f * inq;
  // camera direction and its aberration into the static frame, as the part transverse to
  // e_x' (n0, n1, n2) and the radial component nr
  float nc0 = q0 * v.ew[0] + q1 * v.eh[0] + q2 * v.ed[0];
  float nc1 = q0 * v.ew[1] + q1 * v.eh[1] + q2 * v.ed[1];
  float nc2 = q0 * v.ew[2] + q1 * v.eh[2] + q2 * v.ed[2];
  float ncr = q0 * v.er[0] + q1 * v.er[1] + q2 * v.er[2];
  float nv = nc0 * v.vhat[0] + nc1 * v.vhat[1] + nc2 * v.vhat[2] + ncr * v.er[3];
  float ka = (v.gamma - 1.0f) * nv - v.gamma * v.vmag;
  // coordinate direction d: the transverse part as is, the radial component scaled by
  // sqrt(1 - u) (eq. staticbasis)
  const float d0 = nc0 + ka * v.vhat[0], d1 = nc1 + ka * v.vhat[1], d2 = nc2 + ka * v.vhat[2];
  const float dr = v.sq1mu * (ncr + ka * v.er[3]);
  float dcam = fdiv(v.inv_sq1mu, v.gamma * (1.0f - v.vmag * nv));
  // e_z' = e_x' x d / |e_x' x d|, and |e_x' x d| = |transverse part|
  float cz0 = v.rhat[1] * d2 - v.rhat[2] * d1;
  float cz1 = v.rhat[2] * d0 - v.rhat[0] * d2;
  float cz2 = v.rhat[0] * d1 - v.rhat[1] * d0;
  const float ncz2 = d0 * d0 + d1 * d1 + d2 * d2;
  const float dn2 = ncz2 + dr * dr;
  float ncz, inv_ncz;  // |e_x' x d| and its inverse
  float ey0, ey1, ey2;  // e_y' = e_z' x e_x'
  unsigned bits = 0;
  float u_ic = v.u_ic, u_oc = v.u_oc;
  if (!(ncz2 > 1e-14f * dn2)) {
    // radial beam: any plane through it; pick one containing a fixed axis
    bits |= BH_DEGENERATE_BIT;
    float ax0 = fabsf(v.rhat[0]) < 0.9f ? 1.0f : 0.0f, ax1 = 1.0f - ax0;
    cz0 = v.rhat[1] * 0.0f - v.rhat[2] * ax1;
    cz1 = v.rhat[2] * ax0 - v.rhat[0] * 0.0f;
    cz2 = v.rhat[0] * ax1 - v.rhat[1] * ax0;
    float n2 = __builtin_amdgcn_rsqf(cz0 * cz0 + cz1 * cz1 + cz2 * cz2);
    cz0 *= n2; cz1 *= n2; cz2 *= n2;
    ey0 = cz1 * v.rhat[2] - cz2 * v.rhat[1];
    ey1 = cz2 * v.rhat[0] - cz0 * v.rhat[2];
    ey2 = cz0 * v.rhat[1] - cz1 * v.rhat[0];
    ncz = fmaxf(fsqrt(ncz2), 1e-7f * fsqrt(dn2));
    inv_ncz = fdiv(1.0f, ncz);
    u_ic = -1.0f;
  } else {
    inv_ncz = __builtin_amdgcn_rsqf(ncz2);
    ncz = ncz2 * inv_ncz;
    cz0 *= inv_ncz; cz1 *= inv_ncz; cz2 *= inv_ncz;
    // (e_x' x d) x e_x' is d's transverse part
    ey0 = d0 * inv_ncz; ey1 = d1 * inv_ncz; ey2 = d2 * inv_ncz;
  }
  float delta = fatan2_pos(ncz, dr);
  // t = +-(e_z x e_z') with t.e_y' >= 0; alpha = angle(e_x', t)
  float t0 = -cz1, t1 = cz0;
  float nt = fsqrt(t0 * t0 + t1 * t1);
  float alpha = 0.0f;
  if (!(nt > 1e-7f)) {
    bits |= BH_DEGENERATE_BIT;
    u_ic = -1.0f;
  } else {
    float int_ = fdiv(1.0f, nt);
    float tx = (t0 * v.rhat[0] + t1 * v.rhat[1]) * int_;
    float ty = (t0 * ey0 + t1 * ey1) * int_;
    if (ty < 0.0f) {
      tx = -tx;
      ty = -ty;
      t0 = -t0;  // t now points along the line of nodes with t.e_y' >= 0
      t1 = -t1;
    }
    alpha = fatan2_pos(ty, tx);
  }
  float zeta = cz2;

  // ---- TraceRay (Algorithm 1)
  const float cotd = dr * inv_ncz;
  TraceOut tr;
  if constexpr (MARCH)
    tr = march_ray(v.u_c, alpha, cotd, u_ic, u_oc, v.march_steps, v.march_h);
  else
    tr = trace_ray<ANIM>(T, v.u_c, delta, alpha, cotd, u_ic, u_oc,
                         v.rho >= 1.0f && v.density_mode == 0 && !v.aov);
  bits |= tr.bits;
  const bool captured = (tr.bits & BH_CAPTURED_BIT) != 0;
  uint32_t req = tr.req;  // bytes requested (COUNT only)

  // ---- disc (Sections 3.3.3, 3.4.2), front to back
  float cr = 0.0f, cg = 0.0f, cb = 0.0f, trans = 1.0f;
  if (tr.ncross > 0) {
    const float ie = fdiv(1.0f, tr.e);
    // animated disc: crossing k sits at (-1)^m_k t, i.e. at disc azimuth az0 + m_k pi
    const bool anim = ANIM && v.density_mode == 1;
    float az0 = 0.0f;
    if (anim) az0 = fatan2_any(t1, t0);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      // a crossing behind an opaque one (transmittance exactly 0) adds nothing
      if (k >= tr.ncross || !(trans > 0.0f)) break;
      float uk = k == 0 ? tr.ucr[0] : tr.ucr[1];
      float Tp = disc_temperature(v, uk);
      // 1 / k'^t = sqrt(1 - 3u/2) and Omega' = sqrt(u^3 / 2) on the circular orbit at u
      float ikt = fsqrt(1.0f - 1.5f * uk);
      float om = fsqrt(0.5f * uk * uk * uk);
      float D = dcam * ikt * fdiv(1.0f, 1.0f + om * zeta * ie);
      float4 Lb = band_lookup(L, D * Tp);
      if (COUNT) req += 32;  // two band-table entries
      float rk = v.rho;
      if (anim) {
        float tk = k == 0 ? tr.tret[0] : tr.tret[1];
        int mk = k == 0 ? tr.mcr[0] : tr.mcr[1];
        float dens = disc_density(v, v.time - tk, fdiv(1.0f, uk), az0 + (float)mk * kPi);
        rk = fminf(1.0f, v.rho * dens);
      }
      float w = trans * rk * v.k_disc;
      cr += w * Lb.x;
      cg += w * Lb.y;
      cb += w * Lb.z;
      trans *= 1.0f - rk;
    }
  }

  // Nothing behind a wave of hidden pixels: the stars and area sources of a pixel behind an
  // opaque disc crossing (transmittance exactly 0) add nothing, and a captured pixel receives
  // none.  A wave with no other kind is done (its quads' derivatives serve no one else), unless
  // the per-pixel record wants the mip level.  60% of the 1080p frame's waves: 30.8 -> 29.1 us,
  // 8K 374 -> 336.  (Decided per wave: the same per quad cost more than it saved.)
  int mip = 255;
  const ViewDev& w = LATE ? reread(v0) : v0;
  if (COUNT || w.aov || __ballot(trans > 0.0f && !captured) != 0ull) {
    // ---- stars (Sections 3.3.2, 3.4.1)
    // hardware sine and cosine (argument in turns): the escape direction only places star
    // light, where their ~1e-6 rad error is a thousandth of a pixel
    const float turns = tr.dprime * 0.159154943091895336f;
    const float sdp = __builtin_amdgcn_sinf(turns), cdp = __builtin_amdgcn_cosf(turns);
    float dp0 = captured ? 0.0f : cdp * w.rhat[0] + sdp * ey0;
    float dp1 = captured ? 0.0f : cdp * w.rhat[1] + sdp * ey1;
    float dp2 = captured ? 0.0f : cdp * w.rhat[2] + sdp * ey2;
    int cap = captured ? 1 : 0;
    cap |= __builtin_amdgcn_mov_dpp(cap, 0xB1, 0xF, 0xF, true);
    cap |= __builtin_amdgcn_mov_dpp(cap, 0x4E, 0xF, 0xF, true);
    float dw0 = quad_diff<1>(dp0), dw1 = quad_diff<1>(dp1), dw2 = quad_diff<1>(dp2);
    float dh0 = quad_diff<2>(dp0), dh1 = quad_diff<2>(dp1), dh2 = quad_diff<2>(dp2);
    if (cap) bits |= BH_STAR_ZEROED_BIT;
    ShiftPlane sp{0, 0.0f};
    if constexpr (AREA >= 2) sp = cshift_plane(dcam);
    if (w.has_stars && !cap) {
      const StarsDev& S = w.stars;
      const FaceFootprint ff = face_footprint(dp0, dp1, dp2, dw0, dw1, dw2, dh0, dh1, dh2);
      const float U = ff.U, V = ff.V;
      const float J00 = ff.J00, J01 = ff.J01, J10 = ff.J10, J11 = ff.J11;
      const int face = ff.c.face;
      float hu = fabsf(J00) + fabsf(J01), hv = fabsf(J10) + fabsf(J11);
      float E0 = fmaxf(hu, hv) * (float)S.n0;
      // smallest level with E0 / 2^L <= 8: from the exponent and mantissa of E0 / 8
      int Lv = 0;
      {
        float q = E0 * 0.125f;
        if (q > 1.0f) {
          unsigned b = __float_as_uint(q);
          int ex = (int)((b >> 23) & 255u) - 127;   // q = 1.m * 2^ex, q finite and > 1
          Lv = ex + ((b & 0x7fffffu) != 0u ? 1 : 0);
        }
        if (!(q <= 3.0e38f)) Lv = S.levels - 1;      // infinite or NaN footprint
        Lv = min(Lv, S.levels - 1);
      }
      mip = Lv;
      float det = J00 * J11 - J01 * J10;
      // band-colour star maps are read only by the band variants (AREA 2 and 3)
      const bool bands = AREA >= 2 && S.bands;
      float A = 0.0f, B = 0.0f, Cb = 0.0f;
      // behind an opaque disc crossing (transmittance exactly 0) the stars add nothing: their
      // light is scaled by trans below, so the gather is skipped (the level above is kept)
      if (fabsf(det) >= 1e-20f && trans > 0.0f) {
        float idet = fdiv(1.0f, det);
        Footprint F;
        // inverse face Jacobian
        const float i00 = J11 * idet, i01 = -J01 * idet, i10 = -J10 * idet, i11 = J00 * idet;
        const int nL = S.n0 >> Lv;
        const float fn = (float)nL;
        // clamp before the integer conversion (equal to floor-then-clamp for in-range values)
        const float top = fn - 1.0f;
        int x0 = (int)clampf(0.5f * (U - hu + 1.0f) * fn, 0.0f, top);
        int x1 = (int)clampf(0.5f * (U + hu + 1.0f) * fn, 0.0f, top);
        int y0 = (int)clampf(0.5f * (V - hv + 1.0f) * fn, 0.0f, top);
        int y1 = (int)clampf(0.5f * (V + hv + 1.0f) * fn, 0.0f, top);
        x1 = min(x1, x0 + 8);
        y1 = min(y1, y0 + 8);
        F.nL = nL;
        const int wpr = ((nL + 31) >> 5) + 1;
        F.wpr4 = 4 * wpr;
        F.sh = x0 & 31;
        F.ny = y1 - y0;
        F.span = (1u << (x1 - x0 + 1)) - 1u;  // x1 - x0 <= 8
        F.texel0 = S.level_off[Lv] + ((uint32_t)face * (uint32_t)nL + (uint32_t)y0) * (uint32_t)nL +
                   (uint32_t)x0;
        F.occ = S.occ + S.occ_off[Lv] +
                2u * (((uint32_t)face * (uint32_t)nL + (uint32_t)y0) * (uint32_t)wpr +
                      (uint32_t)(x0 >> 5));
        // a level-L texel is tw = 2 / nL wide in face coordinates; the corner (x0, y0) lies at
        // (cu, cv) from the centre direction (U, V)
        const float tw = __builtin_ldexpf(S.tw0, Lv);  // nL = n0 / 2^L: 2 / nL exactly
        const float cu = (float)x0 * tw - 1.0f - U, cv = (float)y0 * tw - 1.0f - V;
        F.Wc = i00 * tw;
        F.Wr = i01 * tw;
        F.W0 = fmaf(i00, cu, i01 * cv);
        F.Hc = i10 * tw;
        F.Hr = i11 * tw;
        F.H0 = fmaf(i10, cu, i11 * cv);
        F.one = S.one;
        if (COUNT) req += 12;  // level offsets and scale
        if constexpr (AREA >= 2) {
          if (bands) {
            if (S.fp16)
              gather<kTexBand16, COUNT, false>(S.tex, F, cnt, req, A, B, Cb);
            else
              gather<kTexBand32, COUNT, false>(S.tex, F, cnt, req, A, B, Cb);
          }
        }
        if (!bands) {
          if (S.fp16)
            gather<kTexIT16, COUNT, AREA != 3>(S.tex, F, cnt, req, A, B, Cb);
          else
            gather<kTexIT32, COUNT, AREA != 3>(S.tex, F, cnt, req, A, B, Cb);
        }
        const float iscale = S.scale[Lv];
        A *= iscale;
        B *= S.fp16 && !bands ? iscale * 1024.0f : iscale;
        Cb *= iscale;
      }
      float cdx = dw1 * dh2 - dw2 * dh1, cdy = dw2 * dh0 - dw0 * dh2, cdz = dw0 * dh1 - dw1 * dh0;
      // Omega / Omega' = |q_w x q_h| / |d'_w x d'_h| with the same quad differences of the
      // camera-frame direction q = (q^w, q^h, -f) inq.  The row partner shares q^h and the
      // column partner q^w, so with a = quad difference of inq along the row and b along the
      // column, q_w = (dq0, q^h a, -f a) and q_h = (q^w b, dq1, -f b), whose cross product is
      // (f a (dq1 - q^h b), f b (dq0 - q^w a), dq0 dq1 - q^w q^h a b).
      const float qa = quad_diff<1>(inq), qb = quad_diff<2>(inq);
      const float dq0 = quad_diff<1>(q0), dq1 = quad_diff<2>(q1);
      const float cq0 = w.f * qa * (dq1 - qh * qb), cq1 = w.f * qb * (dq0 - qw * qa);
      const float cq2 = dq0 * dq1 - (qw * qh) * (qa * qb);
      const float om2 = cq0 * cq0 + cq1 * cq1 + cq2 * cq2;
      const float omp2 = cdx * cdx + cdy * cdy + cdz * cdz;
      if (bands) {
        // light of any colour: band sum and chromaticity, shifted by C(r, g, D_cam)
        const float Ssum = A + B + Cb;
        if (Ssum > 0.0f && omp2 > 0.0f) {
          const float iS = fdiv(1.0f, Ssum);
          const float3 C = cshift_lookup(S.ctab, A * iS, B * iS, sp);
          const float sc = trans * w.k_star * fsqrt(om2) * __builtin_amdgcn_rsqf(omp2) * Ssum;
          cr += sc * C.x;
          cg += sc * C.y;
          cb += sc * C.z;
        }
      } else if (A > 0.0f && omp2 > 0.0f) {
        float Tpix = fdiv(B, A);
        float4 Lr = band_lookup(L, dcam * Tpix);
        float4 Ln = band_lookup(L, Tpix);
        if (COUNT) req += 64;
        float sc = trans * w.k_star * fsqrt(om2) * __builtin_amdgcn_rsqf(omp2) * fdiv(A, Ln.w);
        cr += sc * Lr.x;
        cg += sc * Lr.y;
        cb += sc * Lr.z;
      }
    }

    // ---- area sources: the footprint's mean radiance, one Doppler shift per pixel as for
    // stars, no lensing amplification (Section 3.4.1).  The face footprint is formed again: kept
    // across the star gather it would spill.
    if ((AREA == 1 || AREA == 2) && w.area.tex && !cap && trans > 0.0f) {
      const FaceFootprint ff = face_footprint(dp0, dp1, dp2, dw0, dw1, dw2, dh0, dh1, dh2);
      float A, B, Cc;
      if (AREA == 2 && w.area.bands) {
        // light of any colour: band sum S and chromaticity (r, g), shifted by C(r, g, D_cam)
        area_filter<true, false>(w.area, ff, A, B, Cc);
        const float S = A + B + Cc;
        if (S > 0.0f) {
          const float iS = fdiv(1.0f, S);
          const float3 C = cshift_lookup(w.area.ctab, A * iS, B * iS, sp);
          const float sc = trans * w.area.k_area * S;
          cr += sc * C.x;
          cg += sc * C.y;
          cb += sc * C.z;
        }
      } else {
        area_filter<false, AREA == 1>(w.area, ff, A, B, Cc);
        if (A > 0.0f) {
          const float Tpix = fdiv(B, A);
          const float4 Lr = band_lookup(L, dcam * Tpix), Ln = band_lookup(L, Tpix);
          const float sc = trans * w.area.k_area * fdiv(A, Ln.w);
          cr += sc * Lr.x;
          cg += sc * Lr.y;
          cb += sc * Lr.z;
        }
      }
    }
  }

  if (COUNT) {
    if (px < w.width && py < w.height) req += w.aov ? 32 : 16;
    unsigned long long t = req;
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
    if ((threadIdx.x & 63) == 0) atomicAdd(cnt->l2_bytes, t);
  }
  if (px < w.width && py < w.height) {
    size_t idx = (size_t)py * w.width + px;
    store_stream(&w.out[idx], make_float4(cr, cg, cb, 1.0f));
    if (w.aov) {
      bits |= (unsigned)mip << 8;
      store_stream(&w.aov[idx], make_float4(captured ? __builtin_inff() : tr.dprime, tr.ucr[0],
                                             tr.ucr[1], __uint_as_float(bits)));
    }
  }
}

template <int TW, int TH, int PPT>
struct TileCfg {
  static constexpr int kBX = TW / 8, kBY = TH / 8;           // 8x8 blocks per tile
  static constexpr int kWaves = kBX * kBY / PPT;
  static constexpr int kThreads = 64 * kWaves;
  static_assert(kBX * kBY % PPT == 0, "blocks must divide by pixels per thread");
  static_assert(kWaves <= 16, "the particle loop keeps one LDS slot per wave, 16 at most");
};

template <int TW, int TH, int PPT, bool COUNT = false, bool ANIM = false, bool MARCH = false,
          int AREA = 0, bool LATE = false>
__device__ __forceinline__ void render_tile(const ViewDev& v, const TablesDev& T, const LutDev& L,
                                            int tx0, int ty0, const CountBufs* cnt = nullptr) {
  using C = TileCfg<TW, TH, PPT>;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int q = lane >> 2;
  const int ox = 2 * (q & 3) + (lane & 1), oy = 2 * (q >> 2) + ((lane >> 1) & 1);
#pragma unroll 1
  for (int p = 0; p < PPT; ++p) {
    int blk = p * C::kWaves + wave;
    int bx = blk % C::kBX, by = blk / C::kBX;
    int px = tx0 + 8 * bx + ox, py = ty0 + 8 * by + oy;
    // skip 8x8 blocks entirely outside the image (uniform per wave)
    if (tx0 + 8 * bx >= v.width || ty0 + 8 * by >= v.height) continue;
    render_pixel<COUNT, ANIM, MARCH, AREA, LATE>(v, T, L, px, py, cnt);
  }
}

// XCD-aware tile order.  Workgroup b runs on XCD b % 8.  The image's tiles are grouped in
// blocks of kXBW x kXBH tiles that stay on one XCD (neighbouring tiles share that XCD's L2),
// and the blocks are dealt to the 8 XCDs in turn, so every XCD gets work from all over the
// image: per-tile cost varies strongly across a frame (shadow, disc, star field), and one
// band of rows per XCD left the lightest XCDs idle for ~10% of the frame.
constexpr int kXBW = 4, kXBH = 2;

__device__ __forceinline__ bool xcd_tile(int b, int tiles_x, int tiles_y, int* col, int* row) {
  int x = b & 7, k = b >> 3;
  int bx = (tiles_x + kXBW - 1) / kXBW;
  int blk = x + 8 * (k / (kXBW * kXBH)), q = k % (kXBW * kXBH);
  *row = (blk / bx) * kXBH + q / kXBW;
  *col = (blk % bx) * kXBW + q % kXBW;
  return *col < tiles_x && *row < tiles_y;
}

// workgroups of a plain launch over tiles_x x tiles_y tiles (a multiple of 8)
static inline int xcd_grid(int tiles_x, int tiles_y) {
  int nblk = ((tiles_x + kXBW - 1) / kXBW) * ((tiles_y + kXBH - 1) / kXBH);
  return ((nblk + 7) / 8) * 8 * kXBW * kXBH;
}

// Resident waves per SIMD the one-launch and per-tile kernels are held to (the register
// budget the compiler keeps to): 8, and 5 for the area-source variants, whose probe loop
// spilled 20 vector registers at 8 waves and 9 at 6 (nebula frame 1599 x 899: 43.5 us at 6 waves,
// 42.4 at 5, one probe in flight; two in flight 38.9 and 33.7, 4K 97.2 and 99.2; at 7 waves 48.5,
// and the any-colour frame 139 us for 109).  With particles too: 64.6 us at 6 waves and 59.8 at 5
// at 1599 x 899, 75.8 and 76.6 at 1080p, 205 and 222 at 4K.  Band star maps without area maps fit
// 8 (64 VGPRs).
template <int FEAT>
constexpr int kMinWaves = (FEAT & kFeatArea) ? 5 : 8;

// the area and band code a feature set needs (render_pixel's AREA): 0 none, 1 (I, I T) area
// maps, 2 area maps of either format and band star maps (run-time branches on the maps'
// formats), 3 band star maps without area maps
template <int FEAT>
constexpr int kAreaOf =
    (FEAT & kFeatBands) ? ((FEAT & kFeatArea) ? 2 : 3) : ((FEAT & kFeatArea) ? 1 : 0);

// One launch per view, tiles in the XCD-aware order above.
// At least 8 resident waves per SIMD: the register budget the compiler keeps to.  The
// animated variant would otherwise take 92 scalar registers and fit only 7 waves; held to
// 8 it spills a few scalars into vector-register lanes and runs 7% faster.  (The
// persistent batch kernel is left unbounded: held to 8 waves it would spill to memory.)
template <int TW, int TH, int PPT, int FEAT>
__global__ void __launch_bounds__((TW / 8) * (TH / 8) * 64 / PPT, kMinWaves<FEAT>)
    k_render(ViewDev v, TablesDev T, LutDev L, int tiles_x, int tiles_y) {
  int col, row;
  if (!xcd_tile(blockIdx.x, tiles_x, tiles_y, &col, &row)) return;
  render_tile<TW, TH, PPT, false, (FEAT & kFeatParticles) != 0, false, kAreaOf<FEAT>, true>(
      v, T, L, col * TW, row * TH);
}

// The render with ray marching in place of TraceRay (16x16 tiles, one pixel per thread);
// AREA as in render_pixel.
template <int AREA>
__global__ void __launch_bounds__(256)
    k_render_march(ViewDev v, LutDev L, int tiles_x, int tiles_y) {
  int col, row;
  if (!xcd_tile(blockIdx.x, tiles_x, tiles_y, &col, &row)) return;
  TablesDev none{};
  render_tile<16, 16, 1, false, false, true, AREA>(v, none, L, col * 16, row * 16);
}

// The run holding flat tile index `it` (wave-uniform): the last run whose start is <= it.
__device__ __forceinline__ TileRun find_run(const TileRun* __restrict__ runs, int nruns,
                                            int it) {
  int lo = 0, hi = nruns - 1;
  while (lo < hi) {
    int mid = (lo + hi + 1) >> 1;
    if (__builtin_amdgcn_readfirstlane(runs[mid].start) <= it)
      lo = mid;
    else
      hi = mid - 1;
  }
  TileRun r = runs[lo];
  r.view = __builtin_amdgcn_readfirstlane(r.view);
  r.tile0 = __builtin_amdgcn_readfirstlane(r.tile0);
  r.start = __builtin_amdgcn_readfirstlane(r.start);
  r.tiles_x = __builtin_amdgcn_readfirstlane(r.tiles_x);
  return r;
}

template <int TW, int TH, int PPT, int FEAT>
__device__ __forceinline__ void render_flat_tile(const ViewDev* __restrict__ views,
                                                 const TileRun* __restrict__ runs, int nruns,
                                                 int it, const TablesDev& T, const LutDev& L) {
  TileRun r = find_run(runs, nruns, it);
  int tile = r.tile0 + (it - r.start);
  // fields are read through the reference as they are needed (wave-uniform scalar loads):
  // a copy of the whole record would hold ~65 scalar registers across the tile
  const ViewDev& v = views[r.view];
  render_tile<TW, TH, PPT, false, (FEAT & kFeatParticles) != 0, false, kAreaOf<FEAT>>(
      v, T, L, (tile % r.tiles_x) * TW,
                                        (tile / r.tiles_x) * TH);
}

// Persistent launch over the tiles of many views.  Every wave works on its own and renders every
// 8x8 block of its tiles, so no tile waits on a barrier and the workgroup shape (4 waves) is the
// same for every tile configuration.  Wave j is dealt the tiles j, j + waves, ..., so that
// neighbouring tiles, which cost alike, go to different waves and no launch leaves waves without
// any.  Up to kDealtBlocks blocks a wave all tiles are dealt.  Beyond, where the sums of uneven
// tiles drift apart, the second half is claimed from an atomic counter, about kClaimBlocks blocks
// at a time: one address takes an atomic every 17 ns, which claims of all tiles ran into.  Tiles of
// 16 blocks are too coarse to deal more than half of.  A wave leaves at its first tile past the
// last; the counter only grows, so every wave reaches that exit.  us, all claimed (with single
// tiles at the end), all dealt, and so: 64 uneven views of 86 Mpixels 1340, 1480, 1240; 24 of 31
// Mpixels 625, 585, 585; 24 of 52 Mpixels 865, 862, 842; eight 1080p frames 372, 272, 277; one 176,
// 59, 63; one 512 x 512 frame 159, 40, 38.  Held to 7 resident waves per SIMD: the loop over tiles
// keeps ~14 more vector registers live than one tile does, so at 8 waves it would spill; with area
// code to 5, as the other launches are (at 7 it spilled 46; four 1599 x 899 nebula views, claimed,
// 1003 us and 727 at 5).  The host sizes the grid to the same.
constexpr int kBatchThreads = 256, kDealtBlocks = 64, kClaimBlocks = 16;

template <int FEAT>
constexpr int kBatchWaves = batch_waves(FEAT);

template <int TW, int TH, int PPT, int FEAT>
__global__ void __launch_bounds__(kBatchThreads, kBatchWaves<FEAT>)
    k_render_batch(const ViewDev* __restrict__ views, const TileRun* __restrict__ runs,
                   int nruns, int ntiles, int* __restrict__ counter, TablesDev T, LutDev L) {
  using C = TileCfg<TW, TH, 1>;
  constexpr int kBlocks = C::kBX * C::kBY;                // 8x8 blocks per tile
  const int lane = threadIdx.x & 63;
  const int q = lane >> 2;
  const int ox = 2 * (q & 3) + (lane & 1), oy = 2 * (q >> 2) + ((lane >> 1) & 1);
  const int waves = (int)(gridDim.x * (kBatchThreads / 64));
  constexpr int kClaim = kBlocks >= kClaimBlocks ? 1 : kClaimBlocks / kBlocks;  // tiles
  const int share = (ntiles + waves - 1) / waves;
  const bool claims = kBlocks >= kClaimBlocks || share * kBlocks > kDealtBlocks;
  const int dealt = claims ? max(ntiles / waves / 2, 1) : share;  // tiles a wave
  const int wave = __builtin_amdgcn_readfirstlane(
      (int)(blockIdx.x * (kBatchThreads / 64) + threadIdx.x / 64));
  for (int r = 0;; ++r) {
    int it0, it1;
    if (r < dealt) {
      it0 = r * waves + wave;
      it1 = it0 + 1;
    } else {
      if (!claims) break;
      int c = 0;
      if (lane == 0) c = atomicAdd(counter, 1);
      it0 = dealt * waves + __builtin_amdgcn_readfirstlane(c) * kClaim;
      it1 = min(it0 + kClaim, ntiles);
    }
    if (it0 >= ntiles) break;
#pragma unroll 1
    for (int it = it0; it < it1; ++it) {
      const TileRun run = find_run(runs, nruns, it);
      const int tile = run.tile0 + (it - run.start);
      const ViewDev& v = views[run.view];
      const int tx0 = (tile % run.tiles_x) * TW, ty0 = (tile / run.tiles_x) * TH;
#pragma unroll 1
      for (int blk = 0; blk < kBlocks; ++blk) {
        const int bx = tx0 + 8 * (blk % C::kBX), by = ty0 + 8 * (blk / C::kBX);
        if (bx >= v.width || by >= v.height) continue;    // block outside the image
        render_pixel<false, (FEAT & kFeatParticles) != 0, false, kAreaOf<FEAT>>(
            v, T, L, bx + ox, by + oy, nullptr);
      }
    }
  }
}

// Tiles of many views without persistence: one workgroup per flat tile index.  Chunks of
// kXChunk consecutive flat tiles (a row segment of one view) stay on one XCD and the chunks
// are dealt to the 8 XCDs in turn, as in the plain launch.
constexpr int kXChunk = kXBW * kXBH;

template <int TW, int TH, int PPT, int FEAT>
__global__ void __launch_bounds__((TW / 8) * (TH / 8) * 64 / PPT, kMinWaves<FEAT>)
    k_render_list(const ViewDev* __restrict__ views, const TileRun* __restrict__ runs,
                  int nruns, int ntiles, TablesDev T, LutDev L) {
  int b = blockIdx.x;
  int k = b >> 3;
  int it = (k / kXChunk) * (8 * kXChunk) + (b & 7) * kXChunk + k % kXChunk;
  if (it >= ntiles) return;
  render_flat_tile<TW, TH, PPT, FEAT>(views, runs, nruns, it, T, L);
}

__global__ void k_reset_counter(int* c) { *c = 0; }

// Measurement variant of the plain launch (16x16 tiles): marks the star-map texels that
// the footprints visit.
__global__ void __launch_bounds__(256)
    k_render_count(ViewDev v, TablesDev T, LutDev L, int tiles_x, int ntiles, CountBufs cnt) {
  int tile = blockIdx.x;
  if (tile >= ntiles) return;
  render_tile<16, 16, 1, true>(v, T, L, (tile % tiles_x) * 16, (tile / tiles_x) * 16, &cnt);
}

__global__ void k_popcount(const uint32_t* __restrict__ bits, int64_t n,
                           unsigned long long* __restrict__ total) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  unsigned c = i < n ? __popc(bits[i]) : 0u;
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
  if ((threadIdx.x & 63) == 0 && c) atomicAdd(total, (unsigned long long)c);
}

// TraceRay alone, for unit tests: rays = [u, delta, alpha, u_ic, u_oc].  TIMED also writes
// (retarded time 0, retarded time 1, m_0, m_1) per ray to out_time.
template <bool TIMED>
__global__ void k_trace_rays(TablesDev T, const float* __restrict__ rays, int64_t n,
                             float4* __restrict__ out, float4* __restrict__ out_time) {
  int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float* r = rays + 5 * i;
  float u = r[0], delta = r[1];
  float sd, cd;
  sincosf(delta, &sd, &cd);
  TraceOut t = trace_ray<TIMED>(T, u, delta, r[2], cd / sd, r[3], r[4]);
  bool cap = (t.bits & BH_CAPTURED_BIT) != 0;
  out[i] = make_float4(cap ? __builtin_inff() : t.dprime, t.ucr[0], t.ucr[1],
                       __uint_as_float(t.bits));
  if (TIMED)
    out_time[i] = make_float4(t.tret[0], t.tret[1], (float)t.mcr[0], (float)t.mcr[1]);
}

__global__ void __launch_bounds__(256)
    k_march_rays(const float* __restrict__ rays, int64_t n, int nsteps, float h,
                 float4* __restrict__ out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float* r = rays + 5 * i;
  float sd, cd;
  sincosf(r[1], &sd, &cd);
  // a radial beam (delta = 0 or pi) keeps a finite slope, as in the render path
  TraceOut t = march_ray(r[0], r[2], cd / fmaxf(sd, 1e-7f), r[3], r[4], nsteps, h);
  bool cap = (t.bits & BH_CAPTURED_BIT) != 0;
  out[i] = make_float4(cap ? __builtin_inff() : t.dprime, t.ucr[0], t.ucr[1],
                       __uint_as_float(t.bits));
}

// ---- scratch of the allocation-free batched launch -------------------------------------------
// Device memory of bh_render_batch_noalloc: the persistent form's claim counter (first 256
// bytes), then up to kNoAllocViews view records and as many tile runs.  A file-scope device
// array: each GPU the library runs on holds its own copy until the process ends, and every
// call on that GPU shares it (it keeps the last call's contents; the counter is reset by a
// kernel before each persistent launch).  In host code `scratch` only names the symbol: its
// device address comes from scratch_address(), once per device.
constexpr int kNoAllocViews = BH_NOALLOC_MAX_VIEWS;
constexpr size_t kNoAllocHead = 256;
constexpr size_t kNoAllocBytes =
    kNoAllocHead + (size_t)kNoAllocViews * (sizeof(ViewDev) + sizeof(TileRun));
static_assert(sizeof(ViewDev) % 16 == 0, "view records keep the tile runs 16-byte aligned");
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

// Address of `scratch` on the current device (call with that device current).
hipError_t scratch_address(void** p) {
  return hipGetSymbolAddress(p, HIP_SYMBOL(scratch));
}

// ---- host-side launchers ------------------------------------------------------------------

struct TileEntry {
  int tw, th, waves, ppt;
  // indexed by the features the views may use: kFeatParticles | kFeatArea | kFeatBands
  // (kFeatBands alone: band star maps without area maps)
  void (*plain[8])(const ViewDev&, const TablesDev&, const LutDev&, hipStream_t);
  void (*batch[8])(const ViewDev*, const TileRun*, int, int, int*, const TablesDev&,
                   const LutDev&, int grid, hipStream_t);
  void (*list[8])(const ViewDev*, const TileRun*, int, int, const TablesDev&, const LutDev&,
                  hipStream_t);
};

template <class Kernel>
struct FirstArgument;
template <class A, class... Rest>
struct FirstArgument<void (*)(A, Rest...)> {
  using type = A;
};

template <int TW, int TH, int PPT, int FEAT>
static void launch_plain(const ViewDev& v, const TablesDev& T, const LutDev& L, hipStream_t s) {
  using C = TileCfg<TW, TH, PPT>;
  using Kernel = decltype(&k_render<TW, TH, PPT, FEAT>);
  static_assert(std::is_same<typename FirstArgument<Kernel>::type, ViewDev>::value,
                "k_render reads its view again at the start of its arguments");
  int tiles_x = (v.width + TW - 1) / TW, tiles_y = (v.height + TH - 1) / TH;
  hipLaunchKernelGGL((k_render<TW, TH, PPT, FEAT>), dim3(xcd_grid(tiles_x, tiles_y)),
                     dim3(C::kThreads), 0, s, v, T, L, tiles_x, tiles_y);
}

template <int TW, int TH, int PPT, int FEAT>
static void launch_batch(const ViewDev* views, const TileRun* runs, int nruns, int ntiles,
                         int* counter, const TablesDev& T, const LutDev& L, int grid,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_reset_counter, dim3(1), dim3(1), 0, s, counter);
  hipLaunchKernelGGL((k_render_batch<TW, TH, PPT, FEAT>), dim3(grid), dim3(kBatchThreads), 0, s,
                     views, runs, nruns, ntiles, counter, T, L);
}

template <int TW, int TH, int PPT, int FEAT>
static void launch_list(const ViewDev* views, const TileRun* runs, int nruns, int ntiles,
                        const TablesDev& T, const LutDev& L, hipStream_t s) {
  using C = TileCfg<TW, TH, PPT>;
  int grid = (ntiles + 8 * kXChunk - 1) / (8 * kXChunk) * (8 * kXChunk);
  hipLaunchKernelGGL((k_render_list<TW, TH, PPT, FEAT>), dim3(grid), dim3(C::kThreads), 0, s,
                     views, runs, nruns, ntiles, T, L);
}

#define BH_FEATS(F, TW, TH, PPT)                                                          \
  {F<TW, TH, PPT, 0>, F<TW, TH, PPT, 1>, F<TW, TH, PPT, 2>, F<TW, TH, PPT, 3>,             \
   F<TW, TH, PPT, 4>, F<TW, TH, PPT, 5>, F<TW, TH, PPT, 6>, F<TW, TH, PPT, 7>}
#define BH_TILE(TW, TH, PPT)                                                                \
  {TW, TH, TileCfg<TW, TH, PPT>::kWaves, PPT, BH_FEATS(launch_plain, TW, TH, PPT),          \
   BH_FEATS(launch_batch, TW, TH, PPT), BH_FEATS(launch_list, TW, TH, PPT)}

static const TileEntry kTiles[] = {
    BH_TILE(16, 16, 1), BH_TILE(32, 8, 1), BH_TILE(16, 8, 1), BH_TILE(8, 8, 1),
    BH_TILE(32, 16, 2), BH_TILE(16, 16, 2), BH_TILE(32, 32, 4), BH_TILE(64, 16, 4),
};

int tile_config_count() { return (int)(sizeof(kTiles) / sizeof(kTiles[0])); }
void tile_config(int i, int* tw, int* th, int* waves, int* ppt) {
  *tw = kTiles[i].tw;
  *th = kTiles[i].th;
  *waves = kTiles[i].waves;
  *ppt = kTiles[i].ppt;
}

hipError_t launch_render(int cfg, const ViewDev& v, const TablesDev& T, const LutDev& L,
                         hipStream_t s) {
  kTiles[cfg].plain[view_features(v)](v, T, L, s);
  return hipGetLastError();
}

// persistent != 0: `grid` persistent workgroups, dealt and claiming tiles;
// otherwise one workgroup per tile.
hipError_t launch_render_batch(int cfg, int persistent, int feat, const ViewDev* views,
                               const TileRun* runs, int nruns, int ntiles, int* counter,
                               const TablesDev& T, const LutDev& L, int grid, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  const int a = feat & (kFeatParticles | kFeatArea | kFeatBands);
  if (persistent)
    kTiles[cfg].batch[a](views, runs, nruns, ntiles, counter, T, L, grid, s);
  else
    kTiles[cfg].list[a](views, runs, nruns, ntiles, T, L, s);
  return hipGetLastError();
}

hipError_t launch_render_count(const ViewDev& v, const TablesDev& T, const LutDev& L,
                               uint32_t* touched, int64_t words, unsigned long long* total,
                               unsigned long long* l2_bytes, hipStream_t s) {
  int tiles_x = (v.width + 15) / 16, ntiles = tiles_x * ((v.height + 15) / 16);
  hipLaunchKernelGGL(k_render_count, dim3(ntiles), dim3(256), 0, s, v, T, L, tiles_x, ntiles,
                     CountBufs{touched, l2_bytes});
  hipLaunchKernelGGL(k_popcount, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, s, touched,
                     words, total);
  return hipGetLastError();
}

hipError_t launch_render_march(const ViewDev& v, const LutDev& L, hipStream_t s) {
  int tiles_x = (v.width + 15) / 16, tiles_y = (v.height + 15) / 16;
  const dim3 grid(xcd_grid(tiles_x, tiles_y));
  if ((v.area.tex && v.area.bands) || (v.has_stars && v.stars.bands))
    hipLaunchKernelGGL(k_render_march<2>, grid, dim3(256), 0, s, v, L, tiles_x, tiles_y);
  else if (v.area.tex)
    hipLaunchKernelGGL(k_render_march<1>, grid, dim3(256), 0, s, v, L, tiles_x, tiles_y);
  else
    hipLaunchKernelGGL(k_render_march<0>, grid, dim3(256), 0, s, v, L, tiles_x, tiles_y);
  return hipGetLastError();
}

hipError_t launch_march_rays(const float* rays, int64_t n, int nsteps, float h, float4* out,
                             hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_march_rays, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, rays, n,
                     nsteps, h, out);
  return hipGetLastError();
}

hipError_t launch_trace_rays(const TablesDev& T, const float* rays, int64_t n, float4* out,
                             float4* out_time, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  dim3 grid((unsigned)((n + 255) / 256));
  if (out_time)
    hipLaunchKernelGGL(k_trace_rays<true>, grid, dim3(256), 0, s, T, rays, n, out, out_time);
  else
    hipLaunchKernelGGL(k_trace_rays<false>, grid, dim3(256), 0, s, T, rays, n, out, out_time);
  return hipGetLastError();
}

}  // namespace bh
