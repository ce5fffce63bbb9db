// Integration of one table column (precompute.hip): the photon orbit equation by RK4 in phi, in
// FP64 while |u - 2/3| < band and in Kahan-compensated FP32 elsewhere, in chunks of one precision.
#pragma once

namespace bh {

enum { kTabFP32 = 0, kTabBand = 1, kTabAll = 2 };

__device__ __forceinline__ double accel64(double u) { return 1.5 * u * u - u; }
__device__ __forceinline__ float accel32(float u) { return 1.5f * u * u - u; }

__device__ __forceinline__ void kahan_add(float& s, float& c, float x) {
  float y = x - c;
  float t = s + y;
  c = (t - s) - y;
  s = t;
}

// The serial part of a column: u and w = du/dphi by RK4, in FP64 or compensated FP32.  The
// regularised time is no part of this chain: its increments depend only on each step's
// start, so the reading wave forms them in parallel (tau_step).
struct Integrator {
  double e2;            // the column's conserved (du/dphi)^2 + u^2 (1 - u)
  double u, w;          // FP64 state (valid when in64)
  float uf, wf, cu, cw; // FP32 state, true value = uf - cu (Kahan)
  bool in64;
  int mode;
  double band;

  __device__ __forceinline__ bool want64(double uu) const {
    return mode == kTabAll || (mode == kTabBand && fabs(uu - 2.0 / 3.0) < band);
  }
  __device__ __forceinline__ void init(double u0, double w0) {
    u = u0;
    w = w0;
    uf = (float)u0;
    wf = (float)w0;
    cu = (float)((double)uf - u0);
    cw = (float)((double)wf - w0);
    in64 = want64(u0);
  }
  __device__ __forceinline__ double get_u() const {
    return in64 ? u : (double)uf - (double)cu;
  }
  __device__ __forceinline__ double get_w() const {
    return in64 ? w : (double)wf - (double)cw;
  }
  // the precision of the next step
  __device__ __forceinline__ void select() {
    const double uc = get_u();
    const bool w64 = want64(uc);
    if (w64 == in64) return;
    if (w64) {
      // entering the FP64 band: keep u and re-derive |du/dphi| from the exact invariant,
      // so FP32 rounding of e^2 is not amplified by the unstable orbit near u = 2/3
      const double wc = get_w();
      u = uc;
      const double w2 = e2 - uc * uc * (1.0 - uc);
      w = w2 > 0.0 ? copysign(sqrt(w2), wc) : 0.0;
    } else {
      uf = (float)u;
      cu = (float)((double)uf - u);
      wf = (float)w;
      cw = (float)((double)wf - w);
    }
    in64 = w64;
  }
  __device__ __forceinline__ void step64(double h) {
    double k1u = w, k1w = accel64(u);
    double k2u = w + 0.5 * h * k1w, k2w = accel64(u + 0.5 * h * k1u);
    double k3u = w + 0.5 * h * k2w, k3w = accel64(u + 0.5 * h * k2u);
    double k4u = w + h * k3w, k4w = accel64(u + h * k3u);
    u += h / 6.0 * (k1u + 2.0 * k2u + 2.0 * k3u + k4u);
    w += h / 6.0 * (k1w + 2.0 * k2w + 2.0 * k3w + k4w);
  }
  __device__ __forceinline__ void step32(float hf) {
    float k1u = wf, k1w = accel32(uf);
    float k2u = wf + 0.5f * hf * k1w, k2w = accel32(uf + 0.5f * hf * k1u);
    float k3u = wf + 0.5f * hf * k2w, k3w = accel32(uf + 0.5f * hf * k2u);
    float k4u = wf + hf * k3w, k4w = accel32(uf + hf * k3u);
    kahan_add(uf, cu, hf / 6.0f * (k1u + 2.0f * k2u + 2.0f * k3u + k4u));
    kahan_add(wf, cw, hf / 6.0f * (k1w + 2.0f * k2w + 2.0f * k3w + k4w));
  }
};

// Steps within which every column ends, at h = step / (1 + e).  Columns differ from mu by
// exp(-12.5) of it at the least (x = 0 and x = 1 of the Appendix A mapping, at every table size),
// and turn or fall in within 14.7 rad there; rows of U lie below 4 rad.  (A fixed limit of 4e6
// steps left the last rows of D unwritten for steps below 5e-6.)
__device__ __forceinline__ int column_steps(double h) { return (int)(20.0 / h) + 1; }

constexpr int kChunk = 256;

struct ChunkInfo {
  int n, first, in64, last;  // steps, index of the state before them, precision, last chunk
};
union State16 {
  float4 f;
  double d[2];
};

__device__ __forceinline__ void state_at(const float4& s, bool in64, double* u, double* w) {
  State16 x;
  x.f = s;
  *u = in64 ? x.d[0] : (double)x.f.x - (double)x.f.y;
  *w = in64 ? x.d[1] : (double)x.f.z - (double)x.f.w;
}

// A column ends where its last row is passed: kApsis at w <= 0, kHorizon at u >= 1, kPhi after
// `max_steps` steps or at u >= 1 (the ray has fallen in).
enum { kApsis = 0, kHorizon = 1, kPhi = 2 };

// a condition that is the same on every lane, as a scalar
__device__ __forceinline__ bool uniform(bool c) {
  return __builtin_amdgcn_readfirstlane((int)c) != 0;
}

// Wave 0: up to kChunk steps of one precision into st (st[0] = the state they start from).
// Steps go in blocks of kBlock, looked at once: u rises until w changes its sign, so a block in
// which w kept it and that ends inside its precision's range and before the column's end was
// inside all along; one that does not is taken back and stepped singly.  (Columns of U go on past
// the apsis, which may lie in the FP64 band with both ends of the block below it.)  Tests and
// branches after every step took more than half of the step: 2.05 against 0.96 ms for a 512 x 512
// set.
constexpr int kBlock = 8;

template <int END>
__device__ __forceinline__ ChunkInfo integrate_chunk(Integrator& I, double h, int done,
                                                     int max_steps, float4* st, float4* dump) {
  const int lane = threadIdx.x & 63;
  float4* dst = lane == 0 ? st : dump + lane;
  const int inc = lane == 0 ? 1 : 0;
  I.select();
  ChunkInfo c;
  c.first = done;
  c.in64 = uniform(I.in64);
  c.last = 0;
  const int most = min(kChunk, max_steps - done);
  int n = 0;
  if (c.in64) {
    const auto put = [&] {
      State16 x;
      x.d[0] = I.u;
      x.d[1] = I.w;
      *dst = x.f;
    };
    const auto ended = [&] { return END == kApsis ? !(I.w > 0.0) : !(I.u < 1.0); };
    const auto left = [&] {
      return I.mode == kTabBand && !(fabs(I.u - 2.0 / 3.0) < I.band);
    };
    put();
    while (n + kBlock <= most) {
      const double u0 = I.u, w0 = I.w;
#pragma unroll
      for (int q = 0; q < kBlock; ++q) {
        I.step64(h);
        dst += inc;
        put();
      }
      if (uniform(ended() || left())) {
        I.u = u0;
        I.w = w0;
        dst -= kBlock * inc;
        break;
      }
      n += kBlock;
    }
#pragma unroll 1
    while (n < most) {
      I.step64(h);
      ++n;
      dst += inc;
      put();
      if (uniform(ended())) {
        c.last = 1;
        break;
      }
      if (uniform(left())) break;
    }
  } else {
    const float hf = (float)h;
    const auto put = [&] { *dst = make_float4(I.uf, I.cu, I.wf, I.cw); };
    // u within a rounding of the FP64 band (never, when there is none) or of the end
    const float near_lo = I.mode == kTabBand ? (float)(2.0 / 3.0 - I.band) - 1e-6f : 2.0f;
    const float near_hi = I.mode == kTabBand ? (float)(2.0 / 3.0 + I.band) + 1e-6f : 2.0f;
    const auto near_band = [&] { return I.uf > near_lo && I.uf < near_hi; };
    const auto near_end = [&] {
      return END == kApsis ? !(I.wf - I.cw > 0.0f) : !(I.uf < 0.999999f);
    };
    put();
    while (n + kBlock <= most) {
      const float u0 = I.uf, w0 = I.wf, cu0 = I.cu, cw0 = I.cw;
#pragma unroll
      for (int q = 0; q < kBlock; ++q) {
        I.step32(hf);
        dst += inc;
        put();
      }
      // a block may not pass the whole band either (a narrow one, wide steps)
      const bool turned = END == kPhi && (w0 > 0.0f) != (I.wf > 0.0f);
      if (uniform(near_end() || near_band() || turned || (u0 <= near_lo) != (I.uf <= near_lo))) {
        I.uf = u0;
        I.wf = w0;
        I.cu = cu0;
        I.cw = cw0;
        dst -= kBlock * inc;
        break;
      }
      n += kBlock;
    }
#pragma unroll 1
    while (n < most) {
      I.step32(hf);
      ++n;
      dst += inc;
      put();
      if (uniform(near_end())) {
        if (END == kApsis || uniform(!(I.get_u() < 1.0))) {
          c.last = 1;
          break;
        }
      }
      if (uniform(near_band())) {
        if (uniform(I.want64(I.get_u()))) break;
      }
    }
  }
  c.n = n;
  if (done + n >= max_steps) c.last = 1;
  return c;
}

}  // namespace bh
