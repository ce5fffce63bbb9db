// Table precompute on the GPU: integrate the photon orbit equation u'' = 3/2 u^2 - u
// (Section 3.3, eq. rayequation) for rays coming from infinity (u = 0, du/dphi = e) and
// record, at the Appendix A texel centres k/(N-1):
//   D(e, u)   = phi - atan2(u, du/dphi) on the incoming branch   (Algorithm 1, Precompute)
//   U(e, phi) = u for 0 <= phi < pi, 1 once the ray has fallen in (Section 3.3.3).
// Classic RK4 in phi, one e column per workgroup.  Precision: FP64 while
// |u - 2/3| < band (near the photon sphere, where the deflection diverges and errors grow
// exponentially with each turn), FP32 elsewhere with Kahan-compensated state updates.
// Values between steps come from cubic Hermite interpolation (u and du/dphi are both
// known at every step), in the variable that is smooth for each table half:
//   - D, e^2 < mu: in y = 1 - s with s = (du/dphi) / sqrt(u_a (u_2 - u)(u - u_3)), the
//     Appendix A row coordinate, which passes smoothly through the apsis (y = 1);
//   - D, e^2 > mu: u is monotone, so phi(u_j) is found by inverting the Hermite cubic;
//   - U: directly in phi.
// Time channels (Algorithm 1 Precompute also stores t, dt/dphi = e / (u^2 - u^3)): the
// time since infinity diverges, so the tables hold e tau with the regularised time
// tau = t - ln(u/(1-u)) + 1/u (+ const), whose rate is dtau/dphi = 1 / (e + du/dphi) on both
// branches (e - du/dphi = u^2 (1 - u) / (e + du/dphi) on a ray with invariant e^2).  tau is
// integrated with the same RK4 stages and read out with the same Hermite interpolation.
#include "bh_dev.h"

#include "bh_column.h"

namespace bh {

// Increment of the regularised time over the step that starts at (u, w): RK4 on
// dtau/dphi = 1 / (e + du/dphi), the stages of step64 and step32 formed again.
__device__ __forceinline__ double tau_step64(double e, double u, double w, double h) {
  double k1u = w, k1w = accel64(u);
  double k2u = w + 0.5 * h * k1w, k2w = accel64(u + 0.5 * h * k1u);
  double k3u = w + 0.5 * h * k2w, k3w = accel64(u + 0.5 * h * k2u);
  double k4u = w + h * k3w;
  return h / 6.0 * (1.0 / (e + k1u) + 2.0 / (e + k2u) + 2.0 / (e + k3u) + 1.0 / (e + k4u));
}
__device__ __forceinline__ float tau_step32(float ef, float uf, float wf, float hf) {
  float k1u = wf, k1w = accel32(uf);
  float k2u = wf + 0.5f * hf * k1w, k2w = accel32(uf + 0.5f * hf * k1u);
  float k3u = wf + 0.5f * hf * k2w, k3w = accel32(uf + 0.5f * hf * k2u);
  float k4u = wf + hf * k3w;
  return hf / 6.0f *
         (1.0f / (ef + k1u) + 2.0f / (ef + k2u) + 2.0f / (ef + k3u) + 1.0f / (ef + k4u));
}

__device__ __forceinline__ double hermite(double t, double f0, double d0, double f1, double d1,
                                          double hh) {
  double t2 = t * t, t3 = t2 * t;
  return (2 * t3 - 3 * t2 + 1) * f0 + (t3 - 2 * t2 + t) * hh * d0 + (-2 * t3 + 3 * t2) * f1 +
         (t3 - t2) * hh * d1;
}
__device__ __forceinline__ double hermite_dt(double t, double f0, double d0, double f1,
                                             double d1, double hh) {
  double t2 = t * t;
  return (6 * t2 - 6 * t) * f0 + (3 * t2 - 4 * t + 1) * hh * d0 + (-6 * t2 + 6 * t) * f1 +
         (3 * t2 - 2 * t) * hh * d1;
}

__device__ double d_col_e2(int n, int i) {
  double x = (double)i / (n - 1);
  if (i < n / 2) {
    double a = 0.5 - x;
    return -kMuD * expm1(-50.0 * a * a);
  }
  double a = x - 0.5;
  return kMuD / (-expm1(-50.0 * a * a));
}

// ---- one workgroup per column ------------------------------------------------------------
// A column is a serial chain of up to ~10^4 RK4 steps (the columns next to mu), and the chip
// has far more lanes than columns, so what counts is the length of one step's dependent
// chain.  Two waves share the column: wave 0 only integrates (u, w), every lane the same
// values (a wave of few active lanes issues each instruction several times slower than a full
// one), and writes the state after each step to LDS; wave 1 reads the chunk before it: the
// time increments (64 lanes, then a prefix sum in FP64) and one lane per table row, which
// finds its step by bisection.  One barrier per chunk.  512 x 512 with 64 x 32, FP64 band,
// with the download and 100 003 traced rays: 18.5 ms as one thread per column, integration
// and readout in turn, 0.96 ms so.
struct ColumnLds {
  float4 st[2][kChunk + 1];  // (uf, cu, wf, cw), or u and w in FP64
  float4 dump[64];           // where the copies of wave 0's other lanes go
  double val[kChunk + 1];    // the row coordinate after each step (y, or u)
  double tau[kChunk + 1];
  ChunkInfo info[2];
};

// orders this wave's LDS writes before its other lanes' reads
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
  __builtin_amdgcn_wave_barrier();
}

// Wave 1: tau after each step of the chunk (tau0 before the first); returns the last.
__device__ __forceinline__ double chunk_tau(const float4* st, const ChunkInfo& c, double e,
                                            double h, double tau0, double* tau) {
  constexpr int kPer = kChunk / 64;
  const int lane = threadIdx.x & 63;
  double inc[kPer], sum = 0.0;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int k = kPer * lane + q;
    inc[q] = 0.0;
    if (k < c.n) {
      State16 x;
      x.f = st[k];
      inc[q] = c.in64 ? tau_step64(e, x.d[0], x.d[1], h)
                      : (double)tau_step32((float)e, x.f.x, x.f.z, (float)h);
    }
    sum += inc[q];
    inc[q] = sum;
  }
  double before = sum;  // inclusive sum over the lanes below and this one
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double up = __shfl_up(before, o);
    if (lane >= o) before += up;
  }
  const double total = __shfl(before, 63);
  before += tau0 - sum;
  if (lane == 0) tau[0] = tau0;
#pragma unroll
  for (int q = 0; q < kPer; ++q)
    if (kPer * lane + q < c.n) tau[kPer * lane + q + 1] = before + inc[q];
  return tau0 + total;
}

// smallest k in [1, n] with val[k] >= v, given val[n] >= v
__device__ __forceinline__ int first_step(const double* val, int n, double v) {
  int lo = 1, hi = n;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (val[mid] >= v)
      hi = mid;
    else
      lo = mid + 1;
  }
  return lo;
}

struct TableOut {
  float* D;
  float* Dt;
  float* U;
  float* Ut;
  int n, ne, nphi;
};

// Wave 0's loop and the chunk hand-over; `read(chunk, states)` runs on wave 1 for each chunk
// in turn.  Both waves leave after the iteration that read the last chunk.
template <int END, class Read>
__device__ __forceinline__ void run_column(ColumnLds& L, Integrator& I, double h, int max_steps,
                                           Read read) {
  const bool integrates = threadIdx.x < 64;
  int done = 0;
  bool ended = false;  // wave 0: the chunk before this iteration was the last
  for (int c = 0;; ++c) {
    bool stop = false;
    if (integrates) {
      stop = ended;
      if (!ended) {
        const ChunkInfo ci =
            integrate_chunk<END>(I, h, done, max_steps, L.st[c & 1], L.dump);
        done += ci.n;
        ended = __builtin_amdgcn_readfirstlane(ci.last) != 0;
        if ((threadIdx.x & 63) == 0) L.info[c & 1] = ci;
      }
    } else if (c > 0) {
      ChunkInfo ci = L.info[(c - 1) & 1];
      ci.n = __builtin_amdgcn_readfirstlane(ci.n);
      ci.first = __builtin_amdgcn_readfirstlane(ci.first);
      ci.in64 = __builtin_amdgcn_readfirstlane(ci.in64);
      ci.last = __builtin_amdgcn_readfirstlane(ci.last);
      read(ci, L.st[(c - 1) & 1]);
      stop = ci.last != 0;
    }
    __syncthreads();
    if (stop) break;
  }
}

__device__ void column_D_low(ColumnLds& L, Integrator& I, const TableOut& O, int i, double e2,
                             double e, double h) {
  const int lane = threadIdx.x & 63, n = O.n;
  // roots u_a < u_2 of u^3 - u^2 + e^2 (u_3 < 0): closed form and sum/product of roots
  const double ua = 1.0 / 3.0 + 2.0 / 3.0 * sin(asin(fmin(2.0 * e2 / kMuD - 1.0, 1.0)) / 3.0);
  const double ssum = 1.0 - ua, prod = -e2 / ua;
  const double disc = sqrt(ssum * ssum - 4.0 * prod);
  const double u2 = 0.5 * (ssum + disc), u3 = 0.5 * (ssum - disc);
  int j0 = 1;
  double tau0 = 0.0;
  run_column<kApsis>(L, I, h, column_steps(h), [&](const ChunkInfo& c, const float4* st) {
    tau0 = chunk_tau(st, c, e, h, tau0, L.tau);
    for (int k = lane; k <= c.n; k += 64) {
      double u, w;
      state_at(st[k], c.in64, &u, &w);
      const double g = sqrt(fmax(ua * (u2 - u) * (u - u3), 1e-300));
      L.val[k] = c.first + k == 0 ? 0.0 : 1.0 - w / g;
    }
    wave_sync();
    const double yend = L.val[c.n];
    // D, its slope in y and the time's slope in y after step k
    auto at = [&](int k, double* f, double* d, double* dt) {
      double u, w;
      state_at(st[k], c.in64, &u, &w);
      const double g2 = ua * (u2 - u) * (u - u3), g = sqrt(fmax(g2, 1e-300));
      const double acc = accel64(u), gp = ua * (u2 + u3 - 2.0 * u) / (2.0 * g);
      const double dydphi = -(acc * g - w * w * gp) / g2;
      *f = (c.first + k) * h - atan2(u, w);
      *d = (1.0 - (w * w - u * acc) / (u * u + w * w)) / dydphi;
      *dt = (1.0 / (e + w)) / dydphi;
    };
    for (;;) {
      const int j = j0 + lane;
      const double yj = (double)j / (n - 1);
      const bool in = j < n && yj <= yend;
      if (in) {
        const int k = first_step(L.val, c.n, yj);
        double fp, dp, dtp, f, d, dt;
        at(k - 1, &fp, &dp, &dtp);
        at(k, &f, &d, &dt);
        const double yp = L.val[k - 1], hh = L.val[k] - yp;
        const double t = hh > 0.0 ? (yj - yp) / hh : 1.0;
        O.D[(size_t)j * n + i] = (float)hermite(t, fp, dp, f, d, hh);
        O.Dt[(size_t)j * n + i] =
            (float)(e * hermite(t, L.tau[k - 1], dtp, L.tau[k], dt, hh));
      }
      const int got = __popcll(__ballot(in));
      j0 += got;
      if (got < 64) break;
    }
    if (c.last) {  // rows past the step limit (not reached in practice)
      double f, d, dt;
      at(c.n, &f, &d, &dt);
      for (int j = j0 + lane; j < n; j += 64) {
        O.D[(size_t)j * n + i] = (float)f;
        O.Dt[(size_t)j * n + i] = (float)(e * L.tau[c.n]);
      }
    }
    wave_sync();  // the next chunk writes val and tau again
  });
}

__device__ void column_D_high(ColumnLds& L, Integrator& I, const TableOut& O, int i, double e2,
                              double e, double h) {
  const int lane = threadIdx.x & 63, n = O.n;
  const double a = sqrt(2.0 / 3.0), b = sqrt(1.0 / 3.0);
  int j0 = 1;
  double tau0 = 0.0;
  run_column<kHorizon>(L, I, h, column_steps(h), [&](const ChunkInfo& c, const float4* st) {
    tau0 = chunk_tau(st, c, e, h, tau0, L.tau);
    for (int k = lane; k <= c.n; k += 64) {
      double u, w;
      state_at(st[k], c.in64, &u, &w);
      L.val[k] = u;
    }
    wave_sync();
    const double uend = L.val[c.n];
    for (;;) {
      const int j = j0 + lane;
      const double z = (double)j / (n - 1) * (a + b) - a;
      double uj = 2.0 / 3.0 + (z >= 0 ? z * z : -z * z);
      if (j == n - 1) uj = 1.0;
      const bool in = j < n && uj <= uend;
      if (in) {
        const int k = first_step(L.val, c.n, uj);
        double up, wp, u, w;
        state_at(st[k - 1], c.in64, &up, &wp);
        state_at(st[k], c.in64, &u, &w);
        const double phi = (c.first + k) * h, phip = (c.first + k - 1) * h, hh = phi - phip;
        double t = (u > up) ? (uj - up) / (u - up) : 1.0;
        for (int it = 0; it < 8; ++it) {
          double r = hermite(t, up, wp, u, w, hh) - uj;
          double dr = hermite_dt(t, up, wp, u, w, hh);
          if (dr > 0.0) t -= r / dr;
          t = fmin(fmax(t, 0.0), 1.0);
        }
        double ph = phip + t * hh;
        double wj = sqrt(fmax(e2 - uj * uj * (1.0 - uj), 0.0));
        O.D[(size_t)j * n + i] = (float)(ph - atan2(uj, wj));
        O.Dt[(size_t)j * n + i] = (float)(e * hermite(t, L.tau[k - 1], 1.0 / (e + wp),
                                                      L.tau[k], 1.0 / (e + w), hh));
      }
      const int got = __popcll(__ballot(in));
      j0 += got;
      if (got < 64) break;
    }
    wave_sync();
  });
}

__device__ void column_U(ColumnLds& L, Integrator& I, const TableOut& O, int i, double e2,
                         double e, double h) {
  const int lane = threadIdx.x & 63, ne = O.ne, nphi = O.nphi;
  const double scale = 3.0 * (1.0 + e2) / (1.0 + 6.0 * e2 * e);  // phi_j = scale * y_j
  const double phi_last = scale * (double)(nphi - 1) / (nphi - 1);
  // steps to the first multiple of h at or past the last row
  const double want = ceil(phi_last / h);
  int steps = __builtin_amdgcn_readfirstlane(max((int)want, 1));
  if (uniform(steps * h < phi_last)) ++steps;
  int j0 = 1;
  double tau0 = 0.0;
  run_column<kPhi>(L, I, h, steps, [&](const ChunkInfo& c, const float4* st) {
    tau0 = chunk_tau(st, c, e, h, tau0, L.tau);
    wave_sync();
    for (;;) {
      const int j = j0 + lane;
      const double phij = scale * (double)j / (nphi - 1);
      const bool in = j < nphi && phij <= (c.first + c.n) * h;
      if (in) {
        int lo = 1, hi = c.n;  // first step whose phi reaches the row
        while (lo < hi) {
          const int mid = (lo + hi) >> 1;
          if ((c.first + mid) * h >= phij)
            hi = mid;
          else
            lo = mid + 1;
        }
        double up, wp, u, w;
        state_at(st[lo - 1], c.in64, &up, &wp);
        state_at(st[lo], c.in64, &u, &w);
        const double phi = (c.first + lo) * h, phip = (c.first + lo - 1) * h, hh = phi - phip;
        const double t = (phij - phip) / hh;
        const double v = hermite(t, up, wp, u, w, hh);
        O.U[(size_t)j * ne + i] = (float)fmin(fmax(v, 0.0), 1.0);
        O.Ut[(size_t)j * ne + i] = (float)(e * hermite(t, L.tau[lo - 1], 1.0 / (e + wp),
                                                       L.tau[lo], 1.0 / (e + w), hh));
      }
      const int got = __popcll(__ballot(in));
      j0 += got;
      if (got < 64) break;
    }
    double u, w;
    state_at(st[c.n], c.in64, &u, &w);
    if (c.last && u >= 1.0)  // fallen in: every later row
      for (int j = j0 + lane; j < nphi; j += 64) {
        O.U[(size_t)j * ne + i] = 1.0f;
        O.Ut[(size_t)j * ne + i] = 0.0f;
      }
    wave_sync();
  });
}

// Columns 0 .. n - 1 of D, then the ne columns of U, one workgroup each.
__global__ void __launch_bounds__(128)
    k_precompute(TableOut O, int mode, double band, double step) {
  __shared__ ColumnLds L;
  const int lane = threadIdx.x & 63;
  const bool reads = threadIdx.x >= 64;
  Integrator I;
  I.mode = mode;
  I.band = band;
  if ((int)blockIdx.x < O.n) {
    const int i = blockIdx.x;
    const double e2 = d_col_e2(O.n, i), e = sqrt(e2);
    if (reads && lane == 0) {
      O.D[i] = 0.0f;  // u = 0 at phi = 0: D = 0 - atan2(0, e)
      O.Dt[i] = 0.0f;
    }
    I.e2 = e2;
    I.init(0.0, e);
    if (i < O.n / 2)
      column_D_low(L, I, O, i, e2, e, step / (1.0 + e));
    else
      column_D_high(L, I, O, i, e2, e, step / (1.0 + e));
    return;
  }
  const int i = blockIdx.x - O.n, ne = O.ne, nphi = O.nphi;
  if (i == 0) {  // e -> infinity: u = e phi along phi = y / (2e), i.e. u = y / 2; e tau -> 0
    for (int j = threadIdx.x; j < nphi; j += 128) {
      O.U[(size_t)j * ne] = 0.5f * (float)j / (float)(nphi - 1);
      O.Ut[(size_t)j * ne] = 0.0f;
    }
    return;
  }
  if (i == ne - 1) {
    // e = 0: the ray stays at infinity (u = 0) along phi = 3y; e tau tends to tan(phi/2)
    // on a straight ray before its closest point (phi = pi/2), 2/sin(phi) - cot(phi/2) after
    for (int j = threadIdx.x; j < nphi; j += 128) {
      double phi = 3.0 * (double)j / (nphi - 1);
      O.U[(size_t)j * ne + i] = 0.0f;
      O.Ut[(size_t)j * ne + i] =
          (float)(phi <= 0.5 * M_PI ? tan(0.5 * phi) : 2.0 / sin(phi) - 1.0 / tan(0.5 * phi));
    }
    return;
  }
  const double x = (double)i / (ne - 1), e2 = (1.0 / x - 1.0) / 6.0, e = sqrt(e2);
  if (reads && lane == 0) {
    O.U[i] = 0.0f;
    O.Ut[i] = 0.0f;
  }
  I.e2 = e2;
  I.init(0.0, e);
  column_U(L, I, O, i, e2, e, step / (1.0 + e));
}

hipError_t launch_precompute(float* D, float* Dt, int d_n, float* U, float* Ut, int u_ne,
                             int u_nphi, int mode, double band, double step, hipStream_t s) {
  const TableOut O{D, Dt, U, Ut, d_n, u_ne, u_nphi};
  hipLaunchKernelGGL(k_precompute, dim3(d_n + u_ne), dim3(128), 0, s, O, mode, band, step);
  return hipGetLastError();
}

}  // namespace bh
