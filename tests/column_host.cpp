// The table columns' integration loop (bh_column.h) on the CPU, one lane.  Each scenario prints
// "<name> ok" or what it found.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_readfirstlane(x) (x)
struct float4 {
  float x, y, z, w;
};
static inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
static struct {
  unsigned x;
} threadIdx;
using std::min;

#include "bh_column.h"

using namespace bh;

static const double kMu = 4.0 / 27.0;

struct Run {
  long steps = 0;   // taken
  bool ended = false;
  double u = 0, w = 0;
  long wrong = 0;   // steps whose precision is not the one their start asks for
};

template <int END>
static Run run(double e2, double step, int mode, double band, int max_steps) {
  const double e = std::sqrt(e2), h = step / (1.0 + e);
  Integrator I;
  I.mode = mode;
  I.band = band;
  I.e2 = e2;
  I.init(0.0, e);
  std::vector<float4> st(kChunk + 1), dump(64);
  Run r;
  for (;;) {
    const ChunkInfo c = integrate_chunk<END>(I, h, (int)r.steps, max_steps, st.data(), dump.data());
    for (int k = 0; k < c.n; ++k) {
      double u, w;
      state_at(st[k], c.in64, &u, &w);
      if (mode == kTabBand && (std::fabs(u - 2.0 / 3.0) < band) != (c.in64 != 0)) ++r.wrong;
    }
    state_at(st[c.n], c.in64, &r.u, &r.w);
    r.steps += c.n;
    if (c.last) break;
  }
  r.ended = END == kApsis ? !(r.w > 0.0) : !(r.u < 1.0);
  return r;
}

// The longest columns of D, at every table size: mu (1 -+ exp(-12.5)) or nearly, to the apsis and
// to the horizon.  They end by themselves, inside the limit, for every step that is accepted.
static bool step_limit() {
  bool ok = true;
  const double far = -std::expm1(-12.5);
  for (int mode : {kTabFP32, kTabBand, kTabAll})
    for (double step : {0.05, 2e-3, 1e-5, 1e-6}) {
      if (mode == kTabAll && step < 1e-5) continue;
      for (int high = 0; high < 2; ++high) {
        const double e2 = high ? kMu / far : kMu * far, h = step / (1.0 + std::sqrt(e2));
        const int most = column_steps(h);
        const Run r = high ? run<kHorizon>(e2, step, mode, 0.05, most)
                           : run<kApsis>(e2, step, mode, 0.05, most);
        if (!r.ended || r.steps * h > 16.0) {
          std::printf("mode %d step %g high %d: %ld steps of %d, u %g w %g\n", mode, step, high,
                      r.steps, most, r.u, r.w);
          ok = false;
        }
      }
    }
  // the smallest accepted step: the limit and the step numbers fit an int
  const double h = 1e-7 / (1.0 + std::sqrt(kMu));
  if (!(column_steps(h) * h > 19.9 && 20.0 / h + 1 < 2147483647.0)) ok = false;
  return ok;
}

// Every step is taken in the precision that its start asks for, in columns of U too, whose u falls
// again past the apsis: apsides from just below the band's edge to well inside it, where the FP64
// steps are a few around the apsis.
static bool band_rule() {
  bool ok = true;
  long in_band = 0;
  for (double step : {5e-4, 2e-3, 1e-2, 0.05})
    for (double band : {1e-3, 0.05, 0.3})
      for (double above : {-1e-6, 3e-8, 3e-7, 3e-6, 1e-5, 1e-4, 3e-4}) {
        if (above >= band) continue;
        const double ua = 2.0 / 3.0 - band + above, e2 = ua * ua * (1.0 - ua);
        const double e = std::sqrt(e2), h = step / (1.0 + e);
        const double phi = 3.0 * (1.0 + e2) / (1.0 + 6.0 * e2 * e);
        const Run r = run<kPhi>(e2, step, kTabBand, band, (int)std::ceil(phi / h));
        if (r.wrong) {
          std::printf("step %g band %g apsis %g above its edge: %ld steps in the other precision\n",
                      step, band, above, r.wrong);
          ok = false;
        }
        in_band += above > 0;
      }
  return ok && in_band > 0;
}

int main(int argc, char** argv) {
  const char* name = argc > 1 ? argv[1] : "";
  bool ok = false;
  if (!std::strcmp(name, "step_limit")) ok = step_limit();
  if (!std::strcmp(name, "band_rule")) ok = band_rule();
  std::printf("%s %s\n", name, ok ? "ok" : "failed");
  return ok ? 0 : 1;
}
