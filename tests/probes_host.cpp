// Which face an area-source probe reads (bh_probes.h), on the CPU: probes exactly on cube edges and
// corners, where two or three components tie, and beside them, for centres on each face.
#include <cmath>
#include <cstdio>
#include <initializer_list>

#define __device__
#define __forceinline__ inline
static inline float fdiv(float a, float b) { return a * (1.0f / b); }

#include "bh_probes.h"

using namespace bh;

// axis argmax |p|, the lowest on ties
static int face_by_definition(const float* p) {
  int k = 0;
  for (int i = 1; i < 3; ++i)
    if (std::fabs(p[i]) > std::fabs(p[k])) k = i;
  return 2 * k + (p[k] < 0.0f);
}

int main() {
  long checked = 0, ties = 0, wrong = 0;
  const float step[] = {0.0f, 0.5f, -0.5f, 1.0f, -1.0f, 0.25f};
  for (int k = 0; k < 3; ++k)
    for (int sign = -1; sign <= 1; sign += 2)
      for (float a : {0.75f, -0.75f, 1.0f, 0.5f})
        for (float b : {0.75f, 1.0f, -1.0f, 0.0f})
          for (float jk : step)
            for (float ja : step)
              for (float jb : step) {
                AreaProbes P{};
                P.k = k;
                P.pk = (float)sign;
                P.pa = a;
                P.pb = b;
                P.face = 2 * k + (sign < 0);
                P.jk = jk;
                P.ja = ja;
                P.jb = jb;
                P.na = 0.5f;
                P.minor = 2;
                P.n = 8;
                P.inv = 0.25f;
                for (int i = 0; i < P.n; ++i) {
                  const float ta = ((float)(i >> 1) + 0.5f) * 0.25f - 0.5f;
                  const float tb = (i & 1) ? 0.25f : -0.25f;
                  float p[3];
                  p[k] = P.pk + ta * jk;
                  p[(k + 1) % 3] = P.pa + ta * ja + tb * P.na;
                  p[(k + 2) % 3] = P.pb + ta * jb;
                  const AreaAt at = area_at(P, i);
                  const int f = face_by_definition(p), kf = f / 2;
                  const float q[] = {std::fabs(p[0]), std::fabs(p[1]), std::fabs(p[2])};
                  ties += q[0] == q[1] || q[1] == q[2] || q[0] == q[2];
                  ++checked;
                  const float m = std::fabs(p[kf]);
                  if (at.face != f || std::fabs(at.u - p[(kf + 1) % 3] / m) > 1e-6f ||
                      std::fabs(at.v - p[(kf + 2) % 3] / m) > 1e-6f) {
                    if (wrong++ < 5)
                      std::printf("(%g, %g, %g), centre axis %d: face %d, not %d\n", p[0], p[1],
                                  p[2], k, at.face, f);
                  }
                }
              }
  std::printf("%ld probes, %ld ties, %ld wrong\n", checked, ties, wrong);
  return wrong != 0 || ties < 1000;
}
