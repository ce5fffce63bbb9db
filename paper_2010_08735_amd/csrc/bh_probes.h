// Cube faces of directions, and where the probes of an area-source footprint read (render.hip).
#pragma once

namespace bh {

// Cube face of a direction: axis k = argmax |p_k| (the lowest on ties), face 2k + (p_k < 0);
// (pk, pa, pb) = (p_k, p_{(k+1)%3}, p_{(k+2)%3})
struct FaceOf {
  int k, face;
  float pk, pa, pb, m;  // m = |p_k|
};

__device__ __forceinline__ FaceOf face_of(float p0, float p1, float p2) {
  const float a0 = fabsf(p0), a1 = fabsf(p1), a2 = fabsf(p2);
  FaceOf f;
  f.k = 0;
  f.m = a0;
  if (a1 > f.m) { f.k = 1; f.m = a1; }
  if (a2 > f.m) { f.k = 2; f.m = a2; }
  f.pk = f.k == 0 ? p0 : (f.k == 1 ? p1 : p2);
  f.pa = f.k == 0 ? p1 : (f.k == 1 ? p2 : p0);
  f.pb = f.k == 0 ? p2 : (f.k == 1 ? p0 : p1);
  f.face = 2 * f.k + (f.pk < 0.0f);
  return f;
}

// The probes of a footprint, in the component order (k, k + 1, k + 2) of the face of d'
struct AreaProbes {
  int k, face;              // axis and face of d'
  bool one_face;            // every probe lies on that face
  float pk, pa, pb;         // d'
  float jk, ja, jb;         // major axis
  float nk, na, nb;         // minor axis
  int n, minor;             // number of probes, and along the minor axis (1 or 2)
  float inv;                // 1 / number along the major axis
};
struct AreaAt { int face; float u, v; };

// where probe i (i < n) reads: the minor axis runs fastest
__device__ __forceinline__ AreaAt area_at(const AreaProbes& P, int i) {
  const float ta = fmaf((float)(i >> (P.minor - 1)) + 0.5f, P.inv, -0.5f);
  const float tb = P.minor == 1 ? 0.0f : ((i & 1) ? 0.25f : -0.25f);
  const float pk = fmaf(tb, P.nk, fmaf(ta, P.jk, P.pk));
  const float pa = fmaf(tb, P.na, fmaf(ta, P.ja, P.pa));
  const float pb = fmaf(tb, P.nb, fmaf(ta, P.jb, P.pb));
  AreaAt at;
  float m = fabsf(pk), u = pa, v = pb;
  at.face = P.face;
  if (!P.one_face) {
    // the components in their own order again, in which a tie goes to the lowest axis
    const FaceOf f = face_of(P.k == 0 ? pk : (P.k == 1 ? pb : pa),
                             P.k == 0 ? pa : (P.k == 1 ? pk : pb),
                             P.k == 0 ? pb : (P.k == 1 ? pa : pk));
    at.face = f.face;
    m = f.m;
    u = f.pa;
    v = f.pb;
  }
  const float im = fdiv(1.0f, m);
  at.u = u * im;
  at.v = v * im;
  return at;
}

}  // namespace bh
