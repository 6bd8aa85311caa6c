// Tree-level |M|^2 of the quark-initiated top-pair + jet channels (HIP,
// gfx950): q(p1) q~(p2) -> t t~ g(k) and q(p1) g(p2) -> t t~ q(k).
//
// Two fermion lines (the light quark line and the top line) joined by one
// gluon, with one more external gluon attached to either line or to the
// connecting gluon through the three-gluon vertex: five Feynman diagrams
// (Feynman gauge).  Their Lorentz parts K_d are built per helicity state from
// the chiral-basis spinors and vertex/propagator forms of amp.h and the
// vector currents psibar gamma^mu chi; their colour factors enter through the
// exact matrix CC[d][d'] = sum_colours C_d C_d'^* (gen/colour_qq.h), so that
// sum_colours |M|^2 = sum_{d,d'} K_d K_d'^* CC[d][d'] (the helicity loop and
// the colour aggregation of Sec. 2.2).  Row spinors times real vectors use
// psibar Jslash = dbar(Jslash psi), valid for real J.  Coupling g = 1.
#pragma once
#include "amp.h"
#include "gen/colour_qq.h"

namespace mf {

// Complex four-vector (contravariant components).
template <class R> struct CV4 {
  C2<R> c[4];
};
template <class R> __device__ __forceinline__ CV4<R> vcur(const Sp<R>& row, const Sp<R>& col) {
  // row gamma^mu col, gamma^mu = [[0, sigma^mu], [sigmabar^mu, 0]]
  CV4<R> j;
  j.c[0] = cmul(row.s0, col.s2) + cmul(row.s1, col.s3) + cmul(row.s2, col.s0) + cmul(row.s3, col.s1);
  j.c[1] = (cmul(row.s0, col.s3) + cmul(row.s1, col.s2)) - (cmul(row.s2, col.s1) + cmul(row.s3, col.s0));
  const C2<R> a = cmul(row.s1, col.s2) - cmul(row.s0, col.s3);
  const C2<R> b = cmul(row.s2, col.s1) - cmul(row.s3, col.s0);
  const C2<R> ab = a + b;
  j.c[2] = C2<R>{R(0.0) - ab.im, ab.re};
  j.c[3] = (cmul(row.s0, col.s2) - cmul(row.s1, col.s3)) - (cmul(row.s2, col.s0) - cmul(row.s3, col.s1));
  return j;
}
template <class R> __device__ __forceinline__ C2<R> mdotc(const CV4<R>& a, const CV4<R>& b) {
  return cmul(a.c[0], b.c[0]) - cmul(a.c[1], b.c[1]) - cmul(a.c[2], b.c[2]) - cmul(a.c[3], b.c[3]);
}
template <class R> __device__ __forceinline__ C2<R> mdotr(const V4<R>& a, const CV4<R>& b) {
  return C2<R>{a.t * b.c[0].re - a.x * b.c[1].re - a.y * b.c[2].re - a.z * b.c[3].re,
               a.t * b.c[0].im - a.x * b.c[1].im - a.y * b.c[2].im - a.z * b.c[3].im};
}
template <class R> __device__ __forceinline__ Sp<R> sbar(const Sp<R>& p) {
  // psi^dagger gamma^0 in the chiral basis
  return Sp<R>{C2<R>{p.s2.re, R(0.0) - p.s2.im}, C2<R>{p.s3.re, R(0.0) - p.s3.im},
               C2<R>{p.s0.re, R(0.0) - p.s0.im}, C2<R>{p.s1.re, R(0.0) - p.s1.im}};
}
template <class R> __device__ __forceinline__ C2<R> cscale(C2<R> a, R s) { return C2<R>{a.re * s, a.im * s}; }
// -i z
template <class R> __device__ __forceinline__ C2<R> mul_mi(C2<R> z) { return C2<R>{z.im, R(0.0) - z.re}; }

// Three-gluon vertex contracted with its legs (a: real polarisation e with
// incoming momentum k; b, c: currents X, Y with incoming momenta p, q):
//   (e.X)((k - p).Y) + (X.Y)((p - q).e) + (Y.e)((q - k).X)
template <class R>
__device__ __forceinline__ C2<R> vertex3(const V4<R>& e, const V4<R>& k, const CV4<R>& X, const V4<R>& p,
                                         const CV4<R>& Y, const V4<R>& q) {
  const C2<R> eX = mdotr(e, X), eY = mdotr(e, Y), XY = mdotc(X, Y);
  const C2<R> kpY = mdotr(k - p, Y), qkX = mdotr(q - k, X);
  const R pqe = mdot(p - q, e);
  return cmul(eX, kpY) + cscale(XY, pqe) + cmul(eY, qkX);
}

// sum_{d,d'} Re(K_d K_d'^* CC[d][d']) with the exact Hermitian matrix
// CC = (QQ_CC_RE + i QQ_CC_IM) / QQ_CC_DEN.
template <class R> __device__ __forceinline__ R colour_form5(const C2<R>* K) {
  R t = R(0.0);
#pragma unroll
  for (int d = 0; d < 5; ++d) {
    t = t + R(QQ_CC_RE[d * 5 + d]) * cabs2(K[d]);
#pragma unroll
    for (int e = d + 1; e < 5; ++e) {
      // 2 Re(K_d K_e^* CC[d][e])
      const C2<R> z = C2<R>{K[d].re * K[e].re + K[d].im * K[e].im, K[d].im * K[e].re - K[d].re * K[e].im};
      t = t + R(2.0) * (R(QQ_CC_RE[d * 5 + e]) * z.re - R(QQ_CC_IM[d * 5 + e]) * z.im);
    }
  }
  return t * R(1.0 / QQ_CC_DEN);
}

// slash(J) psi and row slash(J) for a complex four-vector (contravariant
// components).
template <class R> struct SlashC {
  C2<R> a, b, c, d;  // J0 - J3, J0 + J3, J1 - i J2, J1 + i J2
  __device__ __forceinline__ explicit SlashC(const CV4<R>& J)
      : a(J.c[0] - J.c[3]), b(J.c[0] + J.c[3]),
        c(C2<R>{J.c[1].re + J.c[2].im, J.c[1].im - J.c[2].re}),
        d(C2<R>{J.c[1].re - J.c[2].im, J.c[1].im + J.c[2].re}) {}
  __device__ __forceinline__ Sp<R> col(const Sp<R>& p) const {
    return Sp<R>{cmul(a, p.s2) - cmul(c, p.s3), cmul(b, p.s3) - cmul(d, p.s2), cmul(b, p.s0) + cmul(c, p.s1),
                 cmul(d, p.s0) + cmul(a, p.s1)};
  }
  __device__ __forceinline__ Sp<R> row(const Sp<R>& r) const {
    return Sp<R>{cmul(r.s2, b) + cmul(r.s3, d), cmul(r.s2, c) + cmul(r.s3, a), cmul(r.s0, a) - cmul(r.s1, d),
                 cmul(r.s1, b) - cmul(r.s0, c)};
  }
};

// Which helicities are summed.  The light quark is massless, so a helicity
// assignment of its line that does not conserve chirality contributes exact
// zeros: one helicity of the line fixes the other end.  And with real
// polarisation vectors flipping every helicity conjugates the four diagrams
// of the fermion lines and the three-gluon one up to a common sign each,
// opposite for the two (the factors -i of the former), under which the colour
// form with its real block and imaginary border is invariant; so the light
// helicity + stands for both and the sum is doubled: 8 of the 32 helicity
// states.  What depends on the light line alone is built once per
// polarisation, what depends on one end of the top line once per end, and the
// light current is applied to the top spinors once.  VALU-bound, FP64:
// q g -> t t~ q, two iterations of 1e6 events (1.7e6 kept), 6.17 -> 1.72 ms;
// u u~ -> t t~ g at 1e5 points 248 -> 38 us, its derivatives 1497 -> 322 us.
// The light current and the propagator next to it are applied to the top spinor
// before the polarisation, once per helicity, so that each polarisation costs
// a real contraction; and the two charge assignments of q g share the light
// line: 1.46 -> 1.29 ms, derivatives at 1e5 points 360 -> 253 us (q g) and 171
// -> 130 us (u u~ -> t t~ g).

// Sum over the top and antitop helicities and the polarisations E of the
// gluon.  X0, X1[pol]: the light current with the gluon on its incoming or
// other end, propagators included; JL: without it, times iL at the top line;
// a3, a4: momenta of the top propagators next to the top and the antitop, f3,
// f4 their factors; kg: the gluon's incoming momentum, qL that of JL, q34 the
// top pair's; i5: propagators of the three-gluon diagram.
template <class R>
__device__ __forceinline__ R top_line_sum(const CV4<R>* X0, const CV4<R>* X1, const CV4<R>& JL, R iL, const V4<R>* E,
                                          const V4<R>& pt, const V4<R>& ptb, R mt, const V4<R>& a3, R f3,
                                          const V4<R>& a4, R f4, const V4<R>& kg, const V4<R>& qL, const V4<R>& q34,
                                          R i5) {
  const V4<R> mq34 = R(0.0) * q34 - q34;
  const SlashC<R> sl(JL);
  R total = R(0.0);
#pragma unroll 1
  for (int h = 0; h < 4; ++h) {
    const int l3 = (h & 2) ? 1 : -1, l4 = (h & 1) ? 1 : -1;
    const Sp<R> ub3 = ubar_spinor(pt, mt, l3);
    const Sp<R> v4 = v_spinor(ptb, mt, l4);
    const CV4<R> J34 = vcur(ub3, v4);
    // the light current next to the antitop, then the propagator; next to the
    // top, then the propagator: what is left is linear in the polarisation
    const CV4<R> V2 = vcur(ub3, prop(a3, mt, f3, sl.col(v4)));
    const CV4<R> V3 = vcur(sbar(prop(a4, mt, f4, sbar(sl.row(ub3)))), v4);
#pragma unroll
    for (int pol = 0; pol < 2; ++pol) {
      const V4<R> e = E[pol];
      C2<R> K[5];
      // the gluon on the light line
      K[0] = mul_mi(mdotc(X0[pol], J34));
      K[1] = mul_mi(mdotc(X1[pol], J34));
      // next to the top, next to the antitop
      K[2] = mul_mi(cscale(mdotr(e, V2), iL));
      K[3] = mul_mi(cscale(mdotr(e, V3), iL));
      K[4] = cscale(vertex3(e, kg, JL, qL, J34, mq34), i5);
      total = total + colour_form5(K);
    }
  }
  return R(2.0) * total;
}
template <class R> __device__ __forceinline__ CV4<R> cvscale(const CV4<R>& a, R s) {
  return CV4<R>{{cscale(a.c[0], s), cscale(a.c[1], s), cscale(a.c[2], s), cscale(a.c[3], s)}};
}

// q(p1) q~(p2) -> t(pt) t~(ptb) g(k): colour- and helicity-summed |M|^2, g = 1.
template <class R>
__device__ __forceinline__ R me_qqbar_g(const V4<R>& p1, const V4<R>& p2, const V4<R>& pt, const V4<R>& ptb,
                                        const V4<R>& k, R mt) {
  const R z = R(0.0);
  const V4<R> q12 = p1 + p2, q34 = pt + ptb;
  const R s12 = mdot(q12, q12), s34 = mdot(q34, q34);
  const V4<R> a1 = p1 - k, a2 = k - p2, a3 = pt + k, a4 = z * k - (ptb + k);
  const R i1 = R(1.0) / (mdot(a1, a1) * s34), i2 = R(1.0) / (mdot(a2, a2) * s34);
  const R f3 = R(1.0) / (mdot(a3, a3) - mt * mt), f4 = R(1.0) / (mdot(a4, a4) - mt * mt);
  V4<R> E[2];
  lin_pols(k, E);
  const Sp<R> u1 = sbar(ubar_spinor(p1, z, 1)), v2 = v_spinor(p2, z, -1), vb2 = sbar(v2);
  CV4<R> X0[2], X1[2];
#pragma unroll
  for (int pol = 0; pol < 2; ++pol) {
    // emission from the incoming quark, from the incoming antiquark
    X0[pol] = cvscale(vcur(vb2, slash(a1, slash(E[pol], u1))), i1);
    X1[pol] = cvscale(vcur(sbar(slash(a2, slash(E[pol], v2))), u1), i2);
  }
  // three-gluon vertex: (e, -k), (J12, p1 + p2), (J34, -(pt + ptb))
  return top_line_sum(X0, X1, vcur(vb2, u1), R(1.0) / s12, E, pt, ptb, mt, a3, f3, a4, f4, z * k - k, q12, q34,
                      R(1.0) / (s12 * s34));
}

// q(p1) g(p2) -> t(pt) t~(ptb) q(k): colour- and helicity-summed |M|^2, g = 1;
// and in conj the same with the top and antitop momenta exchanged, which by
// charge conjugation is that of q~ g -> t t~ q~: the light line is the same.
template <class R>
__device__ __forceinline__ R me_qg_q(const V4<R>& p1, const V4<R>& p2, const V4<R>& pt, const V4<R>& ptb,
                                     const V4<R>& k, R mt, R& conj) {
  const R z = R(0.0);
  const V4<R> q12 = p1 + p2, q34 = pt + ptb, q15 = p1 - k;
  const R s12 = mdot(q12, q12), s34 = mdot(q34, q34), t15 = mdot(q15, q15);
  const V4<R> a2 = k - p2;
  const R i0 = R(1.0) / (s12 * s34), i2 = R(1.0) / (mdot(a2, a2) * s34);
  V4<R> E[2];
  lin_pols(p2, E);
  const Sp<R> u1 = sbar(ubar_spinor(p1, z, 1)), ub5 = ubar_spinor(k, z, 1), u5 = sbar(ub5);
  CV4<R> X0[2], X1[2];
#pragma unroll
  for (int pol = 0; pol < 2; ++pol) {
    // the gluon absorbed by the quark line before / after the top pair leaves it
    X0[pol] = cvscale(vcur(ub5, slash(q12, slash(E[pol], u1))), i0);
    X1[pol] = cvscale(vcur(sbar(slash(a2, slash(E[pol], u5))), u1), i2);
  }
  const CV4<R> J15 = vcur(ub5, u1);
  const R iL = R(1.0) / t15, i5 = R(1.0) / (t15 * s34);
  R r = z, rc = z;
#pragma unroll 1
  for (int cc = 0; cc < 2; ++cc) {
    const V4<R> a = cc ? ptb : pt, b = cc ? pt : ptb;
    const V4<R> a3 = a - p2, a4 = p2 - b;
    const R f3 = R(1.0) / (mdot(a3, a3) - mt * mt), f4 = R(1.0) / (mdot(a4, a4) - mt * mt);
    // three-gluon vertex: (e, p2), (J15, p1 - k), (J34, -(pt + ptb))
    const R t = top_line_sum(X0, X1, J15, iL, E, a, b, mt, a3, f3, a4, f4, p2, q15, q34, i5);
    r = cc ? r : t;
    rc = t;
  }
  conj = rc;
  return r;
}

}  // namespace mf
