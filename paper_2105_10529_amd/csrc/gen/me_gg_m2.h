// Generated by gen_me.py for g g -> t t~ + 0 g (2 gluons on the top line,
// 2 colour orderings, 16 helicity/polarisation states). Do not edit.
#pragma once
#include "amp.h"
namespace mf {
constexpr int ME_M2_NF = 2;
constexpr double ME_M2_COLOUR_DEN = 3.0;
// Colour- and polarisation-summed |M|^2 with g = 1.
//   K[i]: outgoing gluon momenta (i = 0,1 the crossed beams), E[i][l]: the two
//   real polarisation vectors of gluon i; UB[l]: ubar(top) for the two top
//   helicities; VS[l]: v(antitop); PTB: antitop momentum; MT: top mass.
//   Per-event invariants and propagator factors are formed in the kinematic
//   type RK (FP64) and only then converted to the amplitude type R, so that
//   denominators such as (p_t + k)^2 - m^2 = 2 p_t.k + k^2 never cancel in R.
template <class R, class RK>
__device__ __forceinline__ R me_gg_m2(const V4<RK>* K, const V4<R> (*E)[2], const Sp<R>* UB,
                                         const Sp<R>* VS, const V4<RK>& PTB, RK MTK) {
  const R MT = cvt<R>(MTK);
  const V4<RK> PK1 = K[0];
  const V4<R> P1 = cvt4<R>(PK1);
  const V4<RK> PK2 = K[1];
  const V4<R> P2 = cvt4<R>(PK2);
  const V4<RK> PK3 = K[0] + K[1];
  const V4<R> P3 = cvt4<R>(PK3);
  const R G3 = cvt<R>(RK(-1.0) / mdot(PK3, PK3));
  const V4<R> Q1 = cvt4<R>(RK(-1.0) * (PTB + PK1));
  const R IQ1 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, PK1) + mdot(PK1, PK1)));
  const V4<R> Q2 = cvt4<R>(RK(-1.0) * (PTB + PK2));
  const R IQ2 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, PK2) + mdot(PK2, PK2)));
  R total = R(0.0);
#pragma unroll 1
  for (int ht = 0; ht < (fp64_amp<R>::value ? 1 : 2); ++ht) {
    const Sp<R> S_ = VS[ht];
#pragma unroll 1
    for (int hg = 0; hg < 4; ++hg) {
      const V4<R> J0 = ((hg >> 1) & 1) ? E[0][1] : E[0][0];
      const V4<R> J1 = ((hg >> 0) & 1) ? E[1][1] : E[1][0];
      const Sp<R> S_1 = prop(Q2, MT, IQ2, slash(J1, S_));
      const V4<R> J01 = G3 * (v3(J0, J1, P1, P2));
      const Sp<R> F0 = slash_acc(J01, S_, slash(J0, S_1));
      const C2<R> A0_0 = ubar_dot(UB[0], F0);
      const C2<R> A1_0 = ubar_dot(UB[1], F0);
      const Sp<R> S_0 = prop(Q1, MT, IQ1, slash(J0, S_));
      const V4<R> J10 = R(-1.0) * J01;
      const Sp<R> F1 = slash_acc(J10, S_, slash(J1, S_0));
      const C2<R> A0_1 = ubar_dot(UB[0], F1);
      const C2<R> A1_1 = ubar_dot(UB[1], F1);
      {
        R s = cre_dot(A0_0, A0_1);
        total = total + R(-4.0) * s;
      }
      {
        R s = cabs2(A0_0);
        s = cabs2_acc(A0_1, s);
        total = total + R(16.0) * s;
      }
      {
        R s = cre_dot(A1_0, A1_1);
        total = total + R(-4.0) * s;
      }
      {
        R s = cabs2(A1_0);
        s = cabs2_acc(A1_1, s);
        total = total + R(16.0) * s;
      }
    }
  }
  return total * R((fp64_amp<R>::value ? 2.0 : 1.0) / 3.0);
}
}  // namespace mf
