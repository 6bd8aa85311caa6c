// Generated by gen_me.py for g g -> t t~ + 1 g (3 gluons on the top line,
// 6 colour orderings, 32 helicity/polarisation states),
// per-ordering schedule, all orderings in one block. Do not edit.
#pragma once
#include "amp.h"
namespace mf {
// Colour- and polarisation-summed |M|^2 with g = 1 (argument meaning as in
// the shared-current schedule).
template <class R, class RK, class RG, class KG>
__device__ __forceinline__ R me_gg_m3_both(const V4<KG>* K, const V4<RG> (*E)[2], const Sp<R>* UB,
                                         const Sp<R>* VS, const V4<RK>& PTB, RK MTK) {
  const R MT = cvt<R>(MTK);
  RG G3;
  { const V4<KG> P = K[0] + K[1]; G3 = cvt<RG>(KG(-1.0) / mdot(P, P)); }
  RG G5;
  { const V4<KG> P = K[0] + K[2]; G5 = cvt<RG>(KG(-1.0) / mdot(P, P)); }
  RG G6;
  { const V4<KG> P = K[1] + K[2]; G6 = cvt<RG>(KG(-1.0) / mdot(P, P)); }
  RG G7;
  { const V4<KG> P = K[0] + K[1] + K[2]; G7 = cvt<RG>(KG(-1.0) / mdot(P, P)); }
  R IQ1;
  { const V4<KG> P = K[0]; IQ1 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  R IQ2;
  { const V4<KG> P = K[1]; IQ2 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  R IQ3;
  { const V4<KG> P = K[0] + K[1]; IQ3 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  R IQ4;
  { const V4<KG> P = K[2]; IQ4 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  R IQ5;
  { const V4<KG> P = K[0] + K[2]; IQ5 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  R IQ6;
  { const V4<KG> P = K[1] + K[2]; IQ6 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  const V4<RG> K0 = cvt4<RG>(K[0]);
  const V4<RG> K1 = cvt4<RG>(K[1]);
  const V4<RG> K2 = cvt4<RG>(K[2]);
  const V4<R> PB = cvt4<R>(PTB);
  R total = R(0.0);
  {
#pragma unroll 1
    for (int hg = 0; hg < 8; ++hg) {
      const V4<RG> E0 = ((hg >> 2) & 1) ? E[0][1] : E[0][0];
      const V4<RG> E1 = ((hg >> 1) & 1) ? E[1][1] : E[1][0];
      const V4<RG> E2 = ((hg >> 0) & 1) ? E[2][1] : E[2][0];
      C2<R> A0h0_0, A1h0_0;
      C2<R> A0h1_0, A1h1_0;
      C2<R> A0h0_1, A1h0_1;
      C2<R> A0h1_1, A1h1_1;
      C2<R> A0h0_2, A1h0_2;
      C2<R> A0h1_2, A1h1_2;
      C2<R> A0h0_3, A1h0_3;
      C2<R> A0h1_3, A1h1_3;
      C2<R> A0h0_4, A1h0_4;
      C2<R> A0h1_4, A1h1_4;
      C2<R> A0h0_5, A1h0_5;
      C2<R> A0h1_5, A1h1_5;
      {  // orderings (0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)
        V4<RG> J0 = E0; opaque4(J0);
        V4<RG> k0 = K0; opaque4(k0);
        V4<RG> J1 = E1; opaque4(J1);
        V4<RG> k1 = K1; opaque4(k1);
        V4<RG> J2 = E2; opaque4(J2);
        V4<RG> k2 = K2; opaque4(k2);
        V4<R> pb = PB; opaque4(pb);
        const V4<RG> J01 = G3 * (v3(J0, J1, k0, k1));
        const V4<RG> J12 = G6 * (v3(J1, J2, k1, k2));
        const V4<RG> p6 = k1 + k2;
        const V4<RG> p3 = k0 + k1;
        const V4<RG> J012 = G7 * (w4_sub(J0, J1, J2, v3_acc(J01, J2, p3, k2, v3(J0, J12, k0, p6))));
        const V4<RG> J02 = G5 * (v3(J0, J2, k0, k2));
        const V4<RG> J21 = RG(-1.0) * J12;
        const V4<RG> p5 = k0 + k2;
        const V4<RG> J021 = G7 * (w4_sub(J0, J2, J1, v3_acc(J02, J1, p5, k1, v3(J0, J21, k0, p6))));
        const V4<RG> J10 = RG(-1.0) * J01;
        const V4<RG> J102 = G7 * (w4_sub(J1, J0, J2, v3_acc(J10, J2, p3, k2, v3(J1, J02, k1, p5))));
        const V4<RG> J20 = RG(-1.0) * J02;
        Sp<R> Sh0_ = VS[0]; opaque_sp(Sh0_);
        const Sp<R> Sh0_2 = prop_neg(pb + k2, MT, IQ4, slash(J2, Sh0_));
        const Sp<R> Sh0_12 = prop_neg(pb + p6, MT, IQ6, slash_acc(J12, Sh0_, slash(J1, Sh0_2)));
        const Sp<R> Fh0_0 = slash_acc(J012, Sh0_, slash_acc(J01, Sh0_2, slash(J0, Sh0_12)));
        A0h0_0 = ubar_dot(UB[0], Fh0_0);
        A1h0_0 = ubar_dot(UB[1], Fh0_0);
        const Sp<R> Sh0_1 = prop_neg(pb + k1, MT, IQ2, slash(J1, Sh0_));
        const Sp<R> Sh0_21 = prop_neg(pb + p6, MT, IQ6, slash_acc(J21, Sh0_, slash(J2, Sh0_1)));
        const Sp<R> Fh0_1 = slash_acc(J021, Sh0_, slash_acc(J02, Sh0_1, slash(J0, Sh0_21)));
        A0h0_1 = ubar_dot(UB[0], Fh0_1);
        A1h0_1 = ubar_dot(UB[1], Fh0_1);
        const Sp<R> Sh0_02 = prop_neg(pb + p5, MT, IQ5, slash_acc(J02, Sh0_, slash(J0, Sh0_2)));
        const Sp<R> Fh0_2 = slash_acc(J102, Sh0_, slash_acc(J10, Sh0_2, slash(J1, Sh0_02)));
        A0h0_2 = ubar_dot(UB[0], Fh0_2);
        A1h0_2 = ubar_dot(UB[1], Fh0_2);
        const Sp<R> Sh0_0 = prop_neg(pb + k0, MT, IQ1, slash(J0, Sh0_));
        const Sp<R> Sh0_20 = prop_neg(pb + p5, MT, IQ5, slash_acc(J20, Sh0_, slash(J2, Sh0_0)));
        const Sp<R> Fh0_3 = slash_acc(J021, Sh0_, slash_acc(J12, Sh0_0, slash(J1, Sh0_20)));
        A0h0_3 = ubar_dot(UB[0], Fh0_3);
        A1h0_3 = ubar_dot(UB[1], Fh0_3);
        const Sp<R> Sh0_01 = prop_neg(pb + p3, MT, IQ3, slash_acc(J01, Sh0_, slash(J0, Sh0_1)));
        const Sp<R> Fh0_4 = slash_acc(J102, Sh0_, slash_acc(J20, Sh0_1, slash(J2, Sh0_01)));
        A0h0_4 = ubar_dot(UB[0], Fh0_4);
        A1h0_4 = ubar_dot(UB[1], Fh0_4);
        const Sp<R> Sh0_10 = prop_neg(pb + p3, MT, IQ3, slash_acc(J10, Sh0_, slash(J1, Sh0_0)));
        const Sp<R> Fh0_5 = slash_acc(J012, Sh0_, slash_acc(J21, Sh0_0, slash(J2, Sh0_10)));
        A0h0_5 = ubar_dot(UB[0], Fh0_5);
        A1h0_5 = ubar_dot(UB[1], Fh0_5);
        Sp<R> Sh1_ = VS[1]; opaque_sp(Sh1_);
        const Sp<R> Sh1_2 = prop_neg(pb + k2, MT, IQ4, slash(J2, Sh1_));
        const Sp<R> Sh1_12 = prop_neg(pb + p6, MT, IQ6, slash_acc(J12, Sh1_, slash(J1, Sh1_2)));
        const Sp<R> Fh1_0 = slash_acc(J012, Sh1_, slash_acc(J01, Sh1_2, slash(J0, Sh1_12)));
        A0h1_0 = ubar_dot(UB[0], Fh1_0);
        A1h1_0 = ubar_dot(UB[1], Fh1_0);
        const Sp<R> Sh1_1 = prop_neg(pb + k1, MT, IQ2, slash(J1, Sh1_));
        const Sp<R> Sh1_21 = prop_neg(pb + p6, MT, IQ6, slash_acc(J21, Sh1_, slash(J2, Sh1_1)));
        const Sp<R> Fh1_1 = slash_acc(J021, Sh1_, slash_acc(J02, Sh1_1, slash(J0, Sh1_21)));
        A0h1_1 = ubar_dot(UB[0], Fh1_1);
        A1h1_1 = ubar_dot(UB[1], Fh1_1);
        const Sp<R> Sh1_02 = prop_neg(pb + p5, MT, IQ5, slash_acc(J02, Sh1_, slash(J0, Sh1_2)));
        const Sp<R> Fh1_2 = slash_acc(J102, Sh1_, slash_acc(J10, Sh1_2, slash(J1, Sh1_02)));
        A0h1_2 = ubar_dot(UB[0], Fh1_2);
        A1h1_2 = ubar_dot(UB[1], Fh1_2);
        const Sp<R> Sh1_0 = prop_neg(pb + k0, MT, IQ1, slash(J0, Sh1_));
        const Sp<R> Sh1_20 = prop_neg(pb + p5, MT, IQ5, slash_acc(J20, Sh1_, slash(J2, Sh1_0)));
        const Sp<R> Fh1_3 = slash_acc(J021, Sh1_, slash_acc(J12, Sh1_0, slash(J1, Sh1_20)));
        A0h1_3 = ubar_dot(UB[0], Fh1_3);
        A1h1_3 = ubar_dot(UB[1], Fh1_3);
        const Sp<R> Sh1_01 = prop_neg(pb + p3, MT, IQ3, slash_acc(J01, Sh1_, slash(J0, Sh1_1)));
        const Sp<R> Fh1_4 = slash_acc(J102, Sh1_, slash_acc(J20, Sh1_1, slash(J2, Sh1_01)));
        A0h1_4 = ubar_dot(UB[0], Fh1_4);
        A1h1_4 = ubar_dot(UB[1], Fh1_4);
        const Sp<R> Sh1_10 = prop_neg(pb + p3, MT, IQ3, slash_acc(J10, Sh1_, slash(J1, Sh1_0)));
        const Sp<R> Fh1_5 = slash_acc(J012, Sh1_, slash_acc(J21, Sh1_0, slash(J2, Sh1_10)));
        A0h1_5 = ubar_dot(UB[0], Fh1_5);
        A1h1_5 = ubar_dot(UB[1], Fh1_5);
      }
      {
        R s = cre_dot(A0h0_0, A0h0_1);
        s = cre_dot_acc(A0h0_0, A0h0_2, s); s = cre_dot_acc(A0h0_1, A0h0_4, s); s = cre_dot_acc(A0h0_2, A0h0_3, s);
        s = cre_dot_acc(A0h0_3, A0h0_5, s); s = cre_dot_acc(A0h0_4, A0h0_5, s);
        total = total + R(-16.0) * s;
      }
      {
        R s = cre_dot(A0h0_0, A0h0_3);
        s = cre_dot_acc(A0h0_0, A0h0_4, s); s = cre_dot_acc(A0h0_1, A0h0_2, s); s = cre_dot_acc(A0h0_1, A0h0_5, s);
        s = cre_dot_acc(A0h0_2, A0h0_5, s); s = cre_dot_acc(A0h0_3, A0h0_4, s);
        total = total + R(2.0) * s;
      }
      {
        R s = cre_dot(A0h0_0, A0h0_5);
        s = cre_dot_acc(A0h0_1, A0h0_3, s); s = cre_dot_acc(A0h0_2, A0h0_4, s);
        total = total + R(20.0) * s;
      }
      {
        R s = cabs2(A0h0_0);
        s = cabs2_acc(A0h0_1, s); s = cabs2_acc(A0h0_2, s); s = cabs2_acc(A0h0_3, s);
        s = cabs2_acc(A0h0_4, s); s = cabs2_acc(A0h0_5, s);
        total = total + R(64.0) * s;
      }
      {
        R s = cre_dot(A1h0_0, A1h0_1);
        s = cre_dot_acc(A1h0_0, A1h0_2, s); s = cre_dot_acc(A1h0_1, A1h0_4, s); s = cre_dot_acc(A1h0_2, A1h0_3, s);
        s = cre_dot_acc(A1h0_3, A1h0_5, s); s = cre_dot_acc(A1h0_4, A1h0_5, s);
        total = total + R(-16.0) * s;
      }
      {
        R s = cre_dot(A1h0_0, A1h0_3);
        s = cre_dot_acc(A1h0_0, A1h0_4, s); s = cre_dot_acc(A1h0_1, A1h0_2, s); s = cre_dot_acc(A1h0_1, A1h0_5, s);
        s = cre_dot_acc(A1h0_2, A1h0_5, s); s = cre_dot_acc(A1h0_3, A1h0_4, s);
        total = total + R(2.0) * s;
      }
      {
        R s = cre_dot(A1h0_0, A1h0_5);
        s = cre_dot_acc(A1h0_1, A1h0_3, s); s = cre_dot_acc(A1h0_2, A1h0_4, s);
        total = total + R(20.0) * s;
      }
      {
        R s = cabs2(A1h0_0);
        s = cabs2_acc(A1h0_1, s); s = cabs2_acc(A1h0_2, s); s = cabs2_acc(A1h0_3, s);
        s = cabs2_acc(A1h0_4, s); s = cabs2_acc(A1h0_5, s);
        total = total + R(64.0) * s;
      }
      {
        R s = cre_dot(A0h1_0, A0h1_1);
        s = cre_dot_acc(A0h1_0, A0h1_2, s); s = cre_dot_acc(A0h1_1, A0h1_4, s); s = cre_dot_acc(A0h1_2, A0h1_3, s);
        s = cre_dot_acc(A0h1_3, A0h1_5, s); s = cre_dot_acc(A0h1_4, A0h1_5, s);
        total = total + R(-16.0) * s;
      }
      {
        R s = cre_dot(A0h1_0, A0h1_3);
        s = cre_dot_acc(A0h1_0, A0h1_4, s); s = cre_dot_acc(A0h1_1, A0h1_2, s); s = cre_dot_acc(A0h1_1, A0h1_5, s);
        s = cre_dot_acc(A0h1_2, A0h1_5, s); s = cre_dot_acc(A0h1_3, A0h1_4, s);
        total = total + R(2.0) * s;
      }
      {
        R s = cre_dot(A0h1_0, A0h1_5);
        s = cre_dot_acc(A0h1_1, A0h1_3, s); s = cre_dot_acc(A0h1_2, A0h1_4, s);
        total = total + R(20.0) * s;
      }
      {
        R s = cabs2(A0h1_0);
        s = cabs2_acc(A0h1_1, s); s = cabs2_acc(A0h1_2, s); s = cabs2_acc(A0h1_3, s);
        s = cabs2_acc(A0h1_4, s); s = cabs2_acc(A0h1_5, s);
        total = total + R(64.0) * s;
      }
      {
        R s = cre_dot(A1h1_0, A1h1_1);
        s = cre_dot_acc(A1h1_0, A1h1_2, s); s = cre_dot_acc(A1h1_1, A1h1_4, s); s = cre_dot_acc(A1h1_2, A1h1_3, s);
        s = cre_dot_acc(A1h1_3, A1h1_5, s); s = cre_dot_acc(A1h1_4, A1h1_5, s);
        total = total + R(-16.0) * s;
      }
      {
        R s = cre_dot(A1h1_0, A1h1_3);
        s = cre_dot_acc(A1h1_0, A1h1_4, s); s = cre_dot_acc(A1h1_1, A1h1_2, s); s = cre_dot_acc(A1h1_1, A1h1_5, s);
        s = cre_dot_acc(A1h1_2, A1h1_5, s); s = cre_dot_acc(A1h1_3, A1h1_4, s);
        total = total + R(2.0) * s;
      }
      {
        R s = cre_dot(A1h1_0, A1h1_5);
        s = cre_dot_acc(A1h1_1, A1h1_3, s); s = cre_dot_acc(A1h1_2, A1h1_4, s);
        total = total + R(20.0) * s;
      }
      {
        R s = cabs2(A1h1_0);
        s = cabs2_acc(A1h1_1, s); s = cabs2_acc(A1h1_2, s); s = cabs2_acc(A1h1_3, s);
        s = cabs2_acc(A1h1_4, s); s = cabs2_acc(A1h1_5, s);
        total = total + R(64.0) * s;
      }
    }
  }
  return total * R(1.0 / 9.0);
}
}  // namespace mf
