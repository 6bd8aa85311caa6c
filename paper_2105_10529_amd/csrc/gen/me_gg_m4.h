// Generated by gen_me.py for g g -> t t~ + 2 g (4 gluons on the top line,
// 24 colour orderings, 64 helicity/polarisation states),
// per-ordering schedule, orderings in pairs. Do not edit.
#pragma once
#include "amp.h"
namespace mf {
constexpr int ME_M4_NF = 24;
constexpr double ME_M4_COLOUR_DEN = 54.0;
// Colour- and polarisation-summed |M|^2 with g = 1 (argument meaning as in
// the shared-current schedule).
template <class R, class RK, class RG, class KG>
__device__ __forceinline__ R me_gg_m4(const V4<KG>* K, const V4<RG> (*E)[2], const Sp<R>* UB,
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
  RG G9;
  { const V4<KG> P = K[0] + K[3]; G9 = cvt<RG>(KG(-1.0) / mdot(P, P)); }
  RG G10;
  { const V4<KG> P = K[1] + K[3]; G10 = cvt<RG>(KG(-1.0) / mdot(P, P)); }
  RG G11;
  { const V4<KG> P = K[0] + K[1] + K[3]; G11 = cvt<RG>(KG(-1.0) / mdot(P, P)); }
  RG G12;
  { const V4<KG> P = K[2] + K[3]; G12 = cvt<RG>(KG(-1.0) / mdot(P, P)); }
  RG G13;
  { const V4<KG> P = K[0] + K[2] + K[3]; G13 = cvt<RG>(KG(-1.0) / mdot(P, P)); }
  RG G14;
  { const V4<KG> P = K[1] + K[2] + K[3]; G14 = cvt<RG>(KG(-1.0) / mdot(P, P)); }
  RG G15;
  { const V4<KG> P = K[0] + K[1] + K[2] + K[3]; G15 = cvt<RG>(KG(-1.0) / mdot(P, P)); }
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
  R IQ7;
  { const V4<KG> P = K[0] + K[1] + K[2]; IQ7 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  R IQ8;
  { const V4<KG> P = K[3]; IQ8 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  R IQ9;
  { const V4<KG> P = K[0] + K[3]; IQ9 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  R IQ10;
  { const V4<KG> P = K[1] + K[3]; IQ10 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  R IQ11;
  { const V4<KG> P = K[0] + K[1] + K[3]; IQ11 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  R IQ12;
  { const V4<KG> P = K[2] + K[3]; IQ12 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  R IQ13;
  { const V4<KG> P = K[0] + K[2] + K[3]; IQ13 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  R IQ14;
  { const V4<KG> P = K[1] + K[2] + K[3]; IQ14 = cvt<R>(RK(-1.0) / (RK(2.0) * mdot(PTB, P) + mdot(P, P))); }
  const V4<RG> K0 = cvt4<RG>(K[0]);
  const V4<RG> K1 = cvt4<RG>(K[1]);
  const V4<RG> K2 = cvt4<RG>(K[2]);
  const V4<RG> K3 = cvt4<RG>(K[3]);
  const V4<R> PB = cvt4<R>(PTB);
  R total = R(0.0);
  {
#pragma unroll 1
    for (int hg = 0; hg < 16; ++hg) {
      const V4<RG> E0 = ((hg >> 3) & 1) ? E[0][1] : E[0][0];
      const V4<RG> E1 = ((hg >> 2) & 1) ? E[1][1] : E[1][0];
      const V4<RG> E2 = ((hg >> 1) & 1) ? E[2][1] : E[2][0];
      const V4<RG> E3 = ((hg >> 0) & 1) ? E[3][1] : E[3][0];
      C2<R> A0h0_0, A1h0_0;
      C2<R> A0h0_6, A1h0_6;
      {  // orderings (0, 1, 2, 3), (1, 0, 2, 3)
        V4<RG> J0 = E0; opaque4(J0);
        V4<RG> k0 = K0; opaque4(k0);
        V4<RG> J1 = E1; opaque4(J1);
        V4<RG> k1 = K1; opaque4(k1);
        V4<RG> J2 = E2; opaque4(J2);
        V4<RG> k2 = K2; opaque4(k2);
        V4<RG> J3 = E3; opaque4(J3);
        V4<RG> k3 = K3; opaque4(k3);
        V4<R> pb = PB; opaque4(pb);
        const V4<RG> J01 = G3 * (v3(J0, J1, k0, k1));
        const V4<RG> J12 = G6 * (v3(J1, J2, k1, k2));
        const V4<RG> p6 = k1 + k2;
        const V4<RG> p3 = k0 + k1;
        const V4<RG> J012 = G7 * (w4_sub(J0, J1, J2, v3_acc(J01, J2, p3, k2, v3(J0, J12, k0, p6))));
        const V4<RG> J23 = G12 * (v3(J2, J3, k2, k3));
        const V4<RG> p12 = k2 + k3;
        const V4<RG> J123 = G14 * (w4_sub(J1, J2, J3, v3_acc(J12, J3, p6, k3, v3(J1, J23, k1, p12))));
        const V4<RG> p14 = k1 + k2 + k3;
        const V4<RG> p7 = k0 + k1 + k2;
        const V4<RG> J0123 = G15 * (w4_sub(J01, J2, J3, w4_sub(J0, J12, J3, w4_sub(J0, J1, J23, v3_acc(J012, J3, p7, k3, v3_acc(J01, J23, p3, p12, v3(J0, J123, k0, p14)))))));
        const V4<RG> J10 = RG(-1.0) * J01;
        const V4<RG> J02 = G5 * (v3(J0, J2, k0, k2));
        const V4<RG> p5 = k0 + k2;
        const V4<RG> J102 = G7 * (w4_sub(J1, J0, J2, v3_acc(J10, J2, p3, k2, v3(J1, J02, k1, p5))));
        const V4<RG> J023 = G13 * (w4_sub(J0, J2, J3, v3_acc(J02, J3, p5, k3, v3(J0, J23, k0, p12))));
        const V4<RG> p13 = k0 + k2 + k3;
        const V4<RG> J1023 = G15 * (w4_sub(J10, J2, J3, w4_sub(J1, J02, J3, w4_sub(J1, J0, J23, v3_acc(J102, J3, p7, k3, v3_acc(J10, J23, p3, p12, v3(J1, J023, k1, p13)))))));
        Sp<R> Sh0_ = VS[0]; opaque_sp(Sh0_);
        const Sp<R> Sh0_3 = prop_neg(pb + k3, MT, IQ8, slash(J3, Sh0_));
        const Sp<R> Sh0_23 = prop_neg(pb + p12, MT, IQ12, slash_acc(J23, Sh0_, slash(J2, Sh0_3)));
        const Sp<R> Sh0_123 = prop_neg(pb + p14, MT, IQ14, slash_acc(J123, Sh0_, slash_acc(J12, Sh0_3, slash(J1, Sh0_23))));
        const Sp<R> Fh0_0 = slash_acc(J0123, Sh0_, slash_acc(J012, Sh0_3, slash_acc(J01, Sh0_23, slash(J0, Sh0_123))));
        A0h0_0 = ubar_dot(UB[0], Fh0_0);
        A1h0_0 = ubar_dot(UB[1], Fh0_0);
        const Sp<R> Sh0_023 = prop_neg(pb + p13, MT, IQ13, slash_acc(J023, Sh0_, slash_acc(J02, Sh0_3, slash(J0, Sh0_23))));
        const Sp<R> Fh0_6 = slash_acc(J1023, Sh0_, slash_acc(J102, Sh0_3, slash_acc(J10, Sh0_23, slash(J1, Sh0_023))));
        A0h0_6 = ubar_dot(UB[0], Fh0_6);
        A1h0_6 = ubar_dot(UB[1], Fh0_6);
      }
      C2<R> A0h0_1, A1h0_1;
      C2<R> A0h0_7, A1h0_7;
      {  // orderings (0, 1, 3, 2), (1, 0, 3, 2)
        V4<RG> J0 = E0; opaque4(J0);
        V4<RG> k0 = K0; opaque4(k0);
        V4<RG> J1 = E1; opaque4(J1);
        V4<RG> k1 = K1; opaque4(k1);
        V4<RG> J2 = E2; opaque4(J2);
        V4<RG> k2 = K2; opaque4(k2);
        V4<RG> J3 = E3; opaque4(J3);
        V4<RG> k3 = K3; opaque4(k3);
        V4<R> pb = PB; opaque4(pb);
        const V4<RG> J01 = G3 * (v3(J0, J1, k0, k1));
        const V4<RG> J13 = G10 * (v3(J1, J3, k1, k3));
        const V4<RG> p10 = k1 + k3;
        const V4<RG> p3 = k0 + k1;
        const V4<RG> J013 = G11 * (w4_sub(J0, J1, J3, v3_acc(J01, J3, p3, k3, v3(J0, J13, k0, p10))));
        const V4<RG> J32 = G12 * (v3(J3, J2, k3, k2));
        const V4<RG> p12 = k2 + k3;
        const V4<RG> J132 = G14 * (w4_sub(J1, J3, J2, v3_acc(J13, J2, p10, k2, v3(J1, J32, k1, p12))));
        const V4<RG> p14 = k1 + k2 + k3;
        const V4<RG> p11 = k0 + k1 + k3;
        const V4<RG> J0132 = G15 * (w4_sub(J01, J3, J2, w4_sub(J0, J13, J2, w4_sub(J0, J1, J32, v3_acc(J013, J2, p11, k2, v3_acc(J01, J32, p3, p12, v3(J0, J132, k0, p14)))))));
        const V4<RG> J10 = RG(-1.0) * J01;
        const V4<RG> J03 = G9 * (v3(J0, J3, k0, k3));
        const V4<RG> p9 = k0 + k3;
        const V4<RG> J103 = G11 * (w4_sub(J1, J0, J3, v3_acc(J10, J3, p3, k3, v3(J1, J03, k1, p9))));
        const V4<RG> J032 = G13 * (w4_sub(J0, J3, J2, v3_acc(J03, J2, p9, k2, v3(J0, J32, k0, p12))));
        const V4<RG> p13 = k0 + k2 + k3;
        const V4<RG> J1032 = G15 * (w4_sub(J10, J3, J2, w4_sub(J1, J03, J2, w4_sub(J1, J0, J32, v3_acc(J103, J2, p11, k2, v3_acc(J10, J32, p3, p12, v3(J1, J032, k1, p13)))))));
        Sp<R> Sh0_ = VS[0]; opaque_sp(Sh0_);
        const Sp<R> Sh0_2 = prop_neg(pb + k2, MT, IQ4, slash(J2, Sh0_));
        const Sp<R> Sh0_32 = prop_neg(pb + p12, MT, IQ12, slash_acc(J32, Sh0_, slash(J3, Sh0_2)));
        const Sp<R> Sh0_132 = prop_neg(pb + p14, MT, IQ14, slash_acc(J132, Sh0_, slash_acc(J13, Sh0_2, slash(J1, Sh0_32))));
        const Sp<R> Fh0_1 = slash_acc(J0132, Sh0_, slash_acc(J013, Sh0_2, slash_acc(J01, Sh0_32, slash(J0, Sh0_132))));
        A0h0_1 = ubar_dot(UB[0], Fh0_1);
        A1h0_1 = ubar_dot(UB[1], Fh0_1);
        const Sp<R> Sh0_032 = prop_neg(pb + p13, MT, IQ13, slash_acc(J032, Sh0_, slash_acc(J03, Sh0_2, slash(J0, Sh0_32))));
        const Sp<R> Fh0_7 = slash_acc(J1032, Sh0_, slash_acc(J103, Sh0_2, slash_acc(J10, Sh0_32, slash(J1, Sh0_032))));
        A0h0_7 = ubar_dot(UB[0], Fh0_7);
        A1h0_7 = ubar_dot(UB[1], Fh0_7);
      }
      C2<R> A0h0_2, A1h0_2;
      C2<R> A0h0_12, A1h0_12;
      {  // orderings (0, 2, 1, 3), (2, 0, 1, 3)
        V4<RG> J0 = E0; opaque4(J0);
        V4<RG> k0 = K0; opaque4(k0);
        V4<RG> J1 = E1; opaque4(J1);
        V4<RG> k1 = K1; opaque4(k1);
        V4<RG> J2 = E2; opaque4(J2);
        V4<RG> k2 = K2; opaque4(k2);
        V4<RG> J3 = E3; opaque4(J3);
        V4<RG> k3 = K3; opaque4(k3);
        V4<R> pb = PB; opaque4(pb);
        const V4<RG> J02 = G5 * (v3(J0, J2, k0, k2));
        const V4<RG> J21 = G6 * (v3(J2, J1, k2, k1));
        const V4<RG> p6 = k1 + k2;
        const V4<RG> p5 = k0 + k2;
        const V4<RG> J021 = G7 * (w4_sub(J0, J2, J1, v3_acc(J02, J1, p5, k1, v3(J0, J21, k0, p6))));
        const V4<RG> J13 = G10 * (v3(J1, J3, k1, k3));
        const V4<RG> p10 = k1 + k3;
        const V4<RG> J213 = G14 * (w4_sub(J2, J1, J3, v3_acc(J21, J3, p6, k3, v3(J2, J13, k2, p10))));
        const V4<RG> p14 = k1 + k2 + k3;
        const V4<RG> p7 = k0 + k1 + k2;
        const V4<RG> J0213 = G15 * (w4_sub(J02, J1, J3, w4_sub(J0, J21, J3, w4_sub(J0, J2, J13, v3_acc(J021, J3, p7, k3, v3_acc(J02, J13, p5, p10, v3(J0, J213, k0, p14)))))));
        const V4<RG> J20 = RG(-1.0) * J02;
        const V4<RG> J01 = G3 * (v3(J0, J1, k0, k1));
        const V4<RG> p3 = k0 + k1;
        const V4<RG> J201 = G7 * (w4_sub(J2, J0, J1, v3_acc(J20, J1, p5, k1, v3(J2, J01, k2, p3))));
        const V4<RG> J013 = G11 * (w4_sub(J0, J1, J3, v3_acc(J01, J3, p3, k3, v3(J0, J13, k0, p10))));
        const V4<RG> p11 = k0 + k1 + k3;
        const V4<RG> J2013 = G15 * (w4_sub(J20, J1, J3, w4_sub(J2, J01, J3, w4_sub(J2, J0, J13, v3_acc(J201, J3, p7, k3, v3_acc(J20, J13, p5, p10, v3(J2, J013, k2, p11)))))));
        Sp<R> Sh0_ = VS[0]; opaque_sp(Sh0_);
        const Sp<R> Sh0_3 = prop_neg(pb + k3, MT, IQ8, slash(J3, Sh0_));
        const Sp<R> Sh0_13 = prop_neg(pb + p10, MT, IQ10, slash_acc(J13, Sh0_, slash(J1, Sh0_3)));
        const Sp<R> Sh0_213 = prop_neg(pb + p14, MT, IQ14, slash_acc(J213, Sh0_, slash_acc(J21, Sh0_3, slash(J2, Sh0_13))));
        const Sp<R> Fh0_2 = slash_acc(J0213, Sh0_, slash_acc(J021, Sh0_3, slash_acc(J02, Sh0_13, slash(J0, Sh0_213))));
        A0h0_2 = ubar_dot(UB[0], Fh0_2);
        A1h0_2 = ubar_dot(UB[1], Fh0_2);
        const Sp<R> Sh0_013 = prop_neg(pb + p11, MT, IQ11, slash_acc(J013, Sh0_, slash_acc(J01, Sh0_3, slash(J0, Sh0_13))));
        const Sp<R> Fh0_12 = slash_acc(J2013, Sh0_, slash_acc(J201, Sh0_3, slash_acc(J20, Sh0_13, slash(J2, Sh0_013))));
        A0h0_12 = ubar_dot(UB[0], Fh0_12);
        A1h0_12 = ubar_dot(UB[1], Fh0_12);
      }
      C2<R> A0h0_3, A1h0_3;
      C2<R> A0h0_13, A1h0_13;
      {  // orderings (0, 2, 3, 1), (2, 0, 3, 1)
        V4<RG> J0 = E0; opaque4(J0);
        V4<RG> k0 = K0; opaque4(k0);
        V4<RG> J1 = E1; opaque4(J1);
        V4<RG> k1 = K1; opaque4(k1);
        V4<RG> J2 = E2; opaque4(J2);
        V4<RG> k2 = K2; opaque4(k2);
        V4<RG> J3 = E3; opaque4(J3);
        V4<RG> k3 = K3; opaque4(k3);
        V4<R> pb = PB; opaque4(pb);
        const V4<RG> J02 = G5 * (v3(J0, J2, k0, k2));
        const V4<RG> J23 = G12 * (v3(J2, J3, k2, k3));
        const V4<RG> p12 = k2 + k3;
        const V4<RG> p5 = k0 + k2;
        const V4<RG> J023 = G13 * (w4_sub(J0, J2, J3, v3_acc(J02, J3, p5, k3, v3(J0, J23, k0, p12))));
        const V4<RG> J31 = G10 * (v3(J3, J1, k3, k1));
        const V4<RG> p10 = k1 + k3;
        const V4<RG> J231 = G14 * (w4_sub(J2, J3, J1, v3_acc(J23, J1, p12, k1, v3(J2, J31, k2, p10))));
        const V4<RG> p14 = k1 + k2 + k3;
        const V4<RG> p13 = k0 + k2 + k3;
        const V4<RG> J0231 = G15 * (w4_sub(J02, J3, J1, w4_sub(J0, J23, J1, w4_sub(J0, J2, J31, v3_acc(J023, J1, p13, k1, v3_acc(J02, J31, p5, p10, v3(J0, J231, k0, p14)))))));
        const V4<RG> J20 = RG(-1.0) * J02;
        const V4<RG> J03 = G9 * (v3(J0, J3, k0, k3));
        const V4<RG> p9 = k0 + k3;
        const V4<RG> J203 = G13 * (w4_sub(J2, J0, J3, v3_acc(J20, J3, p5, k3, v3(J2, J03, k2, p9))));
        const V4<RG> J031 = G11 * (w4_sub(J0, J3, J1, v3_acc(J03, J1, p9, k1, v3(J0, J31, k0, p10))));
        const V4<RG> p11 = k0 + k1 + k3;
        const V4<RG> J2031 = G15 * (w4_sub(J20, J3, J1, w4_sub(J2, J03, J1, w4_sub(J2, J0, J31, v3_acc(J203, J1, p13, k1, v3_acc(J20, J31, p5, p10, v3(J2, J031, k2, p11)))))));
        Sp<R> Sh0_ = VS[0]; opaque_sp(Sh0_);
        const Sp<R> Sh0_1 = prop_neg(pb + k1, MT, IQ2, slash(J1, Sh0_));
        const Sp<R> Sh0_31 = prop_neg(pb + p10, MT, IQ10, slash_acc(J31, Sh0_, slash(J3, Sh0_1)));
        const Sp<R> Sh0_231 = prop_neg(pb + p14, MT, IQ14, slash_acc(J231, Sh0_, slash_acc(J23, Sh0_1, slash(J2, Sh0_31))));
        const Sp<R> Fh0_3 = slash_acc(J0231, Sh0_, slash_acc(J023, Sh0_1, slash_acc(J02, Sh0_31, slash(J0, Sh0_231))));
        A0h0_3 = ubar_dot(UB[0], Fh0_3);
        A1h0_3 = ubar_dot(UB[1], Fh0_3);
        const Sp<R> Sh0_031 = prop_neg(pb + p11, MT, IQ11, slash_acc(J031, Sh0_, slash_acc(J03, Sh0_1, slash(J0, Sh0_31))));
        const Sp<R> Fh0_13 = slash_acc(J2031, Sh0_, slash_acc(J203, Sh0_1, slash_acc(J20, Sh0_31, slash(J2, Sh0_031))));
        A0h0_13 = ubar_dot(UB[0], Fh0_13);
        A1h0_13 = ubar_dot(UB[1], Fh0_13);
      }
      C2<R> A0h0_4, A1h0_4;
      C2<R> A0h0_18, A1h0_18;
      {  // orderings (0, 3, 1, 2), (3, 0, 1, 2)
        V4<RG> J0 = E0; opaque4(J0);
        V4<RG> k0 = K0; opaque4(k0);
        V4<RG> J1 = E1; opaque4(J1);
        V4<RG> k1 = K1; opaque4(k1);
        V4<RG> J2 = E2; opaque4(J2);
        V4<RG> k2 = K2; opaque4(k2);
        V4<RG> J3 = E3; opaque4(J3);
        V4<RG> k3 = K3; opaque4(k3);
        V4<R> pb = PB; opaque4(pb);
        const V4<RG> J03 = G9 * (v3(J0, J3, k0, k3));
        const V4<RG> J31 = G10 * (v3(J3, J1, k3, k1));
        const V4<RG> p10 = k1 + k3;
        const V4<RG> p9 = k0 + k3;
        const V4<RG> J031 = G11 * (w4_sub(J0, J3, J1, v3_acc(J03, J1, p9, k1, v3(J0, J31, k0, p10))));
        const V4<RG> J12 = G6 * (v3(J1, J2, k1, k2));
        const V4<RG> p6 = k1 + k2;
        const V4<RG> J312 = G14 * (w4_sub(J3, J1, J2, v3_acc(J31, J2, p10, k2, v3(J3, J12, k3, p6))));
        const V4<RG> p14 = k1 + k2 + k3;
        const V4<RG> p11 = k0 + k1 + k3;
        const V4<RG> J0312 = G15 * (w4_sub(J03, J1, J2, w4_sub(J0, J31, J2, w4_sub(J0, J3, J12, v3_acc(J031, J2, p11, k2, v3_acc(J03, J12, p9, p6, v3(J0, J312, k0, p14)))))));
        const V4<RG> J30 = RG(-1.0) * J03;
        const V4<RG> J01 = G3 * (v3(J0, J1, k0, k1));
        const V4<RG> p3 = k0 + k1;
        const V4<RG> J301 = G11 * (w4_sub(J3, J0, J1, v3_acc(J30, J1, p9, k1, v3(J3, J01, k3, p3))));
        const V4<RG> J012 = G7 * (w4_sub(J0, J1, J2, v3_acc(J01, J2, p3, k2, v3(J0, J12, k0, p6))));
        const V4<RG> p7 = k0 + k1 + k2;
        const V4<RG> J3012 = G15 * (w4_sub(J30, J1, J2, w4_sub(J3, J01, J2, w4_sub(J3, J0, J12, v3_acc(J301, J2, p11, k2, v3_acc(J30, J12, p9, p6, v3(J3, J012, k3, p7)))))));
        Sp<R> Sh0_ = VS[0]; opaque_sp(Sh0_);
        const Sp<R> Sh0_2 = prop_neg(pb + k2, MT, IQ4, slash(J2, Sh0_));
        const Sp<R> Sh0_12 = prop_neg(pb + p6, MT, IQ6, slash_acc(J12, Sh0_, slash(J1, Sh0_2)));
        const Sp<R> Sh0_312 = prop_neg(pb + p14, MT, IQ14, slash_acc(J312, Sh0_, slash_acc(J31, Sh0_2, slash(J3, Sh0_12))));
        const Sp<R> Fh0_4 = slash_acc(J0312, Sh0_, slash_acc(J031, Sh0_2, slash_acc(J03, Sh0_12, slash(J0, Sh0_312))));
        A0h0_4 = ubar_dot(UB[0], Fh0_4);
        A1h0_4 = ubar_dot(UB[1], Fh0_4);
        const Sp<R> Sh0_012 = prop_neg(pb + p7, MT, IQ7, slash_acc(J012, Sh0_, slash_acc(J01, Sh0_2, slash(J0, Sh0_12))));
        const Sp<R> Fh0_18 = slash_acc(J3012, Sh0_, slash_acc(J301, Sh0_2, slash_acc(J30, Sh0_12, slash(J3, Sh0_012))));
        A0h0_18 = ubar_dot(UB[0], Fh0_18);
        A1h0_18 = ubar_dot(UB[1], Fh0_18);
      }
      C2<R> A0h0_5, A1h0_5;
      C2<R> A0h0_19, A1h0_19;
      {  // orderings (0, 3, 2, 1), (3, 0, 2, 1)
        V4<RG> J0 = E0; opaque4(J0);
        V4<RG> k0 = K0; opaque4(k0);
        V4<RG> J1 = E1; opaque4(J1);
        V4<RG> k1 = K1; opaque4(k1);
        V4<RG> J2 = E2; opaque4(J2);
        V4<RG> k2 = K2; opaque4(k2);
        V4<RG> J3 = E3; opaque4(J3);
        V4<RG> k3 = K3; opaque4(k3);
        V4<R> pb = PB; opaque4(pb);
        const V4<RG> J03 = G9 * (v3(J0, J3, k0, k3));
        const V4<RG> J32 = G12 * (v3(J3, J2, k3, k2));
        const V4<RG> p12 = k2 + k3;
        const V4<RG> p9 = k0 + k3;
        const V4<RG> J032 = G13 * (w4_sub(J0, J3, J2, v3_acc(J03, J2, p9, k2, v3(J0, J32, k0, p12))));
        const V4<RG> J21 = G6 * (v3(J2, J1, k2, k1));
        const V4<RG> p6 = k1 + k2;
        const V4<RG> J321 = G14 * (w4_sub(J3, J2, J1, v3_acc(J32, J1, p12, k1, v3(J3, J21, k3, p6))));
        const V4<RG> p14 = k1 + k2 + k3;
        const V4<RG> p13 = k0 + k2 + k3;
        const V4<RG> J0321 = G15 * (w4_sub(J03, J2, J1, w4_sub(J0, J32, J1, w4_sub(J0, J3, J21, v3_acc(J032, J1, p13, k1, v3_acc(J03, J21, p9, p6, v3(J0, J321, k0, p14)))))));
        const V4<RG> J30 = RG(-1.0) * J03;
        const V4<RG> J02 = G5 * (v3(J0, J2, k0, k2));
        const V4<RG> p5 = k0 + k2;
        const V4<RG> J302 = G13 * (w4_sub(J3, J0, J2, v3_acc(J30, J2, p9, k2, v3(J3, J02, k3, p5))));
        const V4<RG> J021 = G7 * (w4_sub(J0, J2, J1, v3_acc(J02, J1, p5, k1, v3(J0, J21, k0, p6))));
        const V4<RG> p7 = k0 + k1 + k2;
        const V4<RG> J3021 = G15 * (w4_sub(J30, J2, J1, w4_sub(J3, J02, J1, w4_sub(J3, J0, J21, v3_acc(J302, J1, p13, k1, v3_acc(J30, J21, p9, p6, v3(J3, J021, k3, p7)))))));
        Sp<R> Sh0_ = VS[0]; opaque_sp(Sh0_);
        const Sp<R> Sh0_1 = prop_neg(pb + k1, MT, IQ2, slash(J1, Sh0_));
        const Sp<R> Sh0_21 = prop_neg(pb + p6, MT, IQ6, slash_acc(J21, Sh0_, slash(J2, Sh0_1)));
        const Sp<R> Sh0_321 = prop_neg(pb + p14, MT, IQ14, slash_acc(J321, Sh0_, slash_acc(J32, Sh0_1, slash(J3, Sh0_21))));
        const Sp<R> Fh0_5 = slash_acc(J0321, Sh0_, slash_acc(J032, Sh0_1, slash_acc(J03, Sh0_21, slash(J0, Sh0_321))));
        A0h0_5 = ubar_dot(UB[0], Fh0_5);
        A1h0_5 = ubar_dot(UB[1], Fh0_5);
        const Sp<R> Sh0_021 = prop_neg(pb + p7, MT, IQ7, slash_acc(J021, Sh0_, slash_acc(J02, Sh0_1, slash(J0, Sh0_21))));
        const Sp<R> Fh0_19 = slash_acc(J3021, Sh0_, slash_acc(J302, Sh0_1, slash_acc(J30, Sh0_21, slash(J3, Sh0_021))));
        A0h0_19 = ubar_dot(UB[0], Fh0_19);
        A1h0_19 = ubar_dot(UB[1], Fh0_19);
      }
      C2<R> A0h0_8, A1h0_8;
      C2<R> A0h0_14, A1h0_14;
      {  // orderings (1, 2, 0, 3), (2, 1, 0, 3)
        V4<RG> J0 = E0; opaque4(J0);
        V4<RG> k0 = K0; opaque4(k0);
        V4<RG> J1 = E1; opaque4(J1);
        V4<RG> k1 = K1; opaque4(k1);
        V4<RG> J2 = E2; opaque4(J2);
        V4<RG> k2 = K2; opaque4(k2);
        V4<RG> J3 = E3; opaque4(J3);
        V4<RG> k3 = K3; opaque4(k3);
        V4<R> pb = PB; opaque4(pb);
        const V4<RG> J12 = G6 * (v3(J1, J2, k1, k2));
        const V4<RG> J20 = G5 * (v3(J2, J0, k2, k0));
        const V4<RG> p5 = k0 + k2;
        const V4<RG> p6 = k1 + k2;
        const V4<RG> J120 = G7 * (w4_sub(J1, J2, J0, v3_acc(J12, J0, p6, k0, v3(J1, J20, k1, p5))));
        const V4<RG> J03 = G9 * (v3(J0, J3, k0, k3));
        const V4<RG> p9 = k0 + k3;
        const V4<RG> J203 = G13 * (w4_sub(J2, J0, J3, v3_acc(J20, J3, p5, k3, v3(J2, J03, k2, p9))));
        const V4<RG> p13 = k0 + k2 + k3;
        const V4<RG> p7 = k0 + k1 + k2;
        const V4<RG> J1203 = G15 * (w4_sub(J12, J0, J3, w4_sub(J1, J20, J3, w4_sub(J1, J2, J03, v3_acc(J120, J3, p7, k3, v3_acc(J12, J03, p6, p9, v3(J1, J203, k1, p13)))))));
        const V4<RG> J21 = RG(-1.0) * J12;
        const V4<RG> J10 = G3 * (v3(J1, J0, k1, k0));
        const V4<RG> p3 = k0 + k1;
        const V4<RG> J210 = G7 * (w4_sub(J2, J1, J0, v3_acc(J21, J0, p6, k0, v3(J2, J10, k2, p3))));
        const V4<RG> J103 = G11 * (w4_sub(J1, J0, J3, v3_acc(J10, J3, p3, k3, v3(J1, J03, k1, p9))));
        const V4<RG> p11 = k0 + k1 + k3;
        const V4<RG> J2103 = G15 * (w4_sub(J21, J0, J3, w4_sub(J2, J10, J3, w4_sub(J2, J1, J03, v3_acc(J210, J3, p7, k3, v3_acc(J21, J03, p6, p9, v3(J2, J103, k2, p11)))))));
        Sp<R> Sh0_ = VS[0]; opaque_sp(Sh0_);
        const Sp<R> Sh0_3 = prop_neg(pb + k3, MT, IQ8, slash(J3, Sh0_));
        const Sp<R> Sh0_03 = prop_neg(pb + p9, MT, IQ9, slash_acc(J03, Sh0_, slash(J0, Sh0_3)));
        const Sp<R> Sh0_203 = prop_neg(pb + p13, MT, IQ13, slash_acc(J203, Sh0_, slash_acc(J20, Sh0_3, slash(J2, Sh0_03))));
        const Sp<R> Fh0_8 = slash_acc(J1203, Sh0_, slash_acc(J120, Sh0_3, slash_acc(J12, Sh0_03, slash(J1, Sh0_203))));
        A0h0_8 = ubar_dot(UB[0], Fh0_8);
        A1h0_8 = ubar_dot(UB[1], Fh0_8);
        const Sp<R> Sh0_103 = prop_neg(pb + p11, MT, IQ11, slash_acc(J103, Sh0_, slash_acc(J10, Sh0_3, slash(J1, Sh0_03))));
        const Sp<R> Fh0_14 = slash_acc(J2103, Sh0_, slash_acc(J210, Sh0_3, slash_acc(J21, Sh0_03, slash(J2, Sh0_103))));
        A0h0_14 = ubar_dot(UB[0], Fh0_14);
        A1h0_14 = ubar_dot(UB[1], Fh0_14);
      }
      C2<R> A0h0_9, A1h0_9;
      C2<R> A0h0_15, A1h0_15;
      {  // orderings (1, 2, 3, 0), (2, 1, 3, 0)
        V4<RG> J0 = E0; opaque4(J0);
        V4<RG> k0 = K0; opaque4(k0);
        V4<RG> J1 = E1; opaque4(J1);
        V4<RG> k1 = K1; opaque4(k1);
        V4<RG> J2 = E2; opaque4(J2);
        V4<RG> k2 = K2; opaque4(k2);
        V4<RG> J3 = E3; opaque4(J3);
        V4<RG> k3 = K3; opaque4(k3);
        V4<R> pb = PB; opaque4(pb);
        const V4<RG> J12 = G6 * (v3(J1, J2, k1, k2));
        const V4<RG> J23 = G12 * (v3(J2, J3, k2, k3));
        const V4<RG> p12 = k2 + k3;
        const V4<RG> p6 = k1 + k2;
        const V4<RG> J123 = G14 * (w4_sub(J1, J2, J3, v3_acc(J12, J3, p6, k3, v3(J1, J23, k1, p12))));
        const V4<RG> J30 = G9 * (v3(J3, J0, k3, k0));
        const V4<RG> p9 = k0 + k3;
        const V4<RG> J230 = G13 * (w4_sub(J2, J3, J0, v3_acc(J23, J0, p12, k0, v3(J2, J30, k2, p9))));
        const V4<RG> p13 = k0 + k2 + k3;
        const V4<RG> p14 = k1 + k2 + k3;
        const V4<RG> J1230 = G15 * (w4_sub(J12, J3, J0, w4_sub(J1, J23, J0, w4_sub(J1, J2, J30, v3_acc(J123, J0, p14, k0, v3_acc(J12, J30, p6, p9, v3(J1, J230, k1, p13)))))));
        const V4<RG> J21 = RG(-1.0) * J12;
        const V4<RG> J13 = G10 * (v3(J1, J3, k1, k3));
        const V4<RG> p10 = k1 + k3;
        const V4<RG> J213 = G14 * (w4_sub(J2, J1, J3, v3_acc(J21, J3, p6, k3, v3(J2, J13, k2, p10))));
        const V4<RG> J130 = G11 * (w4_sub(J1, J3, J0, v3_acc(J13, J0, p10, k0, v3(J1, J30, k1, p9))));
        const V4<RG> p11 = k0 + k1 + k3;
        const V4<RG> J2130 = G15 * (w4_sub(J21, J3, J0, w4_sub(J2, J13, J0, w4_sub(J2, J1, J30, v3_acc(J213, J0, p14, k0, v3_acc(J21, J30, p6, p9, v3(J2, J130, k2, p11)))))));
        Sp<R> Sh0_ = VS[0]; opaque_sp(Sh0_);
        const Sp<R> Sh0_0 = prop_neg(pb + k0, MT, IQ1, slash(J0, Sh0_));
        const Sp<R> Sh0_30 = prop_neg(pb + p9, MT, IQ9, slash_acc(J30, Sh0_, slash(J3, Sh0_0)));
        const Sp<R> Sh0_230 = prop_neg(pb + p13, MT, IQ13, slash_acc(J230, Sh0_, slash_acc(J23, Sh0_0, slash(J2, Sh0_30))));
        const Sp<R> Fh0_9 = slash_acc(J1230, Sh0_, slash_acc(J123, Sh0_0, slash_acc(J12, Sh0_30, slash(J1, Sh0_230))));
        A0h0_9 = ubar_dot(UB[0], Fh0_9);
        A1h0_9 = ubar_dot(UB[1], Fh0_9);
        const Sp<R> Sh0_130 = prop_neg(pb + p11, MT, IQ11, slash_acc(J130, Sh0_, slash_acc(J13, Sh0_0, slash(J1, Sh0_30))));
        const Sp<R> Fh0_15 = slash_acc(J2130, Sh0_, slash_acc(J213, Sh0_0, slash_acc(J21, Sh0_30, slash(J2, Sh0_130))));
        A0h0_15 = ubar_dot(UB[0], Fh0_15);
        A1h0_15 = ubar_dot(UB[1], Fh0_15);
      }
      C2<R> A0h0_10, A1h0_10;
      C2<R> A0h0_20, A1h0_20;
      {  // orderings (1, 3, 0, 2), (3, 1, 0, 2)
        V4<RG> J0 = E0; opaque4(J0);
        V4<RG> k0 = K0; opaque4(k0);
        V4<RG> J1 = E1; opaque4(J1);
        V4<RG> k1 = K1; opaque4(k1);
        V4<RG> J2 = E2; opaque4(J2);
        V4<RG> k2 = K2; opaque4(k2);
        V4<RG> J3 = E3; opaque4(J3);
        V4<RG> k3 = K3; opaque4(k3);
        V4<R> pb = PB; opaque4(pb);
        const V4<RG> J13 = G10 * (v3(J1, J3, k1, k3));
        const V4<RG> J30 = G9 * (v3(J3, J0, k3, k0));
        const V4<RG> p9 = k0 + k3;
        const V4<RG> p10 = k1 + k3;
        const V4<RG> J130 = G11 * (w4_sub(J1, J3, J0, v3_acc(J13, J0, p10, k0, v3(J1, J30, k1, p9))));
        const V4<RG> J02 = G5 * (v3(J0, J2, k0, k2));
        const V4<RG> p5 = k0 + k2;
        const V4<RG> J302 = G13 * (w4_sub(J3, J0, J2, v3_acc(J30, J2, p9, k2, v3(J3, J02, k3, p5))));
        const V4<RG> p13 = k0 + k2 + k3;
        const V4<RG> p11 = k0 + k1 + k3;
        const V4<RG> J1302 = G15 * (w4_sub(J13, J0, J2, w4_sub(J1, J30, J2, w4_sub(J1, J3, J02, v3_acc(J130, J2, p11, k2, v3_acc(J13, J02, p10, p5, v3(J1, J302, k1, p13)))))));
        const V4<RG> J31 = RG(-1.0) * J13;
        const V4<RG> J10 = G3 * (v3(J1, J0, k1, k0));
        const V4<RG> p3 = k0 + k1;
        const V4<RG> J310 = G11 * (w4_sub(J3, J1, J0, v3_acc(J31, J0, p10, k0, v3(J3, J10, k3, p3))));
        const V4<RG> J102 = G7 * (w4_sub(J1, J0, J2, v3_acc(J10, J2, p3, k2, v3(J1, J02, k1, p5))));
        const V4<RG> p7 = k0 + k1 + k2;
        const V4<RG> J3102 = G15 * (w4_sub(J31, J0, J2, w4_sub(J3, J10, J2, w4_sub(J3, J1, J02, v3_acc(J310, J2, p11, k2, v3_acc(J31, J02, p10, p5, v3(J3, J102, k3, p7)))))));
        Sp<R> Sh0_ = VS[0]; opaque_sp(Sh0_);
        const Sp<R> Sh0_2 = prop_neg(pb + k2, MT, IQ4, slash(J2, Sh0_));
        const Sp<R> Sh0_02 = prop_neg(pb + p5, MT, IQ5, slash_acc(J02, Sh0_, slash(J0, Sh0_2)));
        const Sp<R> Sh0_302 = prop_neg(pb + p13, MT, IQ13, slash_acc(J302, Sh0_, slash_acc(J30, Sh0_2, slash(J3, Sh0_02))));
        const Sp<R> Fh0_10 = slash_acc(J1302, Sh0_, slash_acc(J130, Sh0_2, slash_acc(J13, Sh0_02, slash(J1, Sh0_302))));
        A0h0_10 = ubar_dot(UB[0], Fh0_10);
        A1h0_10 = ubar_dot(UB[1], Fh0_10);
        const Sp<R> Sh0_102 = prop_neg(pb + p7, MT, IQ7, slash_acc(J102, Sh0_, slash_acc(J10, Sh0_2, slash(J1, Sh0_02))));
        const Sp<R> Fh0_20 = slash_acc(J3102, Sh0_, slash_acc(J310, Sh0_2, slash_acc(J31, Sh0_02, slash(J3, Sh0_102))));
        A0h0_20 = ubar_dot(UB[0], Fh0_20);
        A1h0_20 = ubar_dot(UB[1], Fh0_20);
      }
      C2<R> A0h0_11, A1h0_11;
      C2<R> A0h0_21, A1h0_21;
      {  // orderings (1, 3, 2, 0), (3, 1, 2, 0)
        V4<RG> J0 = E0; opaque4(J0);
        V4<RG> k0 = K0; opaque4(k0);
        V4<RG> J1 = E1; opaque4(J1);
        V4<RG> k1 = K1; opaque4(k1);
        V4<RG> J2 = E2; opaque4(J2);
        V4<RG> k2 = K2; opaque4(k2);
        V4<RG> J3 = E3; opaque4(J3);
        V4<RG> k3 = K3; opaque4(k3);
        V4<R> pb = PB; opaque4(pb);
        const V4<RG> J13 = G10 * (v3(J1, J3, k1, k3));
        const V4<RG> J32 = G12 * (v3(J3, J2, k3, k2));
        const V4<RG> p12 = k2 + k3;
        const V4<RG> p10 = k1 + k3;
        const V4<RG> J132 = G14 * (w4_sub(J1, J3, J2, v3_acc(J13, J2, p10, k2, v3(J1, J32, k1, p12))));
        const V4<RG> J20 = G5 * (v3(J2, J0, k2, k0));
        const V4<RG> p5 = k0 + k2;
        const V4<RG> J320 = G13 * (w4_sub(J3, J2, J0, v3_acc(J32, J0, p12, k0, v3(J3, J20, k3, p5))));
        const V4<RG> p13 = k0 + k2 + k3;
        const V4<RG> p14 = k1 + k2 + k3;
        const V4<RG> J1320 = G15 * (w4_sub(J13, J2, J0, w4_sub(J1, J32, J0, w4_sub(J1, J3, J20, v3_acc(J132, J0, p14, k0, v3_acc(J13, J20, p10, p5, v3(J1, J320, k1, p13)))))));
        const V4<RG> J31 = RG(-1.0) * J13;
        const V4<RG> J12 = G6 * (v3(J1, J2, k1, k2));
        const V4<RG> p6 = k1 + k2;
        const V4<RG> J312 = G14 * (w4_sub(J3, J1, J2, v3_acc(J31, J2, p10, k2, v3(J3, J12, k3, p6))));
        const V4<RG> J120 = G7 * (w4_sub(J1, J2, J0, v3_acc(J12, J0, p6, k0, v3(J1, J20, k1, p5))));
        const V4<RG> p7 = k0 + k1 + k2;
        const V4<RG> J3120 = G15 * (w4_sub(J31, J2, J0, w4_sub(J3, J12, J0, w4_sub(J3, J1, J20, v3_acc(J312, J0, p14, k0, v3_acc(J31, J20, p10, p5, v3(J3, J120, k3, p7)))))));
        Sp<R> Sh0_ = VS[0]; opaque_sp(Sh0_);
        const Sp<R> Sh0_0 = prop_neg(pb + k0, MT, IQ1, slash(J0, Sh0_));
        const Sp<R> Sh0_20 = prop_neg(pb + p5, MT, IQ5, slash_acc(J20, Sh0_, slash(J2, Sh0_0)));
        const Sp<R> Sh0_320 = prop_neg(pb + p13, MT, IQ13, slash_acc(J320, Sh0_, slash_acc(J32, Sh0_0, slash(J3, Sh0_20))));
        const Sp<R> Fh0_11 = slash_acc(J1320, Sh0_, slash_acc(J132, Sh0_0, slash_acc(J13, Sh0_20, slash(J1, Sh0_320))));
        A0h0_11 = ubar_dot(UB[0], Fh0_11);
        A1h0_11 = ubar_dot(UB[1], Fh0_11);
        const Sp<R> Sh0_120 = prop_neg(pb + p7, MT, IQ7, slash_acc(J120, Sh0_, slash_acc(J12, Sh0_0, slash(J1, Sh0_20))));
        const Sp<R> Fh0_21 = slash_acc(J3120, Sh0_, slash_acc(J312, Sh0_0, slash_acc(J31, Sh0_20, slash(J3, Sh0_120))));
        A0h0_21 = ubar_dot(UB[0], Fh0_21);
        A1h0_21 = ubar_dot(UB[1], Fh0_21);
      }
      C2<R> A0h0_16, A1h0_16;
      C2<R> A0h0_22, A1h0_22;
      {  // orderings (2, 3, 0, 1), (3, 2, 0, 1)
        V4<RG> J0 = E0; opaque4(J0);
        V4<RG> k0 = K0; opaque4(k0);
        V4<RG> J1 = E1; opaque4(J1);
        V4<RG> k1 = K1; opaque4(k1);
        V4<RG> J2 = E2; opaque4(J2);
        V4<RG> k2 = K2; opaque4(k2);
        V4<RG> J3 = E3; opaque4(J3);
        V4<RG> k3 = K3; opaque4(k3);
        V4<R> pb = PB; opaque4(pb);
        const V4<RG> J23 = G12 * (v3(J2, J3, k2, k3));
        const V4<RG> J30 = G9 * (v3(J3, J0, k3, k0));
        const V4<RG> p9 = k0 + k3;
        const V4<RG> p12 = k2 + k3;
        const V4<RG> J230 = G13 * (w4_sub(J2, J3, J0, v3_acc(J23, J0, p12, k0, v3(J2, J30, k2, p9))));
        const V4<RG> J01 = G3 * (v3(J0, J1, k0, k1));
        const V4<RG> p3 = k0 + k1;
        const V4<RG> J301 = G11 * (w4_sub(J3, J0, J1, v3_acc(J30, J1, p9, k1, v3(J3, J01, k3, p3))));
        const V4<RG> p11 = k0 + k1 + k3;
        const V4<RG> p13 = k0 + k2 + k3;
        const V4<RG> J2301 = G15 * (w4_sub(J23, J0, J1, w4_sub(J2, J30, J1, w4_sub(J2, J3, J01, v3_acc(J230, J1, p13, k1, v3_acc(J23, J01, p12, p3, v3(J2, J301, k2, p11)))))));
        const V4<RG> J32 = RG(-1.0) * J23;
        const V4<RG> J20 = G5 * (v3(J2, J0, k2, k0));
        const V4<RG> p5 = k0 + k2;
        const V4<RG> J320 = G13 * (w4_sub(J3, J2, J0, v3_acc(J32, J0, p12, k0, v3(J3, J20, k3, p5))));
        const V4<RG> J201 = G7 * (w4_sub(J2, J0, J1, v3_acc(J20, J1, p5, k1, v3(J2, J01, k2, p3))));
        const V4<RG> p7 = k0 + k1 + k2;
        const V4<RG> J3201 = G15 * (w4_sub(J32, J0, J1, w4_sub(J3, J20, J1, w4_sub(J3, J2, J01, v3_acc(J320, J1, p13, k1, v3_acc(J32, J01, p12, p3, v3(J3, J201, k3, p7)))))));
        Sp<R> Sh0_ = VS[0]; opaque_sp(Sh0_);
        const Sp<R> Sh0_1 = prop_neg(pb + k1, MT, IQ2, slash(J1, Sh0_));
        const Sp<R> Sh0_01 = prop_neg(pb + p3, MT, IQ3, slash_acc(J01, Sh0_, slash(J0, Sh0_1)));
        const Sp<R> Sh0_301 = prop_neg(pb + p11, MT, IQ11, slash_acc(J301, Sh0_, slash_acc(J30, Sh0_1, slash(J3, Sh0_01))));
        const Sp<R> Fh0_16 = slash_acc(J2301, Sh0_, slash_acc(J230, Sh0_1, slash_acc(J23, Sh0_01, slash(J2, Sh0_301))));
        A0h0_16 = ubar_dot(UB[0], Fh0_16);
        A1h0_16 = ubar_dot(UB[1], Fh0_16);
        const Sp<R> Sh0_201 = prop_neg(pb + p7, MT, IQ7, slash_acc(J201, Sh0_, slash_acc(J20, Sh0_1, slash(J2, Sh0_01))));
        const Sp<R> Fh0_22 = slash_acc(J3201, Sh0_, slash_acc(J320, Sh0_1, slash_acc(J32, Sh0_01, slash(J3, Sh0_201))));
        A0h0_22 = ubar_dot(UB[0], Fh0_22);
        A1h0_22 = ubar_dot(UB[1], Fh0_22);
      }
      C2<R> A0h0_17, A1h0_17;
      C2<R> A0h0_23, A1h0_23;
      {  // orderings (2, 3, 1, 0), (3, 2, 1, 0)
        V4<RG> J0 = E0; opaque4(J0);
        V4<RG> k0 = K0; opaque4(k0);
        V4<RG> J1 = E1; opaque4(J1);
        V4<RG> k1 = K1; opaque4(k1);
        V4<RG> J2 = E2; opaque4(J2);
        V4<RG> k2 = K2; opaque4(k2);
        V4<RG> J3 = E3; opaque4(J3);
        V4<RG> k3 = K3; opaque4(k3);
        V4<R> pb = PB; opaque4(pb);
        const V4<RG> J23 = G12 * (v3(J2, J3, k2, k3));
        const V4<RG> J31 = G10 * (v3(J3, J1, k3, k1));
        const V4<RG> p10 = k1 + k3;
        const V4<RG> p12 = k2 + k3;
        const V4<RG> J231 = G14 * (w4_sub(J2, J3, J1, v3_acc(J23, J1, p12, k1, v3(J2, J31, k2, p10))));
        const V4<RG> J10 = G3 * (v3(J1, J0, k1, k0));
        const V4<RG> p3 = k0 + k1;
        const V4<RG> J310 = G11 * (w4_sub(J3, J1, J0, v3_acc(J31, J0, p10, k0, v3(J3, J10, k3, p3))));
        const V4<RG> p11 = k0 + k1 + k3;
        const V4<RG> p14 = k1 + k2 + k3;
        const V4<RG> J2310 = G15 * (w4_sub(J23, J1, J0, w4_sub(J2, J31, J0, w4_sub(J2, J3, J10, v3_acc(J231, J0, p14, k0, v3_acc(J23, J10, p12, p3, v3(J2, J310, k2, p11)))))));
        const V4<RG> J32 = RG(-1.0) * J23;
        const V4<RG> J21 = G6 * (v3(J2, J1, k2, k1));
        const V4<RG> p6 = k1 + k2;
        const V4<RG> J321 = G14 * (w4_sub(J3, J2, J1, v3_acc(J32, J1, p12, k1, v3(J3, J21, k3, p6))));
        const V4<RG> J210 = G7 * (w4_sub(J2, J1, J0, v3_acc(J21, J0, p6, k0, v3(J2, J10, k2, p3))));
        const V4<RG> p7 = k0 + k1 + k2;
        const V4<RG> J3210 = G15 * (w4_sub(J32, J1, J0, w4_sub(J3, J21, J0, w4_sub(J3, J2, J10, v3_acc(J321, J0, p14, k0, v3_acc(J32, J10, p12, p3, v3(J3, J210, k3, p7)))))));
        Sp<R> Sh0_ = VS[0]; opaque_sp(Sh0_);
        const Sp<R> Sh0_0 = prop_neg(pb + k0, MT, IQ1, slash(J0, Sh0_));
        const Sp<R> Sh0_10 = prop_neg(pb + p3, MT, IQ3, slash_acc(J10, Sh0_, slash(J1, Sh0_0)));
        const Sp<R> Sh0_310 = prop_neg(pb + p11, MT, IQ11, slash_acc(J310, Sh0_, slash_acc(J31, Sh0_0, slash(J3, Sh0_10))));
        const Sp<R> Fh0_17 = slash_acc(J2310, Sh0_, slash_acc(J231, Sh0_0, slash_acc(J23, Sh0_10, slash(J2, Sh0_310))));
        A0h0_17 = ubar_dot(UB[0], Fh0_17);
        A1h0_17 = ubar_dot(UB[1], Fh0_17);
        const Sp<R> Sh0_210 = prop_neg(pb + p7, MT, IQ7, slash_acc(J210, Sh0_, slash_acc(J21, Sh0_0, slash(J2, Sh0_10))));
        const Sp<R> Fh0_23 = slash_acc(J3210, Sh0_, slash_acc(J321, Sh0_0, slash_acc(J32, Sh0_10, slash(J3, Sh0_210))));
        A0h0_23 = ubar_dot(UB[0], Fh0_23);
        A1h0_23 = ubar_dot(UB[1], Fh0_23);
      }
      {
        R s = cre_dot(A0h0_0, A0h0_1);
        s = cre_dot_acc(A0h0_0, A0h0_2, s); s = cre_dot_acc(A0h0_0, A0h0_6, s); s = cre_dot_acc(A0h0_1, A0h0_4, s);
        s = cre_dot_acc(A0h0_1, A0h0_7, s); s = cre_dot_acc(A0h0_2, A0h0_3, s); s = cre_dot_acc(A0h0_2, A0h0_12, s);
        s = cre_dot_acc(A0h0_3, A0h0_5, s); s = cre_dot_acc(A0h0_3, A0h0_13, s); s = cre_dot_acc(A0h0_4, A0h0_5, s);
        s = cre_dot_acc(A0h0_4, A0h0_18, s); s = cre_dot_acc(A0h0_5, A0h0_19, s); s = cre_dot_acc(A0h0_6, A0h0_7, s);
        s = cre_dot_acc(A0h0_6, A0h0_8, s); s = cre_dot_acc(A0h0_7, A0h0_10, s); s = cre_dot_acc(A0h0_8, A0h0_9, s);
        s = cre_dot_acc(A0h0_8, A0h0_14, s); s = cre_dot_acc(A0h0_9, A0h0_11, s); s = cre_dot_acc(A0h0_9, A0h0_15, s);
        s = cre_dot_acc(A0h0_10, A0h0_11, s); s = cre_dot_acc(A0h0_10, A0h0_20, s); s = cre_dot_acc(A0h0_11, A0h0_21, s);
        s = cre_dot_acc(A0h0_12, A0h0_13, s); s = cre_dot_acc(A0h0_12, A0h0_14, s); s = cre_dot_acc(A0h0_13, A0h0_16, s);
        s = cre_dot_acc(A0h0_14, A0h0_15, s); s = cre_dot_acc(A0h0_15, A0h0_17, s); s = cre_dot_acc(A0h0_16, A0h0_17, s);
        s = cre_dot_acc(A0h0_16, A0h0_22, s); s = cre_dot_acc(A0h0_17, A0h0_23, s); s = cre_dot_acc(A0h0_18, A0h0_19, s);
        s = cre_dot_acc(A0h0_18, A0h0_20, s); s = cre_dot_acc(A0h0_19, A0h0_22, s); s = cre_dot_acc(A0h0_20, A0h0_21, s);
        s = cre_dot_acc(A0h0_21, A0h0_23, s); s = cre_dot_acc(A0h0_22, A0h0_23, s);
        total = total + R(-128.0) * s;
      }
      {
        R s = cre_dot(A0h0_0, A0h0_23);
        s = cre_dot_acc(A0h0_1, A0h0_17, s); s = cre_dot_acc(A0h0_2, A0h0_21, s); s = cre_dot_acc(A0h0_3, A0h0_11, s);
        s = cre_dot_acc(A0h0_4, A0h0_15, s); s = cre_dot_acc(A0h0_5, A0h0_9, s); s = cre_dot_acc(A0h0_6, A0h0_22, s);
        s = cre_dot_acc(A0h0_7, A0h0_16, s); s = cre_dot_acc(A0h0_8, A0h0_19, s); s = cre_dot_acc(A0h0_10, A0h0_13, s);
        s = cre_dot_acc(A0h0_12, A0h0_20, s); s = cre_dot_acc(A0h0_14, A0h0_18, s);
        total = total + R(-56.0) * s;
      }
      {
        R s = cre_dot(A0h0_0, A0h0_11);
        s = cre_dot_acc(A0h0_0, A0h0_15, s); s = cre_dot_acc(A0h0_0, A0h0_19, s); s = cre_dot_acc(A0h0_0, A0h0_20, s);
        s = cre_dot_acc(A0h0_1, A0h0_9, s); s = cre_dot_acc(A0h0_1, A0h0_13, s); s = cre_dot_acc(A0h0_1, A0h0_14, s);
        s = cre_dot_acc(A0h0_1, A0h0_21, s); s = cre_dot_acc(A0h0_2, A0h0_9, s); s = cre_dot_acc(A0h0_2, A0h0_17, s);
        s = cre_dot_acc(A0h0_2, A0h0_18, s); s = cre_dot_acc(A0h0_2, A0h0_22, s); s = cre_dot_acc(A0h0_3, A0h0_7, s);
        s = cre_dot_acc(A0h0_3, A0h0_8, s); s = cre_dot_acc(A0h0_3, A0h0_15, s); s = cre_dot_acc(A0h0_3, A0h0_23, s);
        s = cre_dot_acc(A0h0_4, A0h0_11, s); s = cre_dot_acc(A0h0_4, A0h0_12, s); s = cre_dot_acc(A0h0_4, A0h0_16, s);
        s = cre_dot_acc(A0h0_4, A0h0_23, s); s = cre_dot_acc(A0h0_5, A0h0_6, s); s = cre_dot_acc(A0h0_5, A0h0_10, s);
        s = cre_dot_acc(A0h0_5, A0h0_17, s); s = cre_dot_acc(A0h0_5, A0h0_21, s); s = cre_dot_acc(A0h0_6, A0h0_13, s);
        s = cre_dot_acc(A0h0_6, A0h0_18, s); s = cre_dot_acc(A0h0_6, A0h0_21, s); s = cre_dot_acc(A0h0_7, A0h0_12, s);
        s = cre_dot_acc(A0h0_7, A0h0_15, s); s = cre_dot_acc(A0h0_7, A0h0_19, s); s = cre_dot_acc(A0h0_8, A0h0_16, s);
        s = cre_dot_acc(A0h0_8, A0h0_20, s); s = cre_dot_acc(A0h0_8, A0h0_23, s); s = cre_dot_acc(A0h0_9, A0h0_13, s);
        s = cre_dot_acc(A0h0_9, A0h0_22, s); s = cre_dot_acc(A0h0_10, A0h0_14, s); s = cre_dot_acc(A0h0_10, A0h0_17, s);
        s = cre_dot_acc(A0h0_10, A0h0_22, s); s = cre_dot_acc(A0h0_11, A0h0_16, s); s = cre_dot_acc(A0h0_11, A0h0_19, s);
        s = cre_dot_acc(A0h0_12, A0h0_19, s); s = cre_dot_acc(A0h0_12, A0h0_23, s); s = cre_dot_acc(A0h0_13, A0h0_18, s);
        s = cre_dot_acc(A0h0_14, A0h0_21, s); s = cre_dot_acc(A0h0_14, A0h0_22, s); s = cre_dot_acc(A0h0_15, A0h0_20, s);
        s = cre_dot_acc(A0h0_16, A0h0_20, s); s = cre_dot_acc(A0h0_17, A0h0_18, s);
        total = total + R(-20.0) * s;
      }
      {
        R s = cre_dot(A0h0_0, A0h0_9);
        s = cre_dot_acc(A0h0_0, A0h0_10, s); s = cre_dot_acc(A0h0_0, A0h0_13, s); s = cre_dot_acc(A0h0_0, A0h0_18, s);
        s = cre_dot_acc(A0h0_1, A0h0_8, s); s = cre_dot_acc(A0h0_1, A0h0_11, s); s = cre_dot_acc(A0h0_1, A0h0_12, s);
        s = cre_dot_acc(A0h0_1, A0h0_19, s); s = cre_dot_acc(A0h0_2, A0h0_7, s); s = cre_dot_acc(A0h0_2, A0h0_15, s);
        s = cre_dot_acc(A0h0_2, A0h0_16, s); s = cre_dot_acc(A0h0_2, A0h0_19, s); s = cre_dot_acc(A0h0_3, A0h0_6, s);
        s = cre_dot_acc(A0h0_3, A0h0_14, s); s = cre_dot_acc(A0h0_3, A0h0_17, s); s = cre_dot_acc(A0h0_3, A0h0_18, s);
        s = cre_dot_acc(A0h0_4, A0h0_6, s); s = cre_dot_acc(A0h0_4, A0h0_13, s); s = cre_dot_acc(A0h0_4, A0h0_21, s);
        s = cre_dot_acc(A0h0_4, A0h0_22, s); s = cre_dot_acc(A0h0_5, A0h0_7, s); s = cre_dot_acc(A0h0_5, A0h0_12, s);
        s = cre_dot_acc(A0h0_5, A0h0_20, s); s = cre_dot_acc(A0h0_5, A0h0_23, s); s = cre_dot_acc(A0h0_6, A0h0_15, s);
        s = cre_dot_acc(A0h0_6, A0h0_20, s); s = cre_dot_acc(A0h0_7, A0h0_14, s); s = cre_dot_acc(A0h0_7, A0h0_21, s);
        s = cre_dot_acc(A0h0_8, A0h0_13, s); s = cre_dot_acc(A0h0_8, A0h0_17, s); s = cre_dot_acc(A0h0_8, A0h0_21, s);
        s = cre_dot_acc(A0h0_9, A0h0_12, s); s = cre_dot_acc(A0h0_9, A0h0_16, s); s = cre_dot_acc(A0h0_9, A0h0_20, s);
        s = cre_dot_acc(A0h0_10, A0h0_15, s); s = cre_dot_acc(A0h0_10, A0h0_19, s); s = cre_dot_acc(A0h0_10, A0h0_23, s);
        s = cre_dot_acc(A0h0_11, A0h0_14, s); s = cre_dot_acc(A0h0_11, A0h0_18, s); s = cre_dot_acc(A0h0_11, A0h0_22, s);
        s = cre_dot_acc(A0h0_12, A0h0_22, s); s = cre_dot_acc(A0h0_13, A0h0_23, s); s = cre_dot_acc(A0h0_14, A0h0_23, s);
        s = cre_dot_acc(A0h0_15, A0h0_22, s); s = cre_dot_acc(A0h0_16, A0h0_18, s); s = cre_dot_acc(A0h0_16, A0h0_21, s);
        s = cre_dot_acc(A0h0_17, A0h0_19, s); s = cre_dot_acc(A0h0_17, A0h0_20, s);
        total = total + R(-2.0) * s;
      }
      {
        R s = cre_dot(A0h0_0, A0h0_3);
        s = cre_dot_acc(A0h0_0, A0h0_4, s); s = cre_dot_acc(A0h0_0, A0h0_7, s); s = cre_dot_acc(A0h0_0, A0h0_8, s);
        s = cre_dot_acc(A0h0_0, A0h0_12, s); s = cre_dot_acc(A0h0_1, A0h0_2, s); s = cre_dot_acc(A0h0_1, A0h0_5, s);
        s = cre_dot_acc(A0h0_1, A0h0_6, s); s = cre_dot_acc(A0h0_1, A0h0_10, s); s = cre_dot_acc(A0h0_1, A0h0_18, s);
        s = cre_dot_acc(A0h0_2, A0h0_5, s); s = cre_dot_acc(A0h0_2, A0h0_6, s); s = cre_dot_acc(A0h0_2, A0h0_13, s);
        s = cre_dot_acc(A0h0_2, A0h0_14, s); s = cre_dot_acc(A0h0_3, A0h0_4, s); s = cre_dot_acc(A0h0_3, A0h0_12, s);
        s = cre_dot_acc(A0h0_3, A0h0_16, s); s = cre_dot_acc(A0h0_3, A0h0_19, s); s = cre_dot_acc(A0h0_4, A0h0_7, s);
        s = cre_dot_acc(A0h0_4, A0h0_19, s); s = cre_dot_acc(A0h0_4, A0h0_20, s); s = cre_dot_acc(A0h0_5, A0h0_13, s);
        s = cre_dot_acc(A0h0_5, A0h0_18, s); s = cre_dot_acc(A0h0_5, A0h0_22, s); s = cre_dot_acc(A0h0_6, A0h0_9, s);
        s = cre_dot_acc(A0h0_6, A0h0_10, s); s = cre_dot_acc(A0h0_6, A0h0_14, s); s = cre_dot_acc(A0h0_7, A0h0_8, s);
        s = cre_dot_acc(A0h0_7, A0h0_11, s); s = cre_dot_acc(A0h0_7, A0h0_20, s); s = cre_dot_acc(A0h0_8, A0h0_11, s);
        s = cre_dot_acc(A0h0_8, A0h0_12, s); s = cre_dot_acc(A0h0_8, A0h0_15, s); s = cre_dot_acc(A0h0_9, A0h0_10, s);
        s = cre_dot_acc(A0h0_9, A0h0_14, s); s = cre_dot_acc(A0h0_9, A0h0_17, s); s = cre_dot_acc(A0h0_9, A0h0_21, s);
        s = cre_dot_acc(A0h0_10, A0h0_18, s); s = cre_dot_acc(A0h0_10, A0h0_21, s); s = cre_dot_acc(A0h0_11, A0h0_15, s);
        s = cre_dot_acc(A0h0_11, A0h0_20, s); s = cre_dot_acc(A0h0_11, A0h0_23, s); s = cre_dot_acc(A0h0_12, A0h0_15, s);
        s = cre_dot_acc(A0h0_12, A0h0_16, s); s = cre_dot_acc(A0h0_13, A0h0_14, s); s = cre_dot_acc(A0h0_13, A0h0_17, s);
        s = cre_dot_acc(A0h0_13, A0h0_22, s); s = cre_dot_acc(A0h0_14, A0h0_17, s); s = cre_dot_acc(A0h0_15, A0h0_16, s);
        s = cre_dot_acc(A0h0_15, A0h0_23, s); s = cre_dot_acc(A0h0_16, A0h0_19, s); s = cre_dot_acc(A0h0_16, A0h0_23, s);
        s = cre_dot_acc(A0h0_17, A0h0_21, s); s = cre_dot_acc(A0h0_17, A0h0_22, s); s = cre_dot_acc(A0h0_18, A0h0_21, s);
        s = cre_dot_acc(A0h0_18, A0h0_22, s); s = cre_dot_acc(A0h0_19, A0h0_20, s); s = cre_dot_acc(A0h0_19, A0h0_23, s);
        s = cre_dot_acc(A0h0_20, A0h0_23, s); s = cre_dot_acc(A0h0_21, A0h0_22, s);
        total = total + R(16.0) * s;
      }
      {
        R s = cre_dot(A0h0_0, A0h0_17);
        s = cre_dot_acc(A0h0_0, A0h0_21, s); s = cre_dot_acc(A0h0_0, A0h0_22, s); s = cre_dot_acc(A0h0_1, A0h0_15, s);
        s = cre_dot_acc(A0h0_1, A0h0_16, s); s = cre_dot_acc(A0h0_1, A0h0_23, s); s = cre_dot_acc(A0h0_2, A0h0_11, s);
        s = cre_dot_acc(A0h0_2, A0h0_20, s); s = cre_dot_acc(A0h0_2, A0h0_23, s); s = cre_dot_acc(A0h0_3, A0h0_9, s);
        s = cre_dot_acc(A0h0_3, A0h0_10, s); s = cre_dot_acc(A0h0_3, A0h0_21, s); s = cre_dot_acc(A0h0_4, A0h0_9, s);
        s = cre_dot_acc(A0h0_4, A0h0_14, s); s = cre_dot_acc(A0h0_4, A0h0_17, s); s = cre_dot_acc(A0h0_5, A0h0_8, s);
        s = cre_dot_acc(A0h0_5, A0h0_11, s); s = cre_dot_acc(A0h0_5, A0h0_15, s); s = cre_dot_acc(A0h0_6, A0h0_16, s);
        s = cre_dot_acc(A0h0_6, A0h0_19, s); s = cre_dot_acc(A0h0_6, A0h0_23, s); s = cre_dot_acc(A0h0_7, A0h0_13, s);
        s = cre_dot_acc(A0h0_7, A0h0_17, s); s = cre_dot_acc(A0h0_7, A0h0_22, s); s = cre_dot_acc(A0h0_8, A0h0_18, s);
        s = cre_dot_acc(A0h0_8, A0h0_22, s); s = cre_dot_acc(A0h0_9, A0h0_19, s); s = cre_dot_acc(A0h0_10, A0h0_12, s);
        s = cre_dot_acc(A0h0_10, A0h0_16, s); s = cre_dot_acc(A0h0_11, A0h0_13, s); s = cre_dot_acc(A0h0_12, A0h0_18, s);
        s = cre_dot_acc(A0h0_12, A0h0_21, s); s = cre_dot_acc(A0h0_13, A0h0_20, s); s = cre_dot_acc(A0h0_14, A0h0_19, s);
        s = cre_dot_acc(A0h0_14, A0h0_20, s); s = cre_dot_acc(A0h0_15, A0h0_18, s);
        total = total + R(124.0) * s;
      }
      {
        R s = cre_dot(A0h0_0, A0h0_16);
        s = cre_dot_acc(A0h0_1, A0h0_22, s); s = cre_dot_acc(A0h0_2, A0h0_10, s); s = cre_dot_acc(A0h0_3, A0h0_20, s);
        s = cre_dot_acc(A0h0_4, A0h0_8, s); s = cre_dot_acc(A0h0_5, A0h0_14, s); s = cre_dot_acc(A0h0_6, A0h0_17, s);
        s = cre_dot_acc(A0h0_7, A0h0_23, s); s = cre_dot_acc(A0h0_9, A0h0_18, s); s = cre_dot_acc(A0h0_11, A0h0_12, s);
        s = cre_dot_acc(A0h0_13, A0h0_21, s); s = cre_dot_acc(A0h0_15, A0h0_19, s);
        total = total + R(142.0) * s;
      }
      {
        R s = cre_dot(A0h0_0, A0h0_5);
        s = cre_dot_acc(A0h0_0, A0h0_14, s); s = cre_dot_acc(A0h0_1, A0h0_3, s); s = cre_dot_acc(A0h0_1, A0h0_20, s);
        s = cre_dot_acc(A0h0_2, A0h0_4, s); s = cre_dot_acc(A0h0_2, A0h0_8, s); s = cre_dot_acc(A0h0_3, A0h0_22, s);
        s = cre_dot_acc(A0h0_4, A0h0_10, s); s = cre_dot_acc(A0h0_5, A0h0_16, s); s = cre_dot_acc(A0h0_6, A0h0_11, s);
        s = cre_dot_acc(A0h0_6, A0h0_12, s); s = cre_dot_acc(A0h0_7, A0h0_9, s); s = cre_dot_acc(A0h0_7, A0h0_18, s);
        s = cre_dot_acc(A0h0_8, A0h0_10, s); s = cre_dot_acc(A0h0_9, A0h0_23, s); s = cre_dot_acc(A0h0_11, A0h0_17, s);
        s = cre_dot_acc(A0h0_12, A0h0_17, s); s = cre_dot_acc(A0h0_13, A0h0_15, s); s = cre_dot_acc(A0h0_13, A0h0_19, s);
        s = cre_dot_acc(A0h0_14, A0h0_16, s); s = cre_dot_acc(A0h0_15, A0h0_21, s); s = cre_dot_acc(A0h0_18, A0h0_23, s);
        s = cre_dot_acc(A0h0_19, A0h0_21, s); s = cre_dot_acc(A0h0_20, A0h0_22, s);
        total = total + R(160.0) * s;
      }
      {
        R s = cabs2(A0h0_0);
        s = cabs2_acc(A0h0_1, s); s = cabs2_acc(A0h0_2, s); s = cabs2_acc(A0h0_3, s);
        s = cabs2_acc(A0h0_4, s); s = cabs2_acc(A0h0_5, s); s = cabs2_acc(A0h0_6, s);
        s = cabs2_acc(A0h0_7, s); s = cabs2_acc(A0h0_8, s); s = cabs2_acc(A0h0_9, s);
        s = cabs2_acc(A0h0_10, s); s = cabs2_acc(A0h0_11, s); s = cabs2_acc(A0h0_12, s);
        s = cabs2_acc(A0h0_13, s); s = cabs2_acc(A0h0_14, s); s = cabs2_acc(A0h0_15, s);
        s = cabs2_acc(A0h0_16, s); s = cabs2_acc(A0h0_17, s); s = cabs2_acc(A0h0_18, s);
        s = cabs2_acc(A0h0_19, s); s = cabs2_acc(A0h0_20, s); s = cabs2_acc(A0h0_21, s);
        s = cabs2_acc(A0h0_22, s); s = cabs2_acc(A0h0_23, s);
        total = total + R(512.0) * s;
      }
      {
        R s = cre_dot(A1h0_0, A1h0_1);
        s = cre_dot_acc(A1h0_0, A1h0_2, s); s = cre_dot_acc(A1h0_0, A1h0_6, s); s = cre_dot_acc(A1h0_1, A1h0_4, s);
        s = cre_dot_acc(A1h0_1, A1h0_7, s); s = cre_dot_acc(A1h0_2, A1h0_3, s); s = cre_dot_acc(A1h0_2, A1h0_12, s);
        s = cre_dot_acc(A1h0_3, A1h0_5, s); s = cre_dot_acc(A1h0_3, A1h0_13, s); s = cre_dot_acc(A1h0_4, A1h0_5, s);
        s = cre_dot_acc(A1h0_4, A1h0_18, s); s = cre_dot_acc(A1h0_5, A1h0_19, s); s = cre_dot_acc(A1h0_6, A1h0_7, s);
        s = cre_dot_acc(A1h0_6, A1h0_8, s); s = cre_dot_acc(A1h0_7, A1h0_10, s); s = cre_dot_acc(A1h0_8, A1h0_9, s);
        s = cre_dot_acc(A1h0_8, A1h0_14, s); s = cre_dot_acc(A1h0_9, A1h0_11, s); s = cre_dot_acc(A1h0_9, A1h0_15, s);
        s = cre_dot_acc(A1h0_10, A1h0_11, s); s = cre_dot_acc(A1h0_10, A1h0_20, s); s = cre_dot_acc(A1h0_11, A1h0_21, s);
        s = cre_dot_acc(A1h0_12, A1h0_13, s); s = cre_dot_acc(A1h0_12, A1h0_14, s); s = cre_dot_acc(A1h0_13, A1h0_16, s);
        s = cre_dot_acc(A1h0_14, A1h0_15, s); s = cre_dot_acc(A1h0_15, A1h0_17, s); s = cre_dot_acc(A1h0_16, A1h0_17, s);
        s = cre_dot_acc(A1h0_16, A1h0_22, s); s = cre_dot_acc(A1h0_17, A1h0_23, s); s = cre_dot_acc(A1h0_18, A1h0_19, s);
        s = cre_dot_acc(A1h0_18, A1h0_20, s); s = cre_dot_acc(A1h0_19, A1h0_22, s); s = cre_dot_acc(A1h0_20, A1h0_21, s);
        s = cre_dot_acc(A1h0_21, A1h0_23, s); s = cre_dot_acc(A1h0_22, A1h0_23, s);
        total = total + R(-128.0) * s;
      }
      {
        R s = cre_dot(A1h0_0, A1h0_23);
        s = cre_dot_acc(A1h0_1, A1h0_17, s); s = cre_dot_acc(A1h0_2, A1h0_21, s); s = cre_dot_acc(A1h0_3, A1h0_11, s);
        s = cre_dot_acc(A1h0_4, A1h0_15, s); s = cre_dot_acc(A1h0_5, A1h0_9, s); s = cre_dot_acc(A1h0_6, A1h0_22, s);
        s = cre_dot_acc(A1h0_7, A1h0_16, s); s = cre_dot_acc(A1h0_8, A1h0_19, s); s = cre_dot_acc(A1h0_10, A1h0_13, s);
        s = cre_dot_acc(A1h0_12, A1h0_20, s); s = cre_dot_acc(A1h0_14, A1h0_18, s);
        total = total + R(-56.0) * s;
      }
      {
        R s = cre_dot(A1h0_0, A1h0_11);
        s = cre_dot_acc(A1h0_0, A1h0_15, s); s = cre_dot_acc(A1h0_0, A1h0_19, s); s = cre_dot_acc(A1h0_0, A1h0_20, s);
        s = cre_dot_acc(A1h0_1, A1h0_9, s); s = cre_dot_acc(A1h0_1, A1h0_13, s); s = cre_dot_acc(A1h0_1, A1h0_14, s);
        s = cre_dot_acc(A1h0_1, A1h0_21, s); s = cre_dot_acc(A1h0_2, A1h0_9, s); s = cre_dot_acc(A1h0_2, A1h0_17, s);
        s = cre_dot_acc(A1h0_2, A1h0_18, s); s = cre_dot_acc(A1h0_2, A1h0_22, s); s = cre_dot_acc(A1h0_3, A1h0_7, s);
        s = cre_dot_acc(A1h0_3, A1h0_8, s); s = cre_dot_acc(A1h0_3, A1h0_15, s); s = cre_dot_acc(A1h0_3, A1h0_23, s);
        s = cre_dot_acc(A1h0_4, A1h0_11, s); s = cre_dot_acc(A1h0_4, A1h0_12, s); s = cre_dot_acc(A1h0_4, A1h0_16, s);
        s = cre_dot_acc(A1h0_4, A1h0_23, s); s = cre_dot_acc(A1h0_5, A1h0_6, s); s = cre_dot_acc(A1h0_5, A1h0_10, s);
        s = cre_dot_acc(A1h0_5, A1h0_17, s); s = cre_dot_acc(A1h0_5, A1h0_21, s); s = cre_dot_acc(A1h0_6, A1h0_13, s);
        s = cre_dot_acc(A1h0_6, A1h0_18, s); s = cre_dot_acc(A1h0_6, A1h0_21, s); s = cre_dot_acc(A1h0_7, A1h0_12, s);
        s = cre_dot_acc(A1h0_7, A1h0_15, s); s = cre_dot_acc(A1h0_7, A1h0_19, s); s = cre_dot_acc(A1h0_8, A1h0_16, s);
        s = cre_dot_acc(A1h0_8, A1h0_20, s); s = cre_dot_acc(A1h0_8, A1h0_23, s); s = cre_dot_acc(A1h0_9, A1h0_13, s);
        s = cre_dot_acc(A1h0_9, A1h0_22, s); s = cre_dot_acc(A1h0_10, A1h0_14, s); s = cre_dot_acc(A1h0_10, A1h0_17, s);
        s = cre_dot_acc(A1h0_10, A1h0_22, s); s = cre_dot_acc(A1h0_11, A1h0_16, s); s = cre_dot_acc(A1h0_11, A1h0_19, s);
        s = cre_dot_acc(A1h0_12, A1h0_19, s); s = cre_dot_acc(A1h0_12, A1h0_23, s); s = cre_dot_acc(A1h0_13, A1h0_18, s);
        s = cre_dot_acc(A1h0_14, A1h0_21, s); s = cre_dot_acc(A1h0_14, A1h0_22, s); s = cre_dot_acc(A1h0_15, A1h0_20, s);
        s = cre_dot_acc(A1h0_16, A1h0_20, s); s = cre_dot_acc(A1h0_17, A1h0_18, s);
        total = total + R(-20.0) * s;
      }
      {
        R s = cre_dot(A1h0_0, A1h0_9);
        s = cre_dot_acc(A1h0_0, A1h0_10, s); s = cre_dot_acc(A1h0_0, A1h0_13, s); s = cre_dot_acc(A1h0_0, A1h0_18, s);
        s = cre_dot_acc(A1h0_1, A1h0_8, s); s = cre_dot_acc(A1h0_1, A1h0_11, s); s = cre_dot_acc(A1h0_1, A1h0_12, s);
        s = cre_dot_acc(A1h0_1, A1h0_19, s); s = cre_dot_acc(A1h0_2, A1h0_7, s); s = cre_dot_acc(A1h0_2, A1h0_15, s);
        s = cre_dot_acc(A1h0_2, A1h0_16, s); s = cre_dot_acc(A1h0_2, A1h0_19, s); s = cre_dot_acc(A1h0_3, A1h0_6, s);
        s = cre_dot_acc(A1h0_3, A1h0_14, s); s = cre_dot_acc(A1h0_3, A1h0_17, s); s = cre_dot_acc(A1h0_3, A1h0_18, s);
        s = cre_dot_acc(A1h0_4, A1h0_6, s); s = cre_dot_acc(A1h0_4, A1h0_13, s); s = cre_dot_acc(A1h0_4, A1h0_21, s);
        s = cre_dot_acc(A1h0_4, A1h0_22, s); s = cre_dot_acc(A1h0_5, A1h0_7, s); s = cre_dot_acc(A1h0_5, A1h0_12, s);
        s = cre_dot_acc(A1h0_5, A1h0_20, s); s = cre_dot_acc(A1h0_5, A1h0_23, s); s = cre_dot_acc(A1h0_6, A1h0_15, s);
        s = cre_dot_acc(A1h0_6, A1h0_20, s); s = cre_dot_acc(A1h0_7, A1h0_14, s); s = cre_dot_acc(A1h0_7, A1h0_21, s);
        s = cre_dot_acc(A1h0_8, A1h0_13, s); s = cre_dot_acc(A1h0_8, A1h0_17, s); s = cre_dot_acc(A1h0_8, A1h0_21, s);
        s = cre_dot_acc(A1h0_9, A1h0_12, s); s = cre_dot_acc(A1h0_9, A1h0_16, s); s = cre_dot_acc(A1h0_9, A1h0_20, s);
        s = cre_dot_acc(A1h0_10, A1h0_15, s); s = cre_dot_acc(A1h0_10, A1h0_19, s); s = cre_dot_acc(A1h0_10, A1h0_23, s);
        s = cre_dot_acc(A1h0_11, A1h0_14, s); s = cre_dot_acc(A1h0_11, A1h0_18, s); s = cre_dot_acc(A1h0_11, A1h0_22, s);
        s = cre_dot_acc(A1h0_12, A1h0_22, s); s = cre_dot_acc(A1h0_13, A1h0_23, s); s = cre_dot_acc(A1h0_14, A1h0_23, s);
        s = cre_dot_acc(A1h0_15, A1h0_22, s); s = cre_dot_acc(A1h0_16, A1h0_18, s); s = cre_dot_acc(A1h0_16, A1h0_21, s);
        s = cre_dot_acc(A1h0_17, A1h0_19, s); s = cre_dot_acc(A1h0_17, A1h0_20, s);
        total = total + R(-2.0) * s;
      }
      {
        R s = cre_dot(A1h0_0, A1h0_3);
        s = cre_dot_acc(A1h0_0, A1h0_4, s); s = cre_dot_acc(A1h0_0, A1h0_7, s); s = cre_dot_acc(A1h0_0, A1h0_8, s);
        s = cre_dot_acc(A1h0_0, A1h0_12, s); s = cre_dot_acc(A1h0_1, A1h0_2, s); s = cre_dot_acc(A1h0_1, A1h0_5, s);
        s = cre_dot_acc(A1h0_1, A1h0_6, s); s = cre_dot_acc(A1h0_1, A1h0_10, s); s = cre_dot_acc(A1h0_1, A1h0_18, s);
        s = cre_dot_acc(A1h0_2, A1h0_5, s); s = cre_dot_acc(A1h0_2, A1h0_6, s); s = cre_dot_acc(A1h0_2, A1h0_13, s);
        s = cre_dot_acc(A1h0_2, A1h0_14, s); s = cre_dot_acc(A1h0_3, A1h0_4, s); s = cre_dot_acc(A1h0_3, A1h0_12, s);
        s = cre_dot_acc(A1h0_3, A1h0_16, s); s = cre_dot_acc(A1h0_3, A1h0_19, s); s = cre_dot_acc(A1h0_4, A1h0_7, s);
        s = cre_dot_acc(A1h0_4, A1h0_19, s); s = cre_dot_acc(A1h0_4, A1h0_20, s); s = cre_dot_acc(A1h0_5, A1h0_13, s);
        s = cre_dot_acc(A1h0_5, A1h0_18, s); s = cre_dot_acc(A1h0_5, A1h0_22, s); s = cre_dot_acc(A1h0_6, A1h0_9, s);
        s = cre_dot_acc(A1h0_6, A1h0_10, s); s = cre_dot_acc(A1h0_6, A1h0_14, s); s = cre_dot_acc(A1h0_7, A1h0_8, s);
        s = cre_dot_acc(A1h0_7, A1h0_11, s); s = cre_dot_acc(A1h0_7, A1h0_20, s); s = cre_dot_acc(A1h0_8, A1h0_11, s);
        s = cre_dot_acc(A1h0_8, A1h0_12, s); s = cre_dot_acc(A1h0_8, A1h0_15, s); s = cre_dot_acc(A1h0_9, A1h0_10, s);
        s = cre_dot_acc(A1h0_9, A1h0_14, s); s = cre_dot_acc(A1h0_9, A1h0_17, s); s = cre_dot_acc(A1h0_9, A1h0_21, s);
        s = cre_dot_acc(A1h0_10, A1h0_18, s); s = cre_dot_acc(A1h0_10, A1h0_21, s); s = cre_dot_acc(A1h0_11, A1h0_15, s);
        s = cre_dot_acc(A1h0_11, A1h0_20, s); s = cre_dot_acc(A1h0_11, A1h0_23, s); s = cre_dot_acc(A1h0_12, A1h0_15, s);
        s = cre_dot_acc(A1h0_12, A1h0_16, s); s = cre_dot_acc(A1h0_13, A1h0_14, s); s = cre_dot_acc(A1h0_13, A1h0_17, s);
        s = cre_dot_acc(A1h0_13, A1h0_22, s); s = cre_dot_acc(A1h0_14, A1h0_17, s); s = cre_dot_acc(A1h0_15, A1h0_16, s);
        s = cre_dot_acc(A1h0_15, A1h0_23, s); s = cre_dot_acc(A1h0_16, A1h0_19, s); s = cre_dot_acc(A1h0_16, A1h0_23, s);
        s = cre_dot_acc(A1h0_17, A1h0_21, s); s = cre_dot_acc(A1h0_17, A1h0_22, s); s = cre_dot_acc(A1h0_18, A1h0_21, s);
        s = cre_dot_acc(A1h0_18, A1h0_22, s); s = cre_dot_acc(A1h0_19, A1h0_20, s); s = cre_dot_acc(A1h0_19, A1h0_23, s);
        s = cre_dot_acc(A1h0_20, A1h0_23, s); s = cre_dot_acc(A1h0_21, A1h0_22, s);
        total = total + R(16.0) * s;
      }
      {
        R s = cre_dot(A1h0_0, A1h0_17);
        s = cre_dot_acc(A1h0_0, A1h0_21, s); s = cre_dot_acc(A1h0_0, A1h0_22, s); s = cre_dot_acc(A1h0_1, A1h0_15, s);
        s = cre_dot_acc(A1h0_1, A1h0_16, s); s = cre_dot_acc(A1h0_1, A1h0_23, s); s = cre_dot_acc(A1h0_2, A1h0_11, s);
        s = cre_dot_acc(A1h0_2, A1h0_20, s); s = cre_dot_acc(A1h0_2, A1h0_23, s); s = cre_dot_acc(A1h0_3, A1h0_9, s);
        s = cre_dot_acc(A1h0_3, A1h0_10, s); s = cre_dot_acc(A1h0_3, A1h0_21, s); s = cre_dot_acc(A1h0_4, A1h0_9, s);
        s = cre_dot_acc(A1h0_4, A1h0_14, s); s = cre_dot_acc(A1h0_4, A1h0_17, s); s = cre_dot_acc(A1h0_5, A1h0_8, s);
        s = cre_dot_acc(A1h0_5, A1h0_11, s); s = cre_dot_acc(A1h0_5, A1h0_15, s); s = cre_dot_acc(A1h0_6, A1h0_16, s);
        s = cre_dot_acc(A1h0_6, A1h0_19, s); s = cre_dot_acc(A1h0_6, A1h0_23, s); s = cre_dot_acc(A1h0_7, A1h0_13, s);
        s = cre_dot_acc(A1h0_7, A1h0_17, s); s = cre_dot_acc(A1h0_7, A1h0_22, s); s = cre_dot_acc(A1h0_8, A1h0_18, s);
        s = cre_dot_acc(A1h0_8, A1h0_22, s); s = cre_dot_acc(A1h0_9, A1h0_19, s); s = cre_dot_acc(A1h0_10, A1h0_12, s);
        s = cre_dot_acc(A1h0_10, A1h0_16, s); s = cre_dot_acc(A1h0_11, A1h0_13, s); s = cre_dot_acc(A1h0_12, A1h0_18, s);
        s = cre_dot_acc(A1h0_12, A1h0_21, s); s = cre_dot_acc(A1h0_13, A1h0_20, s); s = cre_dot_acc(A1h0_14, A1h0_19, s);
        s = cre_dot_acc(A1h0_14, A1h0_20, s); s = cre_dot_acc(A1h0_15, A1h0_18, s);
        total = total + R(124.0) * s;
      }
      {
        R s = cre_dot(A1h0_0, A1h0_16);
        s = cre_dot_acc(A1h0_1, A1h0_22, s); s = cre_dot_acc(A1h0_2, A1h0_10, s); s = cre_dot_acc(A1h0_3, A1h0_20, s);
        s = cre_dot_acc(A1h0_4, A1h0_8, s); s = cre_dot_acc(A1h0_5, A1h0_14, s); s = cre_dot_acc(A1h0_6, A1h0_17, s);
        s = cre_dot_acc(A1h0_7, A1h0_23, s); s = cre_dot_acc(A1h0_9, A1h0_18, s); s = cre_dot_acc(A1h0_11, A1h0_12, s);
        s = cre_dot_acc(A1h0_13, A1h0_21, s); s = cre_dot_acc(A1h0_15, A1h0_19, s);
        total = total + R(142.0) * s;
      }
      {
        R s = cre_dot(A1h0_0, A1h0_5);
        s = cre_dot_acc(A1h0_0, A1h0_14, s); s = cre_dot_acc(A1h0_1, A1h0_3, s); s = cre_dot_acc(A1h0_1, A1h0_20, s);
        s = cre_dot_acc(A1h0_2, A1h0_4, s); s = cre_dot_acc(A1h0_2, A1h0_8, s); s = cre_dot_acc(A1h0_3, A1h0_22, s);
        s = cre_dot_acc(A1h0_4, A1h0_10, s); s = cre_dot_acc(A1h0_5, A1h0_16, s); s = cre_dot_acc(A1h0_6, A1h0_11, s);
        s = cre_dot_acc(A1h0_6, A1h0_12, s); s = cre_dot_acc(A1h0_7, A1h0_9, s); s = cre_dot_acc(A1h0_7, A1h0_18, s);
        s = cre_dot_acc(A1h0_8, A1h0_10, s); s = cre_dot_acc(A1h0_9, A1h0_23, s); s = cre_dot_acc(A1h0_11, A1h0_17, s);
        s = cre_dot_acc(A1h0_12, A1h0_17, s); s = cre_dot_acc(A1h0_13, A1h0_15, s); s = cre_dot_acc(A1h0_13, A1h0_19, s);
        s = cre_dot_acc(A1h0_14, A1h0_16, s); s = cre_dot_acc(A1h0_15, A1h0_21, s); s = cre_dot_acc(A1h0_18, A1h0_23, s);
        s = cre_dot_acc(A1h0_19, A1h0_21, s); s = cre_dot_acc(A1h0_20, A1h0_22, s);
        total = total + R(160.0) * s;
      }
      {
        R s = cabs2(A1h0_0);
        s = cabs2_acc(A1h0_1, s); s = cabs2_acc(A1h0_2, s); s = cabs2_acc(A1h0_3, s);
        s = cabs2_acc(A1h0_4, s); s = cabs2_acc(A1h0_5, s); s = cabs2_acc(A1h0_6, s);
        s = cabs2_acc(A1h0_7, s); s = cabs2_acc(A1h0_8, s); s = cabs2_acc(A1h0_9, s);
        s = cabs2_acc(A1h0_10, s); s = cabs2_acc(A1h0_11, s); s = cabs2_acc(A1h0_12, s);
        s = cabs2_acc(A1h0_13, s); s = cabs2_acc(A1h0_14, s); s = cabs2_acc(A1h0_15, s);
        s = cabs2_acc(A1h0_16, s); s = cabs2_acc(A1h0_17, s); s = cabs2_acc(A1h0_18, s);
        s = cabs2_acc(A1h0_19, s); s = cabs2_acc(A1h0_20, s); s = cabs2_acc(A1h0_21, s);
        s = cabs2_acc(A1h0_22, s); s = cabs2_acc(A1h0_23, s);
        total = total + R(512.0) * s;
      }
    }
  }
  return total * R(2.0 / 54.0);
}
}  // namespace mf
