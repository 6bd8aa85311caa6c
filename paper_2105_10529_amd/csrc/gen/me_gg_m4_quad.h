// Generated by gen_me.py for g g -> t t~ + 2 g (4 gluons on the top line,
// 24 colour orderings, 64 helicity/polarisation states): four lanes per event,
// six orderings each. Do not edit.
#pragma once
#include "amp.h"
namespace mf {
constexpr int ME_M4_QUAD_TAB = 68;  // table values per lane
// Colour- and polarisation-summed |M|^2 with g = 1, summed over the four
// lanes of the group (every lane returns it).  K[r], E[r]: outgoing momentum
// and polarisation vectors of gluon r ^ role, role = lane & 3; UB: ubar(top)
// of both helicities, VS: v(antitop) of helicity 0; tab: LDS, value i of
// this lane at tab[i * W].
template <class R, int W>
__device__ __forceinline__ R me_gg_m4_quad(const V4<R>* K, const V4<R> (*E)[2], const Sp<R>* UB, const Sp<R>& VS,
                                           const V4<R>& PTB, R MT, int role, R* tab) {
#pragma unroll
  for (int i = 0; i < 8; ++i) quad_put4<W>(tab + 4 * i * W, E[i >> 1][i & 1]);
  quad_put_sp<W>(tab + 32 * W, UB[0]);
  quad_put_sp<W>(tab + 40 * W, UB[1]);
  quad_put_sp<W>(tab + 48 * W, VS);
  { const V4<R> P = K[0] + K[1]; tab[56 * W] = R(-1.0) / mdot(P, P); }
  { const V4<R> P = K[0] + K[2]; tab[57 * W] = R(-1.0) / mdot(P, P); }
  { const V4<R> P = K[0] + K[1] + K[2]; tab[58 * W] = R(-1.0) / mdot(P, P); }
  { const V4<R> P = K[0] + K[3]; tab[59 * W] = R(-1.0) / mdot(P, P); }
  { const V4<R> P = K[0] + K[1] + K[2] + K[3]; tab[60 * W] = R(-1.0) / mdot(P, P); }
  { const V4<R> P = K[3]; tab[61 * W] = R(-1.0) / (R(2.0) * mdot(PTB, P) + mdot(P, P)); }
  { const V4<R> P = K[0] + K[3]; tab[62 * W] = R(-1.0) / (R(2.0) * mdot(PTB, P) + mdot(P, P)); }
  { const V4<R> P = K[1] + K[3]; tab[63 * W] = R(-1.0) / (R(2.0) * mdot(PTB, P) + mdot(P, P)); }
  { const V4<R> P = K[0] + K[1] + K[3]; tab[64 * W] = R(-1.0) / (R(2.0) * mdot(PTB, P) + mdot(P, P)); }
  { const V4<R> P = K[2] + K[3]; tab[65 * W] = R(-1.0) / (R(2.0) * mdot(PTB, P) + mdot(P, P)); }
  { const V4<R> P = K[0] + K[2] + K[3]; tab[66 * W] = R(-1.0) / (R(2.0) * mdot(PTB, P) + mdot(P, P)); }
  { const V4<R> P = K[1] + K[2] + K[3]; tab[67 * W] = R(-1.0) / (R(2.0) * mdot(PTB, P) + mdot(P, P)); }
  R total = R(0.0);
#pragma unroll 1
  for (int hg = 0; hg < 16; ++hg) {
    // bit r: the polarisation of gluon r ^ role (gluon 0 is bit 3 of hg)
    const int hr = quad_roles(hg, role);
    const V4<R> E0 = quad_get4<W>(tab + (4 * (0 + ((hr >> 0) & 1))) * W);
    const V4<R> E1 = quad_get4<W>(tab + (4 * (2 + ((hr >> 1) & 1))) * W);
    const V4<R> E2 = quad_get4<W>(tab + (4 * (4 + ((hr >> 2) & 1))) * W);
    const V4<R> E3 = quad_get4<W>(tab + (4 * (6 + ((hr >> 3) & 1))) * W);
    V4<R> J0 = E0; opaque4(J0);
    V4<R> k0 = K[0]; opaque4(k0);
    V4<R> J1 = E1; opaque4(J1);
    V4<R> k1 = K[1]; opaque4(k1);
    V4<R> J2 = E2; opaque4(J2);
    V4<R> k2 = K[2]; opaque4(k2);
    V4<R> J3 = E3; opaque4(J3);
    V4<R> k3 = K[3]; opaque4(k3);
    V4<R> pb = PTB; opaque4(pb);
    int z_ = 0; opaque(z_);
    V4<R> J01 = tab[z_ + 56 * W] * (v3(J0, J1, k0, k1));
    V4<R> J02 = tab[z_ + 57 * W] * (v3(J0, J2, k0, k2));
    V4<R> J03 = tab[z_ + 59 * W] * (v3(J0, J3, k0, k3));
    const V4<R> J12 = quad4<QX1>(J03);
    const V4<R> p6 = k1 + k2;
    const V4<R> p3 = k0 + k1;
    V4<R> J012 = tab[z_ + 58 * W] * (w4_sub(J0, J1, J2, v3_acc(J01, J2, p3, k2, v3(J0, J12, k0, p6))));
    const V4<R> p5 = k0 + k2;
    const V4<R> J10 = R(-1.0) * J01;
    V4<R> J102 = tab[z_ + 58 * W] * (w4_sub(J1, J0, J2, v3_acc(J10, J2, p3, k2, v3(J1, J02, k1, p5))));
    const V4<R> J21 = R(-1.0) * J12;
    V4<R> J021 = tab[z_ + 58 * W] * (w4_sub(J0, J2, J1, v3_acc(J02, J1, p5, k1, v3(J0, J21, k0, p6))));
    Sp<R> S_3;
    C2<R> A0_0, A1_0, A0_1, A1_1, A0_2, A1_2, A0_3, A1_3, A0_4, A1_4, A0_5, A1_5;
    {  // orderings (x, y, 0, 3)
      opaque4(J0);
      opaque4(J01);
      opaque4(J012);
      opaque4(J02);
      opaque4(J021);
      opaque4(J03);
      opaque4(J1);
      opaque4(J102);
      opaque4(J2);
      opaque4(J3);
      opaque4(k0); opaque4(k1); opaque4(k2); opaque4(k3); opaque4(pb); opaque(z_);
      const Sp<R> S_ = quad_get_sp<W>(tab + z_ + 48 * W);
      S_3 = prop_neg(pb + k3, MT, tab[z_ + 61 * W], slash(J3, S_));
      const V4<R> p9 = k0 + k3;
      const Sp<R> S_03 = prop_neg(pb + p9, MT, tab[z_ + 62 * W], slash_acc(J03, S_, slash(J0, S_3)));
      const V4<R> J20 = R(-1.0) * J02;
      const V4<R> J203 = quad4<QX2>(J021);
      const V4<R> p13 = k0 + k2 + k3;
      const Sp<R> S_203 = prop_neg(pb + p13, MT, tab[z_ + 66 * W], slash_acc(J203, S_, slash_acc(J20, S_3, slash(J2, S_03))));
      const V4<R> J12 = quad4<QX1>(J03);
      const V4<R> p6 = k1 + k2;
      const V4<R> p7 = k0 + k1 + k2;
      const V4<R> J1203 = tab[z_ + 60 * W] * (w4_sub(J12, J0, J3, w4_sub(J1, J20, J3, w4_sub(J1, J2, J03, v3_acc(J021, J3, p7, k3, v3_acc(J12, J03, p6, p9, v3(J1, J203, k1, p13)))))));
      const Sp<R> F3 = slash_acc(J1203, S_, slash_acc(J021, S_3, slash_acc(J12, S_03, slash(J1, S_203))));
      A0_3 = ubar_dot(quad_get_sp<W>(tab + z_ + 32 * W), F3);
      A1_3 = ubar_dot(quad_get_sp<W>(tab + z_ + 40 * W), F3);
      opaque(z_);
      const V4<R> J10 = R(-1.0) * J01;
      const V4<R> J103 = quad4<QX1>(J012);
      const V4<R> p11 = k0 + k1 + k3;
      const Sp<R> S_103 = prop_neg(pb + p11, MT, tab[z_ + 64 * W], slash_acc(J103, S_, slash_acc(J10, S_3, slash(J1, S_03))));
      const V4<R> J21 = R(-1.0) * J12;
      const V4<R> J2103 = tab[z_ + 60 * W] * (w4_sub(J21, J0, J3, w4_sub(J2, J10, J3, w4_sub(J2, J1, J03, v3_acc(J012, J3, p7, k3, v3_acc(J21, J03, p6, p9, v3(J2, J103, k2, p11)))))));
      const Sp<R> F5 = slash_acc(J2103, S_, slash_acc(J012, S_3, slash_acc(J21, S_03, slash(J2, S_103))));
      A0_5 = ubar_dot(quad_get_sp<W>(tab + z_ + 32 * W), F5);
      A1_5 = ubar_dot(quad_get_sp<W>(tab + z_ + 40 * W), F5);
      opaque(z_);
    }
    {  // orderings (x, y, 1, 3)
      opaque4(J0);
      opaque4(J01);
      opaque4(J012);
      opaque4(J02);
      opaque4(J021);
      opaque4(J03);
      opaque4(J1);
      opaque4(J102);
      opaque4(J2);
      opaque4(J3);
      opaque4(k0); opaque4(k1); opaque4(k2); opaque4(k3); opaque4(pb); opaque(z_);
      const Sp<R> S_ = quad_get_sp<W>(tab + z_ + 48 * W);
      opaque_sp(S_3);
      const V4<R> J13 = quad4<QX1>(J02);
      const V4<R> p10 = k1 + k3;
      const Sp<R> S_13 = prop_neg(pb + p10, MT, tab[z_ + 63 * W], slash_acc(J13, S_, slash(J1, S_3)));
      const V4<R> J12 = quad4<QX1>(J03);
      const V4<R> J21 = R(-1.0) * J12;
      const V4<R> J312 = quad4<QX3>(J021);
      const V4<R> p14 = k1 + k2 + k3;
      const Sp<R> S_213 = prop_neg(pb + p14, MT, tab[z_ + 67 * W], slash_acc(J312, S_, slash_acc(J21, S_3, slash(J2, S_13))));
      const V4<R> p5 = k0 + k2;
      const V4<R> p7 = k0 + k1 + k2;
      const V4<R> J0213 = tab[z_ + 60 * W] * (w4_sub(J02, J1, J3, w4_sub(J0, J21, J3, w4_sub(J0, J2, J13, v3_acc(J021, J3, p7, k3, v3_acc(J02, J13, p5, p10, v3(J0, J312, k0, p14)))))));
      const Sp<R> F1 = slash_acc(J0213, S_, slash_acc(J021, S_3, slash_acc(J02, S_13, slash(J0, S_213))));
      A0_1 = ubar_dot(quad_get_sp<W>(tab + z_ + 32 * W), F1);
      A1_1 = ubar_dot(quad_get_sp<W>(tab + z_ + 40 * W), F1);
      opaque(z_);
      const V4<R> J013 = quad4<QX1>(J102);
      const V4<R> p11 = k0 + k1 + k3;
      const Sp<R> S_013 = prop_neg(pb + p11, MT, tab[z_ + 64 * W], slash_acc(J013, S_, slash_acc(J01, S_3, slash(J0, S_13))));
      const V4<R> J20 = R(-1.0) * J02;
      const V4<R> J2013 = tab[z_ + 60 * W] * (w4_sub(J20, J1, J3, w4_sub(J2, J01, J3, w4_sub(J2, J0, J13, v3_acc(J102, J3, p7, k3, v3_acc(J20, J13, p5, p10, v3(J2, J013, k2, p11)))))));
      const Sp<R> F4 = slash_acc(J2013, S_, slash_acc(J102, S_3, slash_acc(J20, S_13, slash(J2, S_013))));
      A0_4 = ubar_dot(quad_get_sp<W>(tab + z_ + 32 * W), F4);
      A1_4 = ubar_dot(quad_get_sp<W>(tab + z_ + 40 * W), F4);
      opaque(z_);
    }
    {  // orderings (x, y, 2, 3)
      opaque4(J0);
      opaque4(J01);
      opaque4(J012);
      opaque4(J02);
      opaque4(J021);
      opaque4(J03);
      opaque4(J1);
      opaque4(J102);
      opaque4(J2);
      opaque4(J3);
      opaque4(k0); opaque4(k1); opaque4(k2); opaque4(k3); opaque4(pb); opaque(z_);
      const Sp<R> S_ = quad_get_sp<W>(tab + z_ + 48 * W);
      opaque_sp(S_3);
      const V4<R> J23 = quad4<QX2>(J01);
      const V4<R> p12 = k2 + k3;
      const Sp<R> S_23 = prop_neg(pb + p12, MT, tab[z_ + 65 * W], slash_acc(J23, S_, slash(J2, S_3)));
      const V4<R> J12 = quad4<QX1>(J03);
      const V4<R> J321 = quad4<QX3>(J012);
      const V4<R> p14 = k1 + k2 + k3;
      const Sp<R> S_123 = prop_neg(pb + p14, MT, tab[z_ + 67 * W], slash_acc(J321, S_, slash_acc(J12, S_3, slash(J1, S_23))));
      const V4<R> p3 = k0 + k1;
      const V4<R> p7 = k0 + k1 + k2;
      const V4<R> J0123 = tab[z_ + 60 * W] * (w4_sub(J01, J2, J3, w4_sub(J0, J12, J3, w4_sub(J0, J1, J23, v3_acc(J012, J3, p7, k3, v3_acc(J01, J23, p3, p12, v3(J0, J321, k0, p14)))))));
      const Sp<R> F0 = slash_acc(J0123, S_, slash_acc(J012, S_3, slash_acc(J01, S_23, slash(J0, S_123))));
      A0_0 = ubar_dot(quad_get_sp<W>(tab + z_ + 32 * W), F0);
      A1_0 = ubar_dot(quad_get_sp<W>(tab + z_ + 40 * W), F0);
      opaque(z_);
      const V4<R> J320 = quad4<QX2>(J102);
      const V4<R> p13 = k0 + k2 + k3;
      const Sp<R> S_023 = prop_neg(pb + p13, MT, tab[z_ + 66 * W], slash_acc(J320, S_, slash_acc(J02, S_3, slash(J0, S_23))));
      const V4<R> J10 = R(-1.0) * J01;
      const V4<R> J1023 = tab[z_ + 60 * W] * (w4_sub(J10, J2, J3, w4_sub(J1, J02, J3, w4_sub(J1, J0, J23, v3_acc(J102, J3, p7, k3, v3_acc(J10, J23, p3, p12, v3(J1, J320, k1, p13)))))));
      const Sp<R> F2 = slash_acc(J1023, S_, slash_acc(J102, S_3, slash_acc(J10, S_23, slash(J1, S_023))));
      A0_2 = ubar_dot(quad_get_sp<W>(tab + z_ + 32 * W), F2);
      A1_2 = ubar_dot(quad_get_sp<W>(tab + z_ + 40 * W), F2);
      opaque(z_);
    }
    {
      const C2<R> B0 = A0_0;
      const C2<R> B1 = A0_1;
      const C2<R> B2 = A0_2;
      const C2<R> B3 = A0_3;
      const C2<R> B4 = A0_4;
      const C2<R> B5 = A0_5;
      total = total + R(-128.0) * cre_dot_acc(A0_4, B5, cre_dot_acc(A0_3, B5, cre_dot_acc(A0_2, B3, cre_dot_acc(A0_1, B4, cre_dot_acc(A0_0, B2, cre_dot(A0_0, B1))))));
      total = total + R(16.0) * cre_dot_acc(A0_3, B4, cre_dot_acc(A0_2, B5, cre_dot_acc(A0_1, B5, cre_dot_acc(A0_1, B2, cre_dot_acc(A0_0, B4, cre_dot(A0_0, B3))))));
      total = total + R(160.0) * cre_dot_acc(A0_2, B4, cre_dot_acc(A0_1, B3, cre_dot(A0_0, B5)));
      total = total + R(512.0) * cre_dot_acc(A0_5, B5, cre_dot_acc(A0_4, B4, cre_dot_acc(A0_3, B3, cre_dot_acc(A0_2, B2, cre_dot_acc(A0_1, B1, cre_dot(A0_0, B0))))));
    }
    {
      const C2<R> B0 = A1_0;
      const C2<R> B1 = A1_1;
      const C2<R> B2 = A1_2;
      const C2<R> B3 = A1_3;
      const C2<R> B4 = A1_4;
      const C2<R> B5 = A1_5;
      total = total + R(-128.0) * cre_dot_acc(A1_4, B5, cre_dot_acc(A1_3, B5, cre_dot_acc(A1_2, B3, cre_dot_acc(A1_1, B4, cre_dot_acc(A1_0, B2, cre_dot(A1_0, B1))))));
      total = total + R(16.0) * cre_dot_acc(A1_3, B4, cre_dot_acc(A1_2, B5, cre_dot_acc(A1_1, B5, cre_dot_acc(A1_1, B2, cre_dot_acc(A1_0, B4, cre_dot(A1_0, B3))))));
      total = total + R(160.0) * cre_dot_acc(A1_2, B4, cre_dot_acc(A1_1, B3, cre_dot(A1_0, B5)));
      total = total + R(512.0) * cre_dot_acc(A1_5, B5, cre_dot_acc(A1_4, B4, cre_dot_acc(A1_3, B3, cre_dot_acc(A1_2, B2, cre_dot_acc(A1_1, B1, cre_dot(A1_0, B0))))));
    }
    {
      const C2<R> B0 = quad2<QX1>(A0_0);
      const C2<R> B1 = quad2<QX1>(A0_1);
      const C2<R> B2 = quad2<QX1>(A0_2);
      const C2<R> B3 = quad2<QX1>(A0_3);
      const C2<R> B4 = quad2<QX1>(A0_4);
      const C2<R> B5 = quad2<QX1>(A0_5);
      total = total + R(-128.0) * cre_dot(A0_0, B2);
      total = total + R(-28.0) * cre_dot_acc(A0_5, B5, cre_dot(A0_4, B4));
      total = total + R(-20.0) * cre_dot_acc(A0_3, B4, cre_dot_acc(A0_2, B5, cre_dot_acc(A0_1, B5, cre_dot(A0_0, B4))));
      total = total + R(-2.0) * cre_dot_acc(A0_2, B4, cre_dot_acc(A0_2, B3, cre_dot_acc(A0_0, B5, cre_dot(A0_0, B1))));
      total = total + R(8.0) * cre_dot_acc(A0_2, B2, cre_dot(A0_0, B0));
      total = total + R(16.0) * cre_dot_acc(A0_1, B2, cre_dot(A0_0, B3));
      total = total + R(71.0) * cre_dot_acc(A0_3, B3, cre_dot(A0_1, B1));
      total = total + R(124.0) * cre_dot_acc(A0_4, B5, cre_dot_acc(A0_3, B5, cre_dot(A0_1, B4)));
      total = total + R(160.0) * cre_dot(A0_1, B3);
    }
    {
      const C2<R> B0 = quad2<QX1>(A1_0);
      const C2<R> B1 = quad2<QX1>(A1_1);
      const C2<R> B2 = quad2<QX1>(A1_2);
      const C2<R> B3 = quad2<QX1>(A1_3);
      const C2<R> B4 = quad2<QX1>(A1_4);
      const C2<R> B5 = quad2<QX1>(A1_5);
      total = total + R(-128.0) * cre_dot(A1_0, B2);
      total = total + R(-28.0) * cre_dot_acc(A1_5, B5, cre_dot(A1_4, B4));
      total = total + R(-20.0) * cre_dot_acc(A1_3, B4, cre_dot_acc(A1_2, B5, cre_dot_acc(A1_1, B5, cre_dot(A1_0, B4))));
      total = total + R(-2.0) * cre_dot_acc(A1_2, B4, cre_dot_acc(A1_2, B3, cre_dot_acc(A1_0, B5, cre_dot(A1_0, B1))));
      total = total + R(8.0) * cre_dot_acc(A1_2, B2, cre_dot(A1_0, B0));
      total = total + R(16.0) * cre_dot_acc(A1_1, B2, cre_dot(A1_0, B3));
      total = total + R(71.0) * cre_dot_acc(A1_3, B3, cre_dot(A1_1, B1));
      total = total + R(124.0) * cre_dot_acc(A1_4, B5, cre_dot_acc(A1_3, B5, cre_dot(A1_1, B4)));
      total = total + R(160.0) * cre_dot(A1_1, B3);
    }
    {
      const C2<R> B0 = quad2<QX2>(A0_0);
      const C2<R> B1 = quad2<QX2>(A0_1);
      const C2<R> B2 = quad2<QX2>(A0_2);
      const C2<R> B3 = quad2<QX2>(A0_3);
      const C2<R> B4 = quad2<QX2>(A0_4);
      const C2<R> B5 = quad2<QX2>(A0_5);
      total = total + R(-128.0) * cre_dot(A0_1, B4);
      total = total + R(-28.0) * cre_dot_acc(A0_3, B3, cre_dot(A0_2, B2));
      total = total + R(-20.0) * cre_dot_acc(A0_3, B4, cre_dot_acc(A0_2, B5, cre_dot_acc(A0_1, B2, cre_dot(A0_0, B3))));
      total = total + R(-2.0) * cre_dot_acc(A0_4, B5, cre_dot_acc(A0_2, B4, cre_dot_acc(A0_1, B3, cre_dot(A0_0, B1))));
      total = total + R(8.0) * cre_dot_acc(A0_4, B4, cre_dot(A0_1, B1));
      total = total + R(16.0) * cre_dot_acc(A0_1, B5, cre_dot(A0_0, B4));
      total = total + R(71.0) * cre_dot_acc(A0_5, B5, cre_dot(A0_0, B0));
      total = total + R(124.0) * cre_dot_acc(A0_3, B5, cre_dot_acc(A0_2, B3, cre_dot(A0_0, B2)));
      total = total + R(160.0) * cre_dot(A0_0, B5);
    }
    {
      const C2<R> B0 = quad2<QX2>(A1_0);
      const C2<R> B1 = quad2<QX2>(A1_1);
      const C2<R> B2 = quad2<QX2>(A1_2);
      const C2<R> B3 = quad2<QX2>(A1_3);
      const C2<R> B4 = quad2<QX2>(A1_4);
      const C2<R> B5 = quad2<QX2>(A1_5);
      total = total + R(-128.0) * cre_dot(A1_1, B4);
      total = total + R(-28.0) * cre_dot_acc(A1_3, B3, cre_dot(A1_2, B2));
      total = total + R(-20.0) * cre_dot_acc(A1_3, B4, cre_dot_acc(A1_2, B5, cre_dot_acc(A1_1, B2, cre_dot(A1_0, B3))));
      total = total + R(-2.0) * cre_dot_acc(A1_4, B5, cre_dot_acc(A1_2, B4, cre_dot_acc(A1_1, B3, cre_dot(A1_0, B1))));
      total = total + R(8.0) * cre_dot_acc(A1_4, B4, cre_dot(A1_1, B1));
      total = total + R(16.0) * cre_dot_acc(A1_1, B5, cre_dot(A1_0, B4));
      total = total + R(71.0) * cre_dot_acc(A1_5, B5, cre_dot(A1_0, B0));
      total = total + R(124.0) * cre_dot_acc(A1_3, B5, cre_dot_acc(A1_2, B3, cre_dot(A1_0, B2)));
      total = total + R(160.0) * cre_dot(A1_0, B5);
    }
    {
      const C2<R> B0 = quad2<QX3>(A0_0);
      const C2<R> B1 = quad2<QX3>(A0_1);
      const C2<R> B2 = quad2<QX3>(A0_2);
      const C2<R> B3 = quad2<QX3>(A0_3);
      const C2<R> B4 = quad2<QX3>(A0_4);
      const C2<R> B5 = quad2<QX3>(A0_5);
      total = total + R(-128.0) * cre_dot(A0_3, B5);
      total = total + R(-28.0) * cre_dot_acc(A0_1, B1, cre_dot(A0_0, B0));
      total = total + R(-20.0) * cre_dot_acc(A0_1, B5, cre_dot_acc(A0_1, B2, cre_dot_acc(A0_0, B4, cre_dot(A0_0, B3))));
      total = total + R(-2.0) * cre_dot_acc(A0_4, B5, cre_dot_acc(A0_2, B3, cre_dot_acc(A0_1, B3, cre_dot(A0_0, B5))));
      total = total + R(8.0) * cre_dot_acc(A0_5, B5, cre_dot(A0_3, B3));
      total = total + R(16.0) * cre_dot_acc(A0_3, B4, cre_dot(A0_2, B5));
      total = total + R(71.0) * cre_dot_acc(A0_4, B4, cre_dot(A0_2, B2));
      total = total + R(124.0) * cre_dot_acc(A0_1, B4, cre_dot_acc(A0_0, B2, cre_dot(A0_0, B1)));
      total = total + R(160.0) * cre_dot(A0_2, B4);
    }
    {
      const C2<R> B0 = quad2<QX3>(A1_0);
      const C2<R> B1 = quad2<QX3>(A1_1);
      const C2<R> B2 = quad2<QX3>(A1_2);
      const C2<R> B3 = quad2<QX3>(A1_3);
      const C2<R> B4 = quad2<QX3>(A1_4);
      const C2<R> B5 = quad2<QX3>(A1_5);
      total = total + R(-128.0) * cre_dot(A1_3, B5);
      total = total + R(-28.0) * cre_dot_acc(A1_1, B1, cre_dot(A1_0, B0));
      total = total + R(-20.0) * cre_dot_acc(A1_1, B5, cre_dot_acc(A1_1, B2, cre_dot_acc(A1_0, B4, cre_dot(A1_0, B3))));
      total = total + R(-2.0) * cre_dot_acc(A1_4, B5, cre_dot_acc(A1_2, B3, cre_dot_acc(A1_1, B3, cre_dot(A1_0, B5))));
      total = total + R(8.0) * cre_dot_acc(A1_5, B5, cre_dot(A1_3, B3));
      total = total + R(16.0) * cre_dot_acc(A1_3, B4, cre_dot(A1_2, B5));
      total = total + R(71.0) * cre_dot_acc(A1_4, B4, cre_dot(A1_2, B2));
      total = total + R(124.0) * cre_dot_acc(A1_1, B4, cre_dot_acc(A1_0, B2, cre_dot(A1_0, B1)));
      total = total + R(160.0) * cre_dot(A1_2, B4);
    }
  }
  total = total + quad1<QX1>(total);
  total = total + quad1<QX2>(total);
  return total * R(2.0 / 54.0);
}
}  // namespace mf
