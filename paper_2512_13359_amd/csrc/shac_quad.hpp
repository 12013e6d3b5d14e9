// The paper task's control step and its reverse-mode derivative with four lanes per
// environment (the layout of quad_env.hpp: lanes c = 0, 1, 2 of a quad hold the x, y, z
// components of every 3-vector and of the quaternion's vector part, lane 3 the quaternion's
// scalar part and zero in 3-vectors).  Same equations as the one-lane form in
// shac_adjoint.hpp, against which a host check compares every function in double.
//
// Cross products: with P1, P2 the quad permutations that read component c + 1, c + 2,
// x x y = P1(x . P1 y) - P2(x . P2 y) (elementwise products).  The permutations are linear, and
// a per-component factor f moves inside them (f . P1 z = P1(z . P2 f), f . P2 z = P2(z . P1 f)),
// so each output that is a sum of cross products takes one P1 and one P2.
//
// Written on a lane type T: float on the device (the permutations are DPP moves), and on the
// host a type that holds the four lanes.  T needs + - *, p1, p2, bcz, bcw (component z, scalar
// part in every lane), sum4, abs_, products with scalars, and elementwise rsqrt_, sign_of, ka_of
// and att_factors (the scalars of the attitude error below).
#pragma once

#if defined(__HIPCC__)
#include "quad_env.hpp"
#define AUV_QD __device__ __forceinline__
#else
#define AUV_QD inline
#endif

namespace auv {
namespace qadj {

#if defined(__HIPCC__)
__device__ __forceinline__ float p1(float x) { return quad::dpp<quad::P1>(x); }
__device__ __forceinline__ float p2(float x) { return quad::dpp<quad::P2>(x); }
__device__ __forceinline__ float bcz(float x) { return quad::dpp<quad::BC2>(x); }
__device__ __forceinline__ float bcw(float x) { return quad::dpp<quad::BC3>(x); }
__device__ __forceinline__ float sum4(float x) { return quad::qsum(x); }
__device__ __forceinline__ float abs_(float x) { return fabsf(x); }
__device__ __forceinline__ float rsqrt_(float x) { return 1.0f / sqrtf(x); }
__device__ __forceinline__ float sign_of(float x) { return x < 0.0f ? -1.0f : 1.0f; }
__device__ __forceinline__ float ka_of(float n2, float ew) { return -2.0f / (n2 + ew * ew); }
// k = 2 atan2(n, aw) / n with the sign of the scalar part in sk, and kn = (dk/dn) / n (by its
// series for small n / aw), n = sqrt(n2), aw = |ew|; ka_of: dk/daw
__device__ __forceinline__ void att_factors(float n2, float ew, float& sk, float& kn) {
  const float n = sqrtf(n2), aw = fabsf(ew), at = 2.0f * atan2f(n, aw);
  const float k = n > 0.0f ? at / n : 2.0f / aw;
  const float t2 = n2 / (aw * aw);
  const float series = 2.0f / (aw * aw * aw) * (-2.0f / 3.0f + t2 * (0.8f + t2 * (-6.0f / 7.0f + t2 * (8.0f / 9.0f))));
  const float closed = (2.0f * aw * n / (n2 + aw * aw) - at) / (n2 * n);
  kn = n < 0.1f * aw ? series : closed;
  sk = ew < 0.0f ? -k : k;
}
#endif

// Lane masks: vector lanes, scalar lane, and the lanes of x, y, z.
template <class T>
struct LaneK {
  T m3, w3, ex, ey, ez;
};

// Model constants of a lane's component (zero in lane 3).  1 and 2: component c + 1, c + 2.
template <class T>
struct QM {
  T iMl, KF1, KF2;         // 1 / Mlin; Mlin_c / Mlin_{c+2}, Mlin_c / Mlin_{c+1}
  T DLi, DQi, BmWi;        // linear-axis damping and (B - gamma W), over Mlin
  T Ma, iMa, A1, DLa, DQa; // angular inertia, linear added mass (Munk term), angular damping
  T Ml, Ml1, Ml2;          // Mlin and its neighbours
  T dM1, dM2, dA1, dA2;    // Ma_{c+1} - Ma_c, Ma_{c+2} - Ma_c; the same of A1
};

template <class T>
AUV_QD void derive(QM<T>& M) {   // the constants formed from Ml, iMl, Ma, A1
  M.Ml1 = p1(M.Ml);
  M.Ml2 = p2(M.Ml);
  M.KF1 = M.Ml * p2(M.iMl);
  M.KF2 = M.Ml * p1(M.iMl);
  M.dM1 = p1(M.Ma) - M.Ma;
  M.dM2 = p2(M.Ma) - M.Ma;
  M.dA1 = p1(M.A1) - M.A1;
  M.dA2 = p2(M.A1) - M.A1;
}

// (q, v, omega) of one environment, or a cotangent of them.
template <class T>
struct QX {
  T q, v, w;
};

// Right side for tfi = tau_f / Mlin and tm = tau_m.
template <class T>
AUV_QD void rhs(const LaneK<T>& K, const QM<T>& M, T tfi, T tm, const QX<T>& x, T& dp, QX<T>& d) {
  const T e = x.q * K.m3, wb = bcw(x.q), e1 = p1(e), e2 = p2(e);
  const T w2 = wb + wb, E2 = e + e, g1 = w2 * e1, g2 = w2 * e2;
  const T s = 1.0f - 2.0f * sum4(e * e);
  dp = sum4(E2 * x.v) * e + s * x.v + p2(g2 * x.v) - p1(g1 * x.v);
  const T k = bcz(E2) * e + s * K.ez - g1 * K.ex + g2 * K.ey;
  const T o1 = p1(x.w), o2 = p2(x.w), v1 = p1(x.v), v2 = p2(x.v);
  d.v = tfi - (M.DQi * abs_(x.v) + M.DLi) * x.v - M.BmWi * k + p1(x.v * o1 * M.KF1) - p2(x.v * o2 * M.KF2);
  const T b = M.Ma * x.w, a = M.A1 * x.v;
  d.w = (tm - (M.DQa * abs_(x.w) + M.DLa) * x.w + p1(b * o1 + a * v1) - p2(b * o2 + a * v2)) * M.iMa;
  d.q = 0.5f * (K.m3 * (wb * x.w + (e1 * o2 - e2 * o1)) - K.w3 * sum4(e * x.w));
}

// Cotangent (gp, g) of the derivative at x -> cotangent h of x; gtf, gtm += that of the wrench.
template <class T>
AUV_QD void rhs_vjp(const LaneK<T>& K, const QM<T>& M, const QX<T>& x, T gp, const QX<T>& g, QX<T>& h, T& gtf, T& gtm) {
  const T e = x.q * K.m3, wb = bcw(x.q), e1 = p1(e), e2 = p2(e);
  const T w2 = wb + wb, g1 = w2 * e1, g2 = w2 * e2;
  const T s = 1.0f - 2.0f * sum4(e * e);
  const T gF = g.v * M.iMl, gG = g.w * M.iMa;
  gtf = gtf + gF;
  gtm = gtm + gG;
  const T f1 = p1(gF), f2 = p2(gF), G1 = p1(gG), G2 = p2(gG);
  const T a = M.Ml * x.v;
  const T gqv = 0.5f * (g.q * K.m3), gqs = 0.5f * bcw(g.q);
  // omega: gF x (Ml v) + gG x (Ma w) + Ma (w x gG), damping, and 1/2 (w gq + gq x e - gqs e)
  h.w = p1(x.w * G1 * M.dM2 - a * f1 + gqv * e1) + p2(a * f2 - x.w * G2 * M.dM1 - gqv * e2) -
        gG * (M.DLa + 2.0f * M.DQa * abs_(x.w)) + wb * gqv - gqs * e;
  // v: Ml (w x gF) + gG x (A1 v) + A1 (v x gG), damping, and R^T gp
  const T eg = sum4(e * gp), ev = sum4(e * x.v);
  h.v = p1(x.w * f1 * M.Ml2 + x.v * G1 * M.dA2 + g1 * gp) - p2(x.w * f2 * M.Ml1 + x.v * G2 * M.dA1 + g2 * gp) -
        g.v * (M.DLi + 2.0f * M.DQi * abs_(x.v)) + s * gp + 2.0f * eg * e;
  // q: through R v (cotangent gp) and k = R^T e3 (cotangent gk), and the kinematics
  const T gk = -1.0f * (M.BmWi * g.v);
  const T z1 = x.v * p1(gp) + gk * K.ey, z2 = x.v * p2(gp) + gk * K.ex;
  const T sc = sum4(gp * x.v + gk * K.ez), egk = sum4(e * gk);
  const T he = 2.0f * (eg * x.v + ev * gp + bcz(e) * gk + egk * K.ez - 2.0f * sc * e) +
               p1(w2 * z1 - gqv * p1(x.w)) - p2(w2 * z2 - gqv * p2(x.w)) - gqs * x.w;
  h.q = he + K.w3 * sum4(2.0f * (z1 * e2 - z2 * e1) + 0.5f * (x.w * g.q));
}

// One RK4 substep of length h (scalar type S), the quaternion divided by its norm.  st: the
// four stage inputs; inv: 1 / |q| before the division.
template <class T, class S>
AUV_QD void substep(const LaneK<T>& K, const QM<T>& M, T tfi, T tm, S h, T& p, QX<T>& x, QX<T> st[4], T& inv) {
  QX<T> d, acc;
  T dp, ap;
  st[0] = x;
  rhs(K, M, tfi, tm, x, ap, acc);
  d = acc;
#if defined(__HIPCC__)
#pragma unroll
#endif
  for (int i = 1; i < 4; ++i) {
    const S cs = i == 3 ? h : S(0.5f) * h, wt = i == 3 ? S(1) : S(2);
    st[i] = QX<T>{x.q + cs * d.q, x.v + cs * d.v, x.w + cs * d.w};
    rhs(K, M, tfi, tm, st[i], dp, d);
    ap = ap + wt * dp;
    acc = QX<T>{acc.q + wt * d.q, acc.v + wt * d.v, acc.w + wt * d.w};
  }
  const S h6 = h / S(6);
  p = p + h6 * ap;
  x = QX<T>{x.q + h6 * acc.q, x.v + h6 * acc.v, x.w + h6 * acc.w};
  inv = rsqrt_(sum4(x.q * x.q));
  x.q = x.q * inv;
}

// (lp, l): cotangent of the substep's end on entry, of its start on return.  qn: the end
// quaternion; st, inv as substep() gave them.
template <class T, class S>
AUV_QD void substep_vjp(const LaneK<T>& K, const QM<T>& M, S h, const QX<T> st[4], T inv, T qn, T lp, QX<T>& l, T& gtf,
                        T& gtm) {
  l.q = (l.q - qn * sum4(qn * l.q)) * inv;
  const S h6 = h / S(6);
  const T gp = h6 * lp, gp2 = gp + gp;
  const QX<T> gk{h6 * l.q, h6 * l.v, h6 * l.w};
  QX<T> g = gk, r;
#if defined(__HIPCC__)
#pragma unroll
#endif
  for (int i = 3; i >= 0; --i) {
    rhs_vjp(K, M, st[i], (i == 3 || i == 0) ? gp : gp2, g, r, gtf, gtm);
    l = QX<T>{l.q + r.q, l.v + r.v, l.w + r.w};
    if (i > 0) {   // cotangent of the stage before: its weight times gk, and its share of this stage's input
      const S c = i == 3 ? h : S(0.5f) * h, wt = i == 1 ? S(1) : S(2);
      g = QX<T>{wt * gk.q + c * r.q, wt * gk.v + c * r.v, wt * gk.w + c * r.w};
    }
  }
}

// The observation's position error and rotation vector rv = sk ev, and the factors sk and kn
// that its derivative needs.
template <class T>
struct QObsK {
  T dpb, rv, sk, kn;
};

// Scalars of the attitude error: error vector ev, its norm's square n2, scalar part ew.
template <class T>
AUV_QD void att_error(const LaneK<T>& K, T q, T qg, T& ev, T& n2, T& ew) {
  const T e = q * K.m3, er = qg * K.m3;
  ew = sum4(q * qg);
  ev = bcw(q) * er - bcw(qg) * e - (p1(e * p1(er)) - p2(e * p2(er)));
  n2 = sum4(ev * ev);
}

template <class T>
AUV_QD QObsK<T> observe(const LaneK<T>& K, T p, T q, T pg, T qg) {
  const T e = q * K.m3, wb = bcw(q), w2 = wb + wb, d = pg - p;
  const T s = 1.0f - 2.0f * sum4(e * e);
  QObsK<T> o;
  o.dpb = s * d + 2.0f * sum4(e * d) * e + p1(w2 * (p1(e) * d)) - p2(w2 * (p2(e) * d));
  T ev, n2, ew;
  att_error(K, q, qg, ev, n2, ew);
  att_factors(n2, ew, o.sk, o.kn);
  o.rv = o.sk * ev;
  return o;
}

// (lp, lq) += cotangent of (p, q) for the cotangents gd of dpb and gr of the rotation vector.
template <class T>
AUV_QD void observe_vjp(const LaneK<T>& K, T p, T q, T pg, T qg, T sk, T kn, T gd, T gr, T& lp, T& lq) {
  const T e = q * K.m3, wb = bcw(q), e1 = p1(e), e2 = p2(e), w2 = wb + wb, d = pg - p;
  const T s = 1.0f - 2.0f * sum4(e * e);
  const T eg = sum4(e * gd), ed = sum4(e * d), dg = sum4(d * gd);
  lp = lp - (s * gd + 2.0f * eg * e + p2(w2 * (e2 * gd)) - p1(w2 * (e1 * gd)));
  const T z1 = gd * p1(d), z2 = gd * p2(d);
  T ev, n2, ew;
  att_error(K, q, qg, ev, n2, ew);
  const T dot = sum4(gr * ev);
  const T gev = sk * gr + sign_of(ew) * (dot * kn) * ev;
  const T gew = dot * ka_of(n2, ew);
  const T er = qg * K.m3, wr = bcw(qg);
  const T he = 2.0f * (ed * gd + eg * d - 2.0f * dg * e) - wr * gev + p1(w2 * z1 + gev * p1(er)) - p2(w2 * z2 + gev * p2(er));
  lq = lq + gew * qg + he + K.w3 * sum4(2.0f * (z1 * e2 - z2 * e1) + gev * er);
}

}  // namespace qadj
}  // namespace auv
