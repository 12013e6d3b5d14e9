// Host check of the four-lane SHAC physics (paper_2512_13359_amd/csrc/shac_quad.hpp) in double:
// the lane type holds the four lanes of a quad and permutes them as the device's moves do, and
// every function is compared with the one-lane form (shac_adjoint.hpp, itself checked against
// finite differences) on seeded random inputs: unequal model constants on every axis, non-unit
// stage quaternions, both signs of the attitude error's scalar part, small and large angles.
#include <cmath>
#include <cstdio>
#include <random>

#include "shac_adjoint.hpp"

namespace lanes {
struct H4 {
  double a[4];
};
#define EACH(expr) H4 r; for (int i = 0; i < 4; ++i) r.a[i] = (expr); return r
inline H4 operator+(H4 x, H4 y) { EACH(x.a[i] + y.a[i]); }
inline H4 operator-(H4 x, H4 y) { EACH(x.a[i] - y.a[i]); }
inline H4 operator*(H4 x, H4 y) { EACH(x.a[i] * y.a[i]); }
inline H4 operator*(double s, H4 y) { EACH(s * y.a[i]); }
inline H4 operator-(double s, H4 y) { EACH(s - y.a[i]); }
inline H4 at(H4 x, int p, int q, int r_, int s) { return H4{{x.a[p], x.a[q], x.a[r_], x.a[s]}}; }
inline H4 p1(H4 x) { return at(x, 1, 2, 0, 3); }
inline H4 p2(H4 x) { return at(x, 2, 0, 1, 3); }
inline H4 bcz(H4 x) { return at(x, 2, 2, 2, 2); }
inline H4 bcw(H4 x) { return at(x, 3, 3, 3, 3); }
inline H4 sum4(H4 x) { const double s = x.a[0] + x.a[1] + x.a[2] + x.a[3]; return H4{{s, s, s, s}}; }
inline H4 abs_(H4 x) { EACH(std::fabs(x.a[i])); }
inline H4 rsqrt_(H4 x) { EACH(1.0 / std::sqrt(x.a[i])); }
inline H4 sign_of(H4 x) { EACH(x.a[i] < 0 ? -1.0 : 1.0); }
inline H4 ka_of(H4 n2, H4 ew) { EACH(-2.0 / (n2.a[i] + ew.a[i] * ew.a[i])); }
inline void att_factors(H4 n2, H4 ew, H4& sk, H4& kn) {
  for (int i = 0; i < 4; ++i) {
    const double n = std::sqrt(n2.a[i]), aw = std::fabs(ew.a[i]), at2 = 2 * std::atan2(n, aw), t = n2.a[i] / (aw * aw);
    sk.a[i] = (ew.a[i] < 0 ? -1.0 : 1.0) * (n > 0 ? at2 / n : 2 / aw);
    kn.a[i] = n < 0.1 * aw ? 2 / (aw * aw * aw) * (-2.0 / 3.0 + t * (0.8 + t * (-6.0 / 7.0 + t * (8.0 / 9.0))))
                           : (2 * aw * n / (n2.a[i] + aw * aw) - at2) / (n2.a[i] * n);
  }
}
}  // namespace lanes

#include "shac_quad.hpp"

using namespace auv;
using lanes::H4;
typedef adj::X13<double> X;

static std::mt19937_64 gen(2024);
static double U(double lo, double hi) { return std::uniform_real_distribution<double>(lo, hi)(gen); }
static H4 vec(const double* v) { return H4{{v[0], v[1], v[2], 0.0}}; }
static H4 quat(const double* q) { return H4{{q[1], q[2], q[3], q[0]}}; }
static qadj::QX<H4> pack(const X& x) { return {quat(x.q), vec(x.v), vec(x.w)}; }

static double worst = 0.0, scale = 0.0;
static void diff(H4 a, H4 b) {
  for (int i = 0; i < 4; ++i) {
    const double d = std::fabs(a.a[i] - b.a[i]);
    if (!(d <= worst)) worst = d;   // a NaN stays
    scale = std::fmax(scale, std::fabs(b.a[i]));
  }
}
static bool done(const char* what) {
  const double rel = worst / scale;
  std::printf("%-24s max rel err %.3e\n", what, rel);
  const bool ok = rel <= 1e-12;   // the same sums in another order, in double
  worst = scale = 0.0;
  return ok;
}

static void models(adj::Model<double>& M, qadj::QM<H4>& Q) {
  for (int i = 0; i < 3; ++i) {
    M.A1[i] = U(4, 15);
    M.Mlin[i] = 11.5 + M.A1[i];
    M.Mang[i] = U(0.1, 0.6);
    M.iMlin[i] = 1 / M.Mlin[i];
    M.iMang[i] = 1 / M.Mang[i];
  }
  for (int i = 0; i < 6; ++i) M.DL[i] = U(0.1, 6), M.DQ[i] = U(0.5, 30);
  M.BmW = U(-5, 8);
  const H4 iMl = vec(M.iMlin);
  Q.iMl = iMl;
  Q.DLi = vec(M.DL) * iMl;
  Q.DQi = vec(M.DQ) * iMl;
  Q.BmWi = M.BmW * iMl;
  Q.Ma = vec(M.Mang);
  Q.iMa = vec(M.iMang);
  Q.A1 = vec(M.A1);
  Q.DLa = vec(M.DL + 3);
  Q.DQa = vec(M.DQ + 3);
  Q.Ml = vec(M.Mlin);
  qadj::derive(Q);
}

static X state(double scale_q) {
  X x;
  for (int i = 0; i < 3; ++i) x.p[i] = U(-2, 2), x.v[i] = U(-1.5, 1.5), x.w[i] = U(-1.5, 1.5);
  double n = 0;
  for (int i = 0; i < 4; ++i) x.q[i] = U(-1, 1), n += x.q[i] * x.q[i];
  for (int i = 0; i < 4; ++i) x.q[i] *= scale_q / std::sqrt(n);
  return x;
}

int main() {
  const qadj::LaneK<H4> K{{{1, 1, 1, 0}}, {{0, 0, 0, 1}}, {{1, 0, 0, 0}}, {{0, 1, 0, 0}}, {{0, 0, 1, 0}}};
  bool ok = true;
  for (int part = 0; part < 6; ++part) {
    for (int trial = 0; trial < 200; ++trial) {
      adj::Model<double> M;
      qadj::QM<H4> Q;
      models(M, Q);
      double tau[6], gt[6] = {0, 0, 0, 0, 0, 0};
      for (double& t : tau) t = U(-40, 40);
      const H4 tfi = vec(tau) * Q.iMl, tm = vec(tau + 3);
      const double h = 0.025;
      if (part == 0) {
        const X x = state(U(0.9, 1.1));
        X d;
        adj::rhs(M, tau, x, d);
        H4 dp;
        qadj::QX<H4> q;
        qadj::rhs(K, Q, tfi, tm, pack(x), dp, q);
        diff(dp, vec(d.p)), diff(q.q, quat(d.q)), diff(q.v, vec(d.v)), diff(q.w, vec(d.w));
      } else if (part == 1) {
        const X x = state(U(0.9, 1.1)), g = state(2.0);
        X r;
        adj::zero(r);
        adj::rhs_vjp(M, x, g, r, gt);
        qadj::QX<H4> q;
        H4 gf{}, gm{};
        qadj::rhs_vjp(K, Q, pack(x), vec(g.p), pack(g), q, gf, gm);
        diff(q.q, quat(r.q)), diff(q.v, vec(r.v)), diff(q.w, vec(r.w)), diff(gf, vec(gt)), diff(gm, vec(gt + 3));
      } else if (part == 2 || part == 3) {
        const X x0 = state(1.0);
        X x1 = x0, g = state(2.0);
        adj::substep(M, tau, h, x1);
        H4 p = vec(x0.p), inv, gf{}, gm{};
        qadj::QX<H4> q = pack(x0), st[4], l = pack(g);
        qadj::substep(K, Q, tfi, tm, h, p, q, st, inv);
        if (part == 2) {
          diff(p, vec(x1.p)), diff(q.q, quat(x1.q)), diff(q.v, vec(x1.v)), diff(q.w, vec(x1.w));
        } else {
          qadj::substep_vjp(K, Q, h, st, inv, q.q, vec(g.p), l, gf, gm);
          adj::substep_vjp(M, tau, h, x0, g, gt);
          diff(l.q, quat(g.q)), diff(l.v, vec(g.v)), diff(l.w, vec(g.w)), diff(gf, vec(gt)), diff(gm, vec(gt + 3));
        }
      } else {
        const X x = state(1.0);
        double pg[3] = {U(-2, 2), U(-2, 2), U(-2, 2)}, qg[4], n = 0, ew = 0;
        const bool small = trial % 3 == 1;   // a goal within a few degrees: the series
        for (int i = 0; i < 4; ++i) qg[i] = small ? x.q[i] + U(-0.01, 0.01) : U(-1, 1), n += qg[i] * qg[i];
        for (int i = 0; i < 4; ++i) qg[i] /= std::sqrt(n), ew += qg[i] * x.q[i];
        if ((trial & 1) != (ew < 0))
          for (double& v : qg) v = -v;
        double o[12], go[12];
        for (double& v : go) v = U(-1, 1);
        adj::observe(x, pg, qg, o);
        const qadj::QObsK<H4> b = qadj::observe(K, vec(x.p), quat(x.q), vec(pg), quat(qg));
        if (part == 4) {
          diff(b.dpb, vec(o)), diff(b.rv, vec(o + 3));
        } else {
          for (int k = 6; k < 12; ++k) go[k] = 0.0;   // velocities pass straight through
          X r;
          adj::zero(r);
          adj::observe_vjp(x, pg, qg, go, r);
          H4 lp{}, lq{};
          qadj::observe_vjp(K, vec(x.p), quat(x.q), vec(pg), quat(qg), b.sk, b.kn, vec(go), vec(go + 3), lp, lq);
          diff(lp, vec(r.p)), diff(lq, quat(r.q));
        }
      }
    }
    const char* names[6] = {"rhs", "rhs_vjp", "substep", "substep_vjp", "observe", "observe_vjp"};
    ok &= done(names[part]);
  }
  std::printf("%s\n", ok ? "OK" : "FAIL");
  return ok ? 0 : 1;
}
