// Reverse-mode (adjoint) building blocks of the Wisdom-Holman step, FP64.
//
// Each function takes the adjoint (gradient) of a sub-step's outputs and
// returns the adjoint of its inputs, accumulating the adjoints of the masses.
// Notation of the forward step: K(tau) maps (Q, V) to (f Q + g V, f' Q + g' V);
// I(tau) adds tau a(Q) to V; J(tau) adds (tau/m0) sum_j m_j V_j to Q; the GR
// kick adds -tau 6 m0^2/c^2 Q/|Q|^4 to V.
#pragma once
#include "wh_device.h"

namespace wh {

// Forward quantities of one Kepler drift at a known anomaly X.
struct KepFwd {
  double r0, ir0, eta, beta, zeta, X;
  double G[6];
  double ir, f, g, fd, gd;
};

// G4 and G5 by series, the lower ones by G_n = X^n/n! - beta G_{n+2}.  The
// reciprocals 1/r0 and 1/r are the refined hardware seeds of the forward
// solve: with the IEEE square root and divisions in their place (1/r0, 1/r
// and the quotients by mu, r0 r and r) a sweep step issued a fifth more
// instructions, and the sweep is bound by their issue.
__device__ __forceinline__ void kepler_at_X(double qx, double qy, double qz, double vx, double vy, double vz,
                                            double mu, double tau, double X, KepFwd& k) {
  const double r2 = fma(qx, qx, fma(qy, qy, qz * qz));
  const double v2 = fma(vx, vx, fma(vy, vy, vz * vz));
  k.eta = fma(qx, vx, fma(qy, vy, qz * vz));
  k.ir0 = rsqrt_full(r2);
  k.r0 = r2 * k.ir0;
  const double mi = mu * k.ir0;
  k.beta = fma(2.0, mi, -v2);
  k.zeta = fma(-k.beta, k.r0, mu);
  k.X = X;
  const double X2 = X * X, X3 = X2 * X, z = k.beta * X2;
  k.G[4] = X2 * X2 * stumpff_series<8, 4>(z);
  k.G[5] = X2 * X3 * stumpff_series<8, 5>(z);
  k.G[2] = fma(-k.beta, k.G[4], 0.5 * X2);
  k.G[3] = fma(-k.beta, k.G[5], (1.0 / 6.0) * X3);
  k.G[1] = fma(-k.beta, k.G[3], X);
  k.G[0] = fma(-k.beta, k.G[2], 1.0);
  const double r = fma(k.eta, k.G[1], fma(k.zeta, k.G[2], k.r0));
  k.ir = rcp_full(r);
  k.f = fma(-mi, k.G[2], 1.0);
  k.g = fma(-mu, k.G[3], tau);
  k.fd = -(mi * k.ir) * k.G[1];
  k.gd = fma(-(mu * k.ir), k.G[2], 1.0);
}

// Adjoint of the Kepler drift.  In: (gQ1, gV1), the adjoint of the output.
// Out: (gQ, gV) the adjoint of the input, gmu += the adjoint of mu = G m0.
// The anomaly X is defined implicitly by F(X; r0, eta, zeta, beta) = 0, so by
// the implicit function theorem dX = -(F_r0 dr0 + F_eta deta + F_zeta dzeta +
// F_beta dbeta) / F_X with F_X = r, F_r0 = X, F_eta = G2, F_zeta = G3 and
// F_beta = eta dG2/dbeta + zeta dG3/dbeta, where dG_n/dbeta =
// (n G_{n+2} - X G_{n+1}) / 2 and dG_n/dX = G_{n-1}.
// The scalars of it, from the products of the output's adjoint with the drift's
// start: gf = gQ1.Q, gg = gQ1.V, gfd = gV1.Q, ggd = gV1.V.  Then
//   gQ = f gQ1 + f' gV1 + eta V + q Q,   gV = g gQ1 + g' gV1 + eta Q + v V.
struct KepAdj {
  double eta, q, v, mu;
};
__device__ __forceinline__ KepAdj kepler_adj(const KepFwd& k, double gf, double gg, double gfd, double ggd,
                                             double mu) {
  const double* G = k.G;
  // f = 1 - mu G2/r0, g = tau - mu G3, f' = -mu G1/(r0 r), g' = 1 - mu G2/r
  const double ir0 = k.ir0, ir = k.ir;
  const double a0 = gf * ir0, a1 = ggd * ir, b = gfd * (ir0 * ir);
  double gm = -(a0 * G[2] + gg * G[3] + b * G[1] + a1 * G[2]);
  double gG1 = -mu * b;
  double gG2 = -mu * (a0 + a1);
  double gG3 = -gg * mu;
  const double w = mu * b * G[1];          // -gfd f'
  double gr0 = ir0 * fma(mu * a0, G[2], w);
  double gr = ir * fma(mu * a1, G[2], w);
  // r = r0 + eta G1 + zeta G2
  gr0 += gr;
  double geta = gr * G[1];
  double gzeta = gr * G[2];
  gG1 += gr * k.eta;
  gG2 += gr * k.zeta;
  // G_n(beta, X)
  const double X = k.X;
  double dG1b = 0.5 * (G[3] - X * G[2]);
  double dG2b = 0.5 * (2.0 * G[4] - X * G[3]);
  double dG3b = 0.5 * (3.0 * G[5] - X * G[4]);
  double gX = gG1 * G[0] + gG2 * G[1] + gG3 * G[2];
  double gbeta = gG1 * dG1b + gG2 * dG2b + gG3 * dG3b;
  // implicit function theorem for X
  double Fb = k.eta * dG2b + k.zeta * dG3b;
  double s = -gX * ir;        // -gX / F_X
  gr0 += s * X;
  geta += s * G[2];
  gzeta += s * G[3];
  gbeta += s * Fb;
  // zeta = mu - beta r0
  gm += gzeta;
  gbeta -= gzeta * k.r0;
  gr0 -= gzeta * k.beta;
  // beta = 2 mu / r0 - |V|^2
  const double gb = 2.0 * gbeta * ir0;
  gm += gb;
  gr0 -= gb * mu * ir0;
  return KepAdj{geta, gr0 * ir0, -2.0 * gbeta, gm};
}

__device__ __forceinline__ void kepler_vjp(const KepFwd& k, double qx, double qy, double qz, double vx, double vy,
                                           double vz, double mu, double& gqx, double& gqy, double& gqz,
                                           double& gvx, double& gvy, double& gvz, double& gmu) {
  // outputs Q1 = f Q + g V, V1 = f' Q + g' V
  const double gf = gqx * qx + gqy * qy + gqz * qz;
  const double gg = gqx * vx + gqy * vy + gqz * vz;
  const double gfd = gvx * qx + gvy * qy + gvz * qz;
  const double ggd = gvx * vx + gvy * vy + gvz * vz;
  const KepAdj a = kepler_adj(k, gf, gg, gfd, ggd, mu);
  // and through eta = Q.V, |V|^2 and r0 = |Q|
  const double nqx = k.f * gqx + k.fd * gvx + (a.eta * vx + a.q * qx);
  const double nqy = k.f * gqy + k.fd * gvy + (a.eta * vy + a.q * qy);
  const double nqz = k.f * gqz + k.fd * gvz + (a.eta * vz + a.q * qz);
  const double nvx = k.g * gqx + k.gd * gvx + (a.eta * qx + a.v * vx);
  const double nvy = k.g * gqy + k.gd * gvy + (a.eta * qy + a.v * vy);
  const double nvz = k.g * gqz + k.gd * gvz + (a.eta * qz + a.v * vz);
  gqx = nqx; gqy = nqy; gqz = nqz;
  gvx = nvx; gvy = nvy; gvz = nvz;
  gmu += a.mu;
}

// Adjoint of the interaction kick V += tau a(Q) inside a group, with the DPP
// rounds of interaction_accel_dpp.  With a_i = -sum_j m_j d_ij/|d_ij|^3,
// d_ij = Q_i - Q_j and T_ij = I/r^3 - 3 d d^T/r^5 (symmetric):
//   gQ_k += tau sum_{j != k} T_kj (m_k gV_j - m_j gV_k)
//   gm_k += tau sum_{i != k} gV_i . (Q_k - Q_i) / r^3
// For a pair computed once, the partner's share is the negative of the
// lane's own share, which two-sided rounds send back.
__device__ __forceinline__ void pair_vjp(double qx, double qy, double qz, double gvx, double gvy, double gvz,
                                         double m, double px, double py, double pz, double pgx, double pgy,
                                         double pgz, double mj, double tau, double& cx, double& cy, double& cz,
                                         double& cm_own, double& cm_partner) {
  double dx = qx - px, dy = qy - py, dz = qz - pz;
  double r2 = dx * dx + dy * dy + dz * dz;
  double ir = rsqrt_full(r2);
  double ir2 = ir * ir;
  double ir3 = ir2 * ir;
  double ux = m * pgx - mj * gvx, uy = m * pgy - mj * gvy, uz = m * pgz - mj * gvz;
  double du = dx * ux + dy * uy + dz * uz;
  double w = 3.0 * du * ir2;
  double t = tau * ir3;
  cx = t * (ux - w * dx);
  cy = t * (uy - w * dy);
  cz = t * (uz - w * dz);
  cm_own = t * (pgx * dx + pgy * dy + pgz * dz);
  cm_partner = -t * (gvx * dx + gvy * dy + gvz * dz);
}

template <int G>
__device__ __forceinline__ void interaction_vjp_dpp(const DppMass& t, double qx, double qy, double qz, double m,
                                                    double tau, double gvx, double gvy, double gvz, double& gqx,
                                                    double& gqy, double& gqz, double& gm) {
  double cx, cy, cz, co, cp;
  if (G == 2) {
    pair_vjp(qx, qy, qz, gvx, gvy, gvz, m, dpp<DPP_XOR1>(qx), dpp<DPP_XOR1>(qy), dpp<DPP_XOR1>(qz),
             dpp<DPP_XOR1>(gvx), dpp<DPP_XOR1>(gvy), dpp<DPP_XOR1>(gvz), t.m[0], tau, cx, cy, cz, co, cp);
    gqx += cx; gqy += cy; gqz += cz; gm += co;
  }
  if (G >= 4) {
    pair_vjp(qx, qy, qz, gvx, gvy, gvz, m, dpp<QP_NEXT>(qx), dpp<QP_NEXT>(qy), dpp<QP_NEXT>(qz),
             dpp<QP_NEXT>(gvx), dpp<QP_NEXT>(gvy), dpp<QP_NEXT>(gvz), t.m[0], tau, cx, cy, cz, co, cp);
    gqx += cx - dpp<QP_PREV>(cx);
    gqy += cy - dpp<QP_PREV>(cy);
    gqz += cz - dpp<QP_PREV>(cz);
    gm += co + dpp<QP_PREV>(cp);
    pair_vjp(qx, qy, qz, gvx, gvy, gvz, m, dpp<DPP_XOR2>(qx), dpp<DPP_XOR2>(qy), dpp<DPP_XOR2>(qz),
             dpp<DPP_XOR2>(gvx), dpp<DPP_XOR2>(gvy), dpp<DPP_XOR2>(gvz), t.m[1], tau, cx, cy, cz, co, cp);
    gqx += cx; gqy += cy; gqz += cz; gm += co;
  }
  if (G == 8) {
    double mx = dpp<DPP_HALF_MIRROR>(qx), my = dpp<DPP_HALF_MIRROR>(qy), mz = dpp<DPP_HALF_MIRROR>(qz);
    double hx = dpp<DPP_HALF_MIRROR>(gvx), hy = dpp<DPP_HALF_MIRROR>(gvy), hz = dpp<DPP_HALF_MIRROR>(gvz);
    pair_vjp(qx, qy, qz, gvx, gvy, gvz, m, dpp<QP_R3>(mx), dpp<QP_R3>(my), dpp<QP_R3>(mz), dpp<QP_R3>(hx),
             dpp<QP_R3>(hy), dpp<QP_R3>(hz), t.m[2], tau, cx, cy, cz, co, cp);
    gqx += cx - dpp<QP_R3_BACK>(dpp<DPP_HALF_MIRROR>(cx));
    gqy += cy - dpp<QP_R3_BACK>(dpp<DPP_HALF_MIRROR>(cy));
    gqz += cz - dpp<QP_R3_BACK>(dpp<DPP_HALF_MIRROR>(cz));
    gm += co + dpp<QP_R3_BACK>(dpp<DPP_HALF_MIRROR>(cp));
    pair_vjp(qx, qy, qz, gvx, gvy, gvz, m, dpp<QP_R4>(mx), dpp<QP_R4>(my), dpp<QP_R4>(mz), dpp<QP_R4>(hx),
             dpp<QP_R4>(hy), dpp<QP_R4>(hz), t.m[3], tau, cx, cy, cz, co, cp);
    gqx += cx; gqy += cy; gqz += cz; gm += co;
    pair_vjp(qx, qy, qz, gvx, gvy, gvz, m, dpp<QP_R5>(mx), dpp<QP_R5>(my), dpp<QP_R5>(mz), dpp<QP_R5>(hx),
             dpp<QP_R5>(hy), dpp<QP_R5>(hz), t.m[4], tau, cx, cy, cz, co, cp);
    gqx += cx; gqy += cy; gqz += cz; gm += co;
  }
}

// Adjoint of the GR kick V += tau * (-kg Q/|Q|^4), kg = 6 mu^2 / c^2:
//   gQ += -tau kg (gV/|Q|^4 - 4 Q (Q.gV)/|Q|^6),  gmu += tau gV.a_GR * 2/mu,
// inv_mu = 1/mu.
__device__ __forceinline__ void gr_vjp(double qx, double qy, double qz, double kg, double inv_mu, double tau,
                                       double gvx, double gvy, double gvz, double& gqx, double& gqy, double& gqz,
                                       double& gmu) {
  double r2 = qx * qx + qy * qy + qz * qz;
  double ir2 = rcp_full(r2);
  double ir4 = ir2 * ir2;
  double qg = qx * gvx + qy * gvy + qz * gvz;
  double s = -tau * kg * ir4;
  double w = -4.0 * qg * ir2;
  gqx += s * (gvx + w * qx);
  gqy += s * (gvy + w * qy);
  gqz += s * (gvz + w * qz);
  gmu += 2.0 * s * qg * inv_mu;
}

}  // namespace wh
