// Reverse mode with four lanes per planet (wh_wide.h): recording a segment and
// sweeping it, for the ensembles whose step runs in that form.
//
// A segment's tape is then [step][wavefront][TAPE_ROWS][16 planets], 1280
// contiguous bytes per wavefront and step, whatever the packing.
//
// The sweep is that of adj_sweep_lane (wh.hip), a component per lane: lane
// c < 3 carries component c of dL/dQ and dL/dV, lane 3 the planet's mass
// (zeros in the place of its component, so that sums over the four lanes are
// sums over three).  The Kepler adjoint's scalars repeat on the four lanes.
// Each pair is evaluated once, on the lane of planet p and distance k = c + 1
// around the group (distance G/2 on the lower half's planets), which leaves
// the shares of both planets in LDS for their lanes to add up: 4 KiB of LDS per
// wavefront.
#pragma once
#include "wh_adjoint.h"
#include "wh_wide.h"

namespace wh {

constexpr int WIDE_ADJ_LDS = 512;    // doubles of LDS per wavefront
constexpr int WIDE_TAPE = wh_host::WH_TAPE_ROWS * WIDE_SLOTS;   // doubles per wavefront and step

// Launch parameters of the reverse pass.
struct AdjParams {
  StepParams sp;
  const double* ck;    // k_adj_init: the final checkpoint
  double* tape;        // tape of the segment being swept
  double* grad;        // adjoint state
  const double* gQ_T;  // caller layout [S*8*3]
  const double* gV_T;
  double* gQ_0;
  double* gV_0;
  double* gm;          // [S*8]
  double* gm0;         // [S]
  int n_seg;           // steps of the segment being swept
  int first_synced;    // it starts from the synchronized initial state
  int sweep_waves;     // wavefronts of the sweeping role (0: the launch only records)
  int wide_waves;      // wavefronts of each role with four lanes per planet (0: a lane per planet)
  const double* ck_rec;  // recording role: checkpoint of the segment to record,
  double* tape_rec;      // the tape to fill,
  int n_rec;             // its steps,
  int rec_first_synced;  // and whether it starts from the synchronized initial state
};

// Recording (adj_record_lane): the checkpoint's state through n_rec steps.
// Lanes 0..2 of a planet write the rows of their component, lane 3 the
// anomaly.  FIN: the run's last segment, stored as the context's state at its
// end.
template <int G, bool GR, int SCHEME, int STORAGE, bool FIN>
__device__ __forceinline__ void wide_record(const StepParams& p, const double* ck, double* tape, int n_waves,
                                            int n_rec, bool first_synced, int w, double* block, int lane) {
  const int slot = wide_slot<STORAGE>(w, lane), c = wide_comp(lane), ns = p.ns;
  const size_t r3 = (size_t)3 * ns;
  const double* cs = ck + (size_t)c * ns + slot;
  WideLane L{};
  L.q = cs[0];
  L.v = cs[r3];
  L.cq = cs[2 * r3];
  L.cv = cs[3 * r3];
  L.m = p.st[(size_t)6 * ns + slot];
  L.m0 = p.m0s[slot];
  const double dt = p.dts[slot], h = 0.5 * dt;
  const double inv_m0 = 1.0 / L.m0;
  const double kg = GR ? p.kgr * L.m0 * L.m0 : 0.0;
  const bool comp = (lane & 3) < 3;
  WideKick<G, STORAGE> wk;
  wk.init(block, lane, L.m);
  KepDiag dg{0.0, 1.0e300};
  wait_loads();
  double vk;
  double* row = tape + (size_t)w * WIDE_TAPE + (lane >> 2);
  const size_t step = (size_t)n_waves * WIDE_TAPE;
  auto put_state = [&]() {
    if (comp) {
      row[c * WIDE_SLOTS] = L.q;
      row[(3 + c) * WIDE_SLOTS] = L.v;
    }
  };
  auto put_rest = [&](double X) {
    row[(comp ? 7 + c : 6) * WIDE_SLOTS] = comp ? vk : X;
    row += step;
  };
  if constexpr (SCHEME == SCHEME_SABA) {
    const int nu = p.saba_n;
    const double c1dt = p.sc[0] * dt;
    for (int s = 0; s < n_rec; ++s)
      for (int k = 0; k < nu; ++k) {
        const double tau = k > 0 ? p.sc[k] * dt : (first_synced && s == 0 ? c1dt : 2.0 * c1dt);
        const double tb = p.sd[k] * dt;
        put_state();
        const double X = wide_drift<0>(L, L.m0, tau, dg);
        wide_kick<G, false>(L, wk, inv_m0, 0.0, 0.5 * tb, tb, 0.5 * tb, vk);
        put_rest(X);
      }
  } else if constexpr (SCHEME == WH_KDK) {
    double ta = first_synced ? 0.0 : h;
    double ti = first_synced ? h : dt;
    for (int s = 0; s < n_rec; ++s) {
      put_state();
      wide_kick<G, GR>(L, wk, inv_m0, kg, ta, ti, h, vk);
      ta = h;
      ti = dt;
      put_rest(wide_drift<0>(L, L.m0, dt, dg));
    }
  } else {
    double tk = first_synced ? h : dt;
    for (int s = 0; s < n_rec; ++s) {
      put_state();
      const double X = wide_drift<0>(L, L.m0, tk, dg);
      tk = dt;
      wide_kick<G, GR>(L, wk, inv_m0, kg, h, dt, h, vk);
      put_rest(X);
    }
  }
  if (FIN) {
    L.sys = p.slot_sys[slot];
    L.pl = p.slot_pl[slot];
    wide_flags<G>(p, L, dg, lane);
    wide_store<STORAGE>(p, L, slot, c, lane);
  }
}

// ---------------------------------------------------------------------------
// Sum over a planet's four lanes, in all of them.
__device__ __forceinline__ double quad_sum(double v) {
  v += dpp<DPP_XOR1>(v);
  return v + dpp<DPP_XOR2>(v);
}
// Sum over the planets of a group, of the lane's component.
template <int G> __device__ __forceinline__ double wide_sum(double v) {
  if (G >= 2) v += wide_xor1(v);
  if (G >= 4) v += dpp<DPP_ROR8>(v);
  if (G >= 8) {
    int l0, l1, h0, h1;
    row_pair(__double2loint(v), l0, l1);
    row_pair(__double2hiint(v), h0, h1);
    v = __hiloint2double(h0, l0) + __hiloint2double(h1, l1);
  }
  return v;
}

// The lane's share of the adjoint state: component of dL/dQ and dL/dV (zero on
// lane 3), the mass's (on lane 3) and the planet's share of the star mass's.
struct WideGrad {
  double q, v, m, m0;
};

// Places in the wavefront's LDS block: positions [planet][4], dL/dV at 64 +
// [planet][4], the pairs' shares at 128 + [planet][c][6] (of the evaluating
// planet: position x, y, z and mass; of its partner: the mass, the position's
// negated).
template <int G> struct WidePairs {
  double* lds;
  double m, mj, sign;
  int iq, in, ip, iw, io[4], ij[4];
  bool on, third;

  __device__ __forceinline__ void init(double* block, int lane, double mass) {
    lds = block;
    m = mass;
    const int c = lane & 3, pl = lane >> 2, base = pl & ~(G - 1), p = pl & (G - 1);
    third = c == 3;
    in = pl * 4;
    iq = in + c;
    mj = 0.0;
    on = false;
    ip = in;
    iw = 128 + (pl * 4 + c) * 6;
    sign = third ? 1.0 : -1.0;
    if (G == 1) return;
    const int k = c + 1;
    on = 2 * k < G || (2 * k == G && p < G / 2);
    ip = (base + ((p + k) & (G - 1))) * 4;
#pragma unroll
    for (int d = 0; d < G / 2; ++d) {
      io[d] = 128 + (pl * 4 + d) * 6 + c;
      ij[d] = 128 + ((base + ((p - d - 1) & (G - 1))) * 4 + d) * 6 + (third ? 4 : c);
    }
    lds[iq] = m;
    wave_lds_fence();
    mj = lds[ip];
    wave_lds_fence();
  }

  // Adjoint of the interaction kick V += tau a(Q) at positions whose component
  // on this lane is q (zero on lane 3): adds dL/dQ to g.q and dL/dm to g.m.
  // (x..), (gx..): receive the planet's position and dL/dV.
  __device__ __forceinline__ void vjp(WideGrad& g, double q, double tau, double& x, double& y, double& z, double& gx,
                                      double& gy, double& gz) const {
    lds[iq] = q;
    lds[iq + 64] = g.v;
    wave_lds_fence();
    x = lds[in]; y = lds[in + 1]; z = lds[in + 2];
    gx = lds[in + 64]; gy = lds[in + 65]; gz = lds[in + 66];
    if (G == 1) {
      wave_lds_fence();
      return;
    }
    double cx, cy, cz, co, cp;
    pair_vjp(x, y, z, gx, gy, gz, m, lds[ip], lds[ip + 1], lds[ip + 2], lds[ip + 64], lds[ip + 65], lds[ip + 66], mj,
             tau, cx, cy, cz, co, cp);
    lds[iw] = on ? cx : 0.0;
    lds[iw + 1] = on ? cy : 0.0;
    lds[iw + 2] = on ? cz : 0.0;
    lds[iw + 3] = on ? co : 0.0;
    lds[iw + 4] = on ? cp : 0.0;
    wave_lds_fence();
    double own = lds[io[0]], other = lds[ij[0]];
#pragma unroll
    for (int d = 1; d < G / 2; ++d) {
      own += lds[io[d]];
      other += lds[ij[d]];
    }
    const double s = fma(sign, other, own);
    g.q += third ? 0.0 : s;
    g.m += third ? s : 0.0;
  }
};

// Adjoint of the jump Q += kj sum_j m_j V_j (jump_vjp), v: the component of V.
template <int G>
__device__ __forceinline__ void wide_jump_vjp(WideGrad& g, double m, double v, double kj, double inv_m0) {
  const double S = wide_sum<G>(g.q);
  g.v = fma(kj * m, S, g.v);
  const double t = kj * quad_sum(v * S);
  g.m += t;
  g.m0 -= inv_m0 * m * t;
}

// Adjoint of the kick block (kick_block_vjp) at the component q, v of the
// state before it, vk the velocity after the kick.
template <int G, bool GR>
__device__ __forceinline__ void wide_kick_vjp(WideGrad& g, const WidePairs<G>& wp, double inv_m0, double kg, double q,
                                              double v, double vk, double ta, double ti, double tc) {
  double x, y, z, gx, gy, gz;
  if (GR) {
    const double k1 = ta * inv_m0;
    const double q2 = fma(k1, wide_sum<G>(wp.m * v), q);
    wide_jump_vjp<G>(g, wp.m, vk, tc * inv_m0, inv_m0);
    wp.vjp(g, q2, ti, x, y, z, gx, gy, gz);
    // gr_vjp
    const double ir2 = rcp_full(fma(x, x, fma(y, y, z * z)));
    const double qg = fma(x, gx, fma(y, gy, z * gz));
    const double s = -ti * kg * ir2 * ir2;
    g.q = fma(s, fma(-4.0 * qg * ir2, q2, g.v), g.q);
    g.m0 += 2.0 * s * qg * inv_m0;
    wide_jump_vjp<G>(g, wp.m, v, k1, inv_m0);
  } else {
    wide_jump_vjp<G>(g, wp.m, vk, (ta + tc) * inv_m0, inv_m0);
    wp.vjp(g, q, ti, x, y, z, gx, gy, gz);
  }
}

// Adjoint of the Kepler drift (kepler_vjp) from the component q, v of its
// start.
__device__ __forceinline__ void wide_kepler_vjp(WideGrad& g, const KepFwd& k, double q, double v, double m0) {
  double qx = dpp<DPP_QUAD_0>(q), qy = dpp<DPP_QUAD_1>(q), qz = dpp<DPP_QUAD_2>(q);
  double vx = dpp<DPP_QUAD_0>(v), vy = dpp<DPP_QUAD_1>(v), vz = dpp<DPP_QUAD_2>(v);
  double gqx = dpp<DPP_QUAD_0>(g.q), gqy = dpp<DPP_QUAD_1>(g.q), gqz = dpp<DPP_QUAD_2>(g.q);
  double gvx = dpp<DPP_QUAD_0>(g.v), gvy = dpp<DPP_QUAD_1>(g.v), gvz = dpp<DPP_QUAD_2>(g.v);
  const KepAdj a = kepler_adj(k, fma(gqx, qx, fma(gqy, qy, gqz * qz)), fma(gqx, vx, fma(gqy, vy, gqz * vz)),
                              fma(gvx, qx, fma(gvy, qy, gvz * qz)), fma(gvx, vx, fma(gvy, vy, gvz * vz)), m0);
  const double nq = k.f * g.q + k.fd * g.v + a.eta * v + a.q * q;
  g.v = k.g * g.q + k.gd * g.v + a.eta * q + a.v * v;
  g.q = nq;
  g.m0 += a.mu;
}

__device__ __forceinline__ void wide_kepler_at_X(double q, double v, double m0, double tau, double X, KepFwd& k) {
  kepler_at_X(dpp<DPP_QUAD_0>(q), dpp<DPP_QUAD_1>(q), dpp<DPP_QUAD_2>(q), dpp<DPP_QUAD_0>(v), dpp<DPP_QUAD_1>(v),
              dpp<DPP_QUAD_2>(v), m0, tau, X, k);
}

// Reverse sweep of a recorded segment (adj_sweep_lane).  The next step's
// values are loaded while a step is swept.
template <int G, bool GR, int SCHEME, int STORAGE>
__device__ __forceinline__ void wide_sweep(const StepParams& p, double* grad, const double* tape, int n_waves,
                                           int n_seg, bool first_synced, int w, double* block, int lane) {
  const int slot = wide_slot<STORAGE>(w, lane), ns = p.ns, c = lane & 3;
  const bool comp = c < 3;
  const double m = p.st[(size_t)6 * ns + slot], m0 = p.m0s[slot], dt = p.dts[slot], h = 0.5 * dt;
  const double inv_m0 = 1.0 / m0;
  const double kg = GR ? p.kgr * m0 * m0 : 0.0;
  double* gs = grad + slot;
  WideGrad g;
  g.q = comp ? gs[(size_t)c * ns] : 0.0;
  g.v = comp ? gs[(size_t)(3 + c) * ns] : 0.0;
  g.m = gs[(size_t)6 * ns];
  g.m0 = gs[(size_t)7 * ns];
  WidePairs<G> wp;
  wp.init(block, lane, m);
  const int nu = SCHEME == SCHEME_SABA ? p.saba_n : 1;
  const int units = n_seg * nu;
  const size_t step = (size_t)n_waves * WIDE_TAPE;
  const double* row = tape + (size_t)w * WIDE_TAPE + (lane >> 2) + (size_t)(units > 0 ? units - 1 : 0) * step;
  double nq = 0.0, nv = 0.0, nk = 0.0, nX = 0.0;
  auto load = [&]() {
    nq = comp ? row[c * WIDE_SLOTS] : 0.0;
    nv = comp ? row[(3 + c) * WIDE_SLOTS] : 0.0;
    nk = comp ? row[(7 + c) * WIDE_SLOTS] : 0.0;
    nX = row[6 * WIDE_SLOTS];
  };
  if (units > 0) load();
  for (int u = units - 1; u >= 0; --u) {
    const double q0 = nq, v0 = nv, vk = nk, X = nX;
    row -= step;
    if (u > 0) load();
    KepFwd k;
    if constexpr (SCHEME == WH_KDK) {
      const bool first = first_synced && u == 0;
      const double ta = first ? 0.0 : h, ti = first ? h : dt;
      const double s2 = wide_sum<G>(m * vk);
      const double q3 = GR ? fma(h * inv_m0, s2, fma(ta * inv_m0, wide_sum<G>(m * v0), q0))
                           : fma((ta + h) * inv_m0, s2, q0);
      wide_kepler_at_X(q3, vk, m0, dt, X, k);
      wide_kepler_vjp(g, k, q3, vk, m0);
      wide_kick_vjp<G, GR>(g, wp, inv_m0, kg, q0, v0, vk, ta, ti, h);
    } else {
      double tau, ta, ti;
      if constexpr (SCHEME == SCHEME_SABA) {
        const int s = u / nu, kk = u - s * nu;
        tau = kk > 0 ? p.sc[kk] * dt : (first_synced && s == 0 ? p.sc[0] * dt : 2.0 * (p.sc[0] * dt));
        ti = p.sd[kk] * dt;
        ta = 0.5 * ti;
      } else {
        tau = first_synced && u == 0 ? h : dt;
        ta = h;
        ti = dt;
      }
      wide_kepler_at_X(q0, v0, m0, tau, X, k);
      wide_kick_vjp<G, GR>(g, wp, inv_m0, kg, k.f * q0 + k.g * v0, k.fd * q0 + k.gd * v0, vk, ta, ti, ta);
      wide_kepler_vjp(g, k, q0, v0, m0);
    }
  }
  if (comp) {
    wide_put<STORAGE>(gs + (size_t)c * ns, g.q);
    wide_put<STORAGE>(gs + (size_t)(3 + c) * ns, g.v);
  } else {
    wide_put<STORAGE>(gs + (size_t)6 * ns, g.m);
    wide_put<STORAGE>(gs + (size_t)7 * ns, g.m0);
  }
}

// The kernel of reverse mode in this form (k_adj_segment's counterpart), defined
// and instantiated in wh_wide_adjoint.hip: wavefronts [0, sweep_waves) sweep one
// segment, the following ones record the previous one (the same bits as the
// step, which recording repeats).
template <bool GR, bool SPLIT, int SCH, bool FIN> __global__ __launch_bounds__(64) void k_adj_wide(AdjParams q);

}  // namespace wh
