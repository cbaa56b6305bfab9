// Four lanes per planet: how small ensembles run the one-planet step and the
// split layout's.  VALU instructions per lane-step on eight-planet groups,
// without and with GR: 271 and 303, and 15 LDS instructions (one lane per
// planet: 474 and 522); in the split layout's order 273 and 301 (399 and 447).
// In Jacobi coordinates, on groups of 8, 4 and 2 planets: 418, 325 and 302
// (671, 529 and 447).
//
// An ensemble with few wavefronts leaves most SIMDs idle, and a step's time is
// then the instructions one wavefront issues.  Here a wavefront runs 16 planet
// slots instead of 64.  The four lanes of a planet repeat its Kepler solve (a
// serial chain) and divide the rest: lane c < 3 carries component c of the
// compensated state (lane 3 repeats lane 0), so the drift's map, the kicks'
// increments, the momentum sum and the renormalization run once per lane
// instead of three times, and every pair of a system is evaluated on a lane of
// its own.  Each operation and each order of summation is that of the
// packing's own step (drift, kick_block, group_momentum, interaction_accel_dpp
// or accel_split, with the products that the compiler fuses there fused here),
// so the results are the same bits and the forms mix freely: reverse mode's
// recording, the per-size path, batches of either size.
//
// Exchange goes through LDS, 2 KiB per wavefront.  A wavefront's own LDS
// operations stay in order, so writing and reading need no wait between them,
// only that the compiler keeps them apart (wave_lds_fence).  Per kick:
//   1. every lane writes its component of the position and reads its own
//      planet's and one partner's position whole, and its component of each
//      partner's position;
//   2. it evaluates 1/r^3 of its pair, writes it, and reads those of its
//      planet's pairs;
//   3. it adds the pairs' accelerations of its component, in the layout's order.
#pragma once
#include "wh_step.h"

namespace wh {

constexpr int WIDE_SLOTS = 16;   // planet slots per wavefront
constexpr int WIDE_LDS = 256;    // doubles of LDS per wavefront

constexpr int DPP_QUAD_0 = 0x00, DPP_QUAD_1 = 0x55, DPP_QUAD_2 = 0xAA;   // quad_perm: all lanes read lane 0, 1, 2
constexpr int DPP_QUAD_REV = 0x1B;                                       // quad_perm [3,2,1,0]
constexpr int DPP_ROW_MIRROR = 0x140;                                    // lane l of a row reads lane 15 - l

__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Values of the even and odd row of the lane's row pair, in every lane.
__device__ __forceinline__ void row_pair(int v, int& even, int& odd) {
  const auto s = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
  even = (int)s[0];
  odd = (int)s[1];
}

// Planet p ^ 1's lane of the same component (half-row mirror, then each quad
// reversed), and planet 3 - r's of the row (row mirror, then reversed).
__device__ __forceinline__ double wide_xor1(double v) { return dpp<DPP_QUAD_REV>(dpp<DPP_HALF_MIRROR>(v)); }
__device__ __forceinline__ double wide_flip(double v) { return dpp<DPP_QUAD_REV>(dpp<DPP_ROW_MIRROR>(v)); }

// group_momentum of the lane's component: sum over the group's planets of
// m v.  The butterfly's first stage adds the neighbour's rounded product to
// the lane's own by an FMA, so the sums of two neighbours may differ in the
// last bit, and every later stage has to read the planet it reads there: in
// the one-planet groups p ^ 2, then 7 - p; in the split layout 3 - p of the
// half-row, then p ^ 4.
template <int G, int STORAGE> __device__ __forceinline__ double wide_momentum(double m, double v) {
#pragma clang fp contract(off)
  if (G == 1) return m * v;
  double t = fma(m, v, wide_xor1(m * v));
  if (G == 2) return t;
  if (STORAGE == 1) t += wide_flip(t);
  else t += dpp<DPP_ROR8>(t);
  if (G == 4) return t;
  int l0, l1, h0, h1;
  if (STORAGE == 1) {
    row_pair(__double2loint(t), l0, l1);
    row_pair(__double2hiint(t), h0, h1);
    return __hiloint2double(h0, l0) + __hiloint2double(h1, l1);
  }
  const double u = wide_flip(t);
  row_pair(__double2loint(u), l0, l1);
  row_pair(__double2hiint(u), h0, h1);
  const bool odd = threadIdx.x & 16;
  return t + __hiloint2double(odd ? h0 : h1, odd ? l0 : l1);
}
template <int G> __device__ __forceinline__ int wide_or(int f) {
  if (G >= 2) f |= dpp_i<DPP_QUAD_REV>(dpp_i<DPP_HALF_MIRROR>(f));
  if (G >= 4) f |= dpp_i<DPP_ROR8>(f);
  if (G >= 8) {
    int a, b;
    row_pair(f, a, b);
    f = a | b;
  }
  return f;
}

// The kick of the one-planet groups.  Row h of 16 lanes holds four planets;
// an eight-planet group takes two rows.  Lane c of planet (h, r) evaluates the
// pair with
//   c = 0: (h, r + 1)   R1            c = 1: (h, r + 2)   R2
//   c = 2: (h', r + 1)  R3            c = 3: (h', r) R4 if h = 0, (h', r + 2) R5 if h = 1
// (r modulo 4, h' the other row; R1..R5 the rounds of interaction_accel_dpp,
// in whose order step 3 adds).  Positions ([row][8][4]) and 1/r^3 (128 +
// [row][c][8]) are stored twice along r, so that "r + k modulo 4" is a
// constant offset.
template <int G, int STORAGE> struct WideKick {
  double* lds;
  int iq, io, in, ip;            // own and other row's component, own planet, pair partner
  int iw, ie, ier3, ie4, ie5;    // 1/r^3: the lane's own, its planet's
  double m1, m1r, m2, m3, m3r, m4, m5;

  __device__ __forceinline__ void init(double* block, int lane, double m) {
    lds = block;
    const int c = lane & 3, comp = c == 3 ? 0 : c, r = (lane >> 2) & 3, row = lane >> 4, odd = row & 1;
    iq = row * 32 + r * 4 + comp;
    in = row * 32 + r * 4;
    io = (row ^ 1) * 32 + r * 4 + comp;
    if (G == 8)
      ip = c == 0 ? in + 4 : c == 1 ? in + 8 : (row ^ 1) * 32 + (r + (c == 2 ? 1 : 2 * odd)) * 4;
    else if (G == 4)
      ip = c == 1 ? in + 8 : in + 4;
    else
      ip = row * 32 + (r ^ 1) * 4;
    iw = 128 + row * 32 + c * 8 + r;
    ie = 128 + row * 32 + r;
    ier3 = 128 + (row ^ 1) * 32 + 16 + r + 3;
    ie4 = 128 + (row & ~1) * 32 + 24 + r;
    ie5 = 128 + (row | 1) * 32 + 24 + (odd ? r : r + 2);
    m1 = m1r = m2 = m3 = m3r = m4 = m5 = 0.0;
    if (G == 1) return;
    lds[iq] = m;
    lds[iq + 16] = m;
    wave_lds_fence();
    if (G == 2) {
      m1 = lds[ip];
    } else {
      m1 = lds[iq + 4]; m2 = lds[iq + 8]; m1r = lds[iq + 12];
      if (G == 8) { m4 = lds[io]; m3 = lds[io + 4]; m5 = lds[io + 8]; m3r = lds[io + 12]; }
    }
    wave_lds_fence();
  }

  // Acceleration of the lane's component; q: the component of the position,
  // (x, y, z): receives the planet's position.
  __device__ __forceinline__ double accel(double q, double& x, double& y, double& z) const {
#pragma clang fp contract(off)
    lds[iq] = q;
    if (G >= 4) lds[iq + 16] = q;
    wave_lds_fence();
    x = lds[in]; y = lds[in + 1]; z = lds[in + 2];
    if (G == 1) return 0.0;
    const double px = lds[ip], py = lds[ip + 1], pz = lds[ip + 2];
    if (G == 2) {
      const double q1 = lds[ip + (iq - in)];
      const double dx = x - px, dy = y - py, dz = z - pz;
      const double w = m1 * rsqrt3_full(fma(dx, dx, fma(dy, dy, dz * dz)));
      return fma(-w, q - q1, 0.0);
    }
    const double q1 = lds[iq + 4], q2 = lds[iq + 8], q1r = lds[iq + 12];
    double q4 = 0.0, q3 = 0.0, q5 = 0.0, q3r = 0.0;
    if (G == 8) { q4 = lds[io]; q3 = lds[io + 4]; q5 = lds[io + 8]; q3r = lds[io + 12]; }
    const double dx = x - px, dy = y - py, dz = z - pz;
    const double ir3 = rsqrt3_full(fma(dx, dx, fma(dy, dy, dz * dz)));
    lds[iw] = ir3;
    lds[iw + 4] = ir3;
    wave_lds_fence();
    const double e1 = lds[ie], e1r = lds[ie + 3], e2 = lds[ie + 8];
    double a = fma(-(m1 * e1), q - q1, 0.0);
    a += (m1r * e1r) * (q1r - q);
    a = fma(-(m2 * e2), q - q2, a);
    if (G == 8) {
      const double e3 = lds[ie + 16], e3r = lds[ier3], e4 = lds[ie4], e5 = lds[ie5];
      a = fma(-(m3 * e3), q - q3, a);
      a += (m3r * e3r) * (q3r - q);
      a = fma(-(m4 * e4), q - q4, a);
      a = fma(-(m5 * e5), q - q5, a);
    }
    return a;
  }
};

// The split layout's kick: planet p of the ring of eight, lane c evaluates the
// pair with p + c + 1.  Step 3 adds the pairs of the layout's copy 0, those of
// copy 1, then the two (accel_split); pairs at distance 4 count once, with
// zero masses on the side that repeats them.  Positions ([system][16][4]) and
// 1/r^3 (128 + [system][c][16]) are stored twice along the ring.
template <> struct WideKick<8, 1> {
  double* lds;
  int iq, in, ip, iw, ie;
  double m1, m2, m3, m4, m1r, m2r, m3r, m4r;   // partners p + k, and p - k whose reaction comes back

  __device__ __forceinline__ void init(double* block, int lane, double m) {
    lds = block;
    const int c = lane & 3, comp = c == 3 ? 0 : c, p = (lane >> 2) & 7, sys = lane >> 5;
    in = sys * 64 + p * 4;
    iq = in + comp;
    ip = in + (c + 1) * 4;
    ie = 128 + sys * 64 + p;
    iw = ie + c * 16;
    lds[iq] = m;
    lds[iq + 32] = m;
    wave_lds_fence();
    m1 = lds[iq + 4]; m2 = lds[iq + 8]; m3 = lds[iq + 12];
    m1r = lds[iq + 28]; m2r = lds[iq + 24]; m3r = lds[iq + 20];
    const double mo = lds[iq + 16];
    m4 = p >= 4 ? 0.0 : mo;
    m4r = p >= 4 ? mo : 0.0;
    wave_lds_fence();
  }

  __device__ __forceinline__ double accel(double q, double& x, double& y, double& z) const {
#pragma clang fp contract(off)
    lds[iq] = q;
    lds[iq + 32] = q;
    wave_lds_fence();
    x = lds[in]; y = lds[in + 1]; z = lds[in + 2];
    const double px = lds[ip], py = lds[ip + 1], pz = lds[ip + 2];
    const double q1 = lds[iq + 4], q2 = lds[iq + 8], q3 = lds[iq + 12], q4 = lds[iq + 16];
    const double q3r = lds[iq + 20], q2r = lds[iq + 24], q1r = lds[iq + 28];
    const double dx = x - px, dy = y - py, dz = z - pz;
    const double ir3 = rsqrt3_full(fma(dx, dx, fma(dy, dy, dz * dz)));
    lds[iw] = ir3;
    lds[iw + 8] = ir3;
    wave_lds_fence();
    const double e1 = lds[ie], e1r = lds[ie + 7], e2 = lds[ie + 16], e2r = lds[ie + 22];
    const double e3 = lds[ie + 32], e3r = lds[ie + 37], e4 = lds[ie + 48], e4r = lds[ie + 52];
    double a0 = fma(-(m1 * e1), q - q1, 0.0);
    a0 += (m2r * e2r) * (q2r - q);
    a0 = fma(-(m3 * e3), q - q3, a0);
    a0 += (m4r * e4r) * (q4 - q);
    double a1 = fma(-(m2 * e2), q - q2, 0.0);
    a1 += (m1r * e1r) * (q1r - q);
    a1 = fma(-(m4 * e4), q - q4, a1);
    a1 += (m3r * e3r) * (q3r - q);
    return a0 + a1;
  }
};

// The lane's component of its planet's compensated state, and the planet's
// constants.
struct WideLane {
  double q, v, cq, cv, m, m0, dt;
  int sys, pl, first;
};

__device__ __forceinline__ int wide_comp(int lane) { return (lane & 3) == 3 ? 0 : lane & 3; }

// Kepler drift (drift of wh_step.h) about mass mu: the whole planet's
// coefficients, the lane's component of the map.  Returns the anomaly.
template <int KC>
__device__ __forceinline__ double wide_drift(WideLane& L, double mu, double tau, KepDiag& dg) {
  KepCoef k;
  const double X = kepler_coeffs<KepSet<KC>::NH, KepSet<KC>::NN, KepSet<KC>::KH, KepSet<KC>::KN>(
      dpp<DPP_QUAD_0>(L.q), dpp<DPP_QUAD_1>(L.q), dpp<DPP_QUAD_2>(L.q), dpp<DPP_QUAD_0>(L.v), dpp<DPP_QUAD_1>(L.v),
      dpp<DPP_QUAD_2>(L.v), mu, tau, dg, k);
  double hq, lq, hv, lv;
  lin2_dd(k.fm1, L.q, k.g, L.v, hq, lq);
  lin2_dd(k.gdm1, L.v, k.fd, L.q, hv, lv);
  lq = fma(k.fm1, L.cq, fma(k.g, L.cv, lq));
  lv = fma(k.fd, L.cq, fma(k.gdm1, L.cv, lv));
  add_hi(L.q, L.cq, hq, lq);
  add_hi(L.v, L.cv, hv, lv);
  return X;
}

// kick_block on the lane's component; vk: its velocity after the kick.
template <int G, bool GR, int STORAGE>
__device__ __forceinline__ void wide_kick(WideLane& L, const WideKick<G, STORAGE>& wk, double inv_m0, double kg, double ta,
                                          double ti, double tc, double& vk) {
  double q = L.q, x, y, z;
  if (GR) {
    const double s = wide_momentum<G, STORAGE>(L.m, L.v), k1 = ta * inv_m0;
    L.cq = fma(k1, s, L.cq);
    q = fma(k1, s, q);
  }
  double a = wk.accel(q, x, y, z);
  if (GR) {
    const double ir2 = rcp_full(fma(x, x, fma(y, y, z * z)));   // gr_accel
    a = fma(-kg * ir2 * ir2, q, a);
  }
  L.cv = fma(ti, a, L.cv);
  vk = fma(ti, a, L.v);
  const double s = wide_momentum<G, STORAGE>(L.m, vk);
  L.cq = fma((GR ? tc : ta + tc) * inv_m0, s, L.cq);
  renorm(L.q, L.cq);
  renorm(L.v, L.cv);
}

// Group scans of a component over planets (group_scan_incl and the others of
// wh_device.h): planet p's neighbour n places on is 4n lanes on in its row;
// in a group of two rows, also in the other row, found by rotating both.
// DOWN: reads planet p + n, else p - n.
template <int G, int N, bool DOWN> __device__ __forceinline__ double wide_shift(double v) {
  if (G <= 4) return dpp<(DOWN ? 0x100 : 0x110) + 4 * N>(v);
  const double t = N == 4 ? v : dpp<0x120 + (DOWN ? 16 - 4 * (N & 3) : 4 * (N & 3))>(v);
  int l0, l1, h0, h1;
  row_pair(__double2loint(t), l0, l1);
  row_pair(__double2hiint(t), h0, h1);
  const int r = (threadIdx.x >> 2) & 3;
  const bool odd = threadIdx.x & 16;
  if (DOWN) return odd || r + N >= 4 ? __hiloint2double(h1, l1) : __hiloint2double(h0, l0);
  return odd && r >= N ? __hiloint2double(h1, l1) : __hiloint2double(h0, l0);
}
template <int G> __device__ __forceinline__ double wide_scan_excl(double v, int p) {
  if (G == 1) return 0.0;
  double t = wide_shift<G, 1, false>(v);
  v = p >= 1 ? t : 0.0;
  t = wide_shift<G, 1, false>(v);
  v += p >= 1 ? t : 0.0;
  if (G >= 4) { t = wide_shift<G, 2, false>(v); v += p >= 2 ? t : 0.0; }
  if (G >= 8) { t = wide_shift<G, 4, false>(v); v += p >= 4 ? t : 0.0; }
  return v;
}
// v: the sum over the planet and the next one
template <int G> __device__ __forceinline__ double wide_suffix_rest(double v, int p) {
  if (G >= 4) { const double t = wide_shift<G, 2, true>(v); v += p + 2 < G ? t : 0.0; }
  if (G >= 8) { const double t = wide_shift<G, 4, true>(v); v += p + 4 < G ? t : 0.0; }
  return v;
}
template <int G> __device__ __forceinline__ double wide_suffix_excl(double v, int p) {
  if (G == 1) return 0.0;
  double t = wide_shift<G, 1, true>(v);
  v = p + 1 < G ? t : 0.0;
  t = wide_shift<G, 1, true>(v);
  v += p + 1 < G ? t : 0.0;
  return wide_suffix_rest<G>(v, p);
}

// The planet's constants in Jacobi coordinates (jac_const) and the kick there
// (kick_jacobi) on the lane's component.
struct WideJac {
  double Mi, inv_Mim1, w, ratio;
  int p;
};
template <int G> __device__ __forceinline__ WideJac wide_jac(double m0, double m, int lane) {
  WideJac c;
  c.p = (lane >> 2) & (G - 1);
  const double Mim1 = m0 + wide_scan_excl<G>(m, c.p);
  c.Mi = Mim1 + m;
  c.inv_Mim1 = 1.0 / Mim1;
  c.w = m / c.Mi;
  c.ratio = m0 / Mim1;
  return c;
}
template <int G, bool GR>
__device__ __forceinline__ void wide_kick_jacobi(WideLane& L, const WideKick<G, 0>& wk, const WideJac& jc, double kg,
                                                 double tau) {
#pragma clang fp contract(off)
  const double q = L.q + wide_scan_excl<G>(jc.w * L.q, jc.p);
  double x, y, z;
  const double a = wk.accel(q, x, y, z);
  const double jx = dpp<DPP_QUAD_0>(L.q), jy = dpp<DPP_QUAD_1>(L.q), jz = dpp<DPP_QUAD_2>(L.q);
  const double irq3 = rsqrt3_full(fma(x, x, fma(y, y, z * z)));
  const double kp = jc.Mi * rsqrt3_full(fma(jx, jx, fma(jy, jy, jz * jz)));
  const double kq = (jc.Mi * jc.ratio) * irq3;
  const double wq = L.m * irq3;
  const double c = fma(jc.ratio, wide_suffix_excl<G>(wq * q, jc.p), wide_scan_excl<G>(L.m * a, jc.p) * jc.inv_Mim1);
  const double s = (a - c) + (kp * L.q - kq * q);
  if (GR) {
    const double ir2 = rcp_full(fma(x, x, fma(y, y, z * z)));   // gr_accel
    const double g = (-kg * ir2 * ir2) * q;
    double u = L.m * g;
    if (G >= 2) {
      const double t = wide_shift<G, 1, true>(u);
      u = wide_suffix_rest<G>(fma(L.m, g, jc.p + 1 < G ? t : 0.0), jc.p);
    }
    L.cv += fma(tau, fma(u, jc.inv_Mim1, g), tau * s);
  } else {
    L.cv = fma(tau, s, L.cv);
  }
  renorm(L.q, L.cq);
  renorm(L.v, L.cv);
}

// The system's flags at a launch's end.
template <int G>
__device__ __forceinline__ void wide_flags(const StepParams& p, const WideLane& L, const KepDiag& dg, int lane) {
  int f = 0;
  if (L.pl >= 0) {
    if (!__builtin_isfinite(L.q) || !__builtin_isfinite(L.v)) f |= WH_F_NONFINITE;
    if (!(dg.bmin > 0.0)) f |= WH_F_HYPERBOLIC;
    if (!(dg.zmax <= p.zlim)) f |= WH_F_ZMAX;
  }
  f |= dpp_i<DPP_QUAD_0>(f) | dpp_i<DPP_QUAD_1>(f) | dpp_i<DPP_QUAD_2>(f);   // the planet's three components
  f = wide_or<G>(f);
  if ((lane & (4 * G - 1)) == 0 && L.sys >= 0) {
    p.flags[L.sys] |= (uint32_t)f;
    p.synced[L.sys] = 0;
  }
}

// step_lane for four lanes per planet.
template <int G, bool GR, int SCHEME, int KC, int STORAGE, bool JAC>
__device__ __forceinline__ void wide_steps(const StepParams& p, WideLane& L, double* block, int lane) {
  WideKick<G, STORAGE> wk;
  wk.init(block, lane, L.m);
  const double dt = L.dt, h = 0.5 * dt;
  const double inv_m0 = 1.0 / L.m0;
  const double kg = GR ? p.kgr * L.m0 * L.m0 : 0.0;
  KepDiag dg{0.0, 1.0e300};
  double vk;
  WideJac jc{};
  if constexpr (JAC) jc = wide_jac<G>(L.m0, L.m, lane);
  const double mu = JAC ? jc.Mi : L.m0;
  const int n_steps = p.n_steps;
  if constexpr (SCHEME == SCHEME_SABA) {
    const double c1dt = p.sc[0] * dt;
    const double sc1 = p.sc[1], sc2 = p.sc[2], sc3 = p.sc[3], sd0 = p.sd[0], sd1 = p.sd[1], sd2 = p.sd[2], sd3 = p.sd[3];
    const int n_units = p.saba_n;
    double tk = L.first ? c1dt : 2.0 * c1dt;
    for (int s = 0; s < n_steps; ++s) {
#pragma unroll 1
      for (int k = 0; k < n_units; ++k) {
        wide_drift<0>(L, mu, tk, dg);
        const double tb = (k == 0 ? sd0 : k == 1 ? sd1 : k == 2 ? sd2 : sd3) * dt;
        if constexpr (JAC) wide_kick_jacobi<G, GR>(L, wk, jc, kg, tb);
        else wide_kick<G, false, STORAGE>(L, wk, inv_m0, 0.0, 0.5 * tb, tb, 0.5 * tb, vk);
        tk = k + 1 < n_units ? (k == 0 ? sc1 : k == 1 ? sc2 : sc3) * dt : 2.0 * c1dt;
      }
    }
  } else if (SCHEME == WH_DKD) {
    double tk = L.first ? h : dt;
    for (int s = 0; s < n_steps; ++s) {
      wide_drift<KC>(L, mu, tk, dg);
      tk = dt;
      if constexpr (JAC) wide_kick_jacobi<G, GR>(L, wk, jc, kg, dt);
      else wide_kick<G, GR, STORAGE>(L, wk, inv_m0, kg, h, dt, h, vk);
    }
  } else {
    double ta = L.first ? 0.0 : h;
    double ti = L.first ? h : dt;
    for (int s = 0; s < n_steps; ++s) {
      if constexpr (JAC) wide_kick_jacobi<G, GR>(L, wk, jc, kg, ti);
      else wide_kick<G, GR, STORAGE>(L, wk, inv_m0, kg, ta, ti, h, vk);
      ta = h;
      ti = dt;
      wide_drift<KC>(L, mu, dt, dg);
    }
  }
  wide_flags<G>(p, L, dg, lane);
}

// Slot of a lane's planet.  STORAGE 0: one planet per lane (the groups of
// the pow2 and G8 packings lie in planet order, so wavefront w takes slots 16 w
// and on); 1: the split packing, whose 16-lane groups hold planet p in slots
// 2p and 2p + 1 (both are written).
template <int STORAGE> __device__ __forceinline__ int wide_slot(int w, int lane) {
  const int k = w * WIDE_SLOTS + (lane >> 2);
  return STORAGE == 1 ? 2 * k : k;
}

// Lanes 0..2 of a planet store their component; in the split packing's storage
// both of a planet's slots, adjacent, take the value.
template <int STORAGE> __device__ __forceinline__ void wide_put(double* row, double x) {
  if (STORAGE == 1) *(double2*)row = make_double2(x, x);
  else *row = x;
}
template <int STORAGE>
__device__ __forceinline__ void wide_store(const StepParams& p, const WideLane& L, int slot, int c, int lane) {
  if ((lane & 3) == 3) return;
  const int ns = p.ns;
  double* st = p.st + (size_t)c * ns + slot;
  const size_t r3 = (size_t)3 * ns;
  wide_put<STORAGE>(st, L.q);
  wide_put<STORAGE>(st + r3, L.v);
  wide_put<STORAGE>(st + 2 * r3 + ns, L.cq);
  wide_put<STORAGE>(st + 3 * r3 + ns, L.cv);
}

template <int G, bool GR, int SCHEME, int KC, int STORAGE, bool JAC>
__device__ __forceinline__ void wide_group(const StepParams& p, int w, double* block, int lane) {
  const int slot = wide_slot<STORAGE>(w, lane), c = wide_comp(lane), ns = p.ns;
  double* st = p.st + (size_t)c * ns + slot;
  const size_t r3 = (size_t)3 * ns;
  WideLane L;
  L.q = st[0];
  L.v = st[r3];
  L.cq = st[2 * r3 + ns];
  L.cv = st[3 * r3 + ns];
  L.m = p.st[(size_t)6 * ns + slot];
  L.m0 = p.m0s[slot];
  L.dt = p.dts[slot];
  L.sys = p.slot_sys[slot];
  L.pl = p.slot_pl[slot];
  L.first = L.sys >= 0 ? p.synced[L.sys] : 1;
  wide_steps<G, GR, SCHEME, KC, STORAGE, JAC>(p, L, block, lane);
  wide_store<STORAGE>(p, L, slot, c, lane);
}

// The persistent step kernel of this form, defined and instantiated in
// wh_wide_step.hip.  Up to four wavefronts per workgroup.
template <bool GR, int SCHEME, int KC, int STORAGE, bool JAC = false>
__global__ __launch_bounds__(256) void k_step_wide(StepParams p);

}  // namespace wh
