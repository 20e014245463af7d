// pm_adjoint.hip -- discrete adjoint of one time step of the update, for
// gradients of the hot-wall Nusselt number (Eq. 24) with respect to the
// per-cell log10(Da) field, the power-law index n and the Rayleigh number.
//
// One step maps the pre-collision state S_k to S_{k+1} = Stream(Collide(S_k)).
// Given lambda_{k+1} = dJ/dS_{k+1} (FP64, natural layout [14][ny][nx]):
//   1. mu* = Stream^T lambda_{k+1}: for each node x and direction q,
//      mu*_q(x) = lambda_q(x + e_q) when x + e_q is inside, otherwise
//      lambda_opp(q)(x) (bounce-back) -- with a minus sign for the thermal
//      populations leaving through the Dirichlet walls (anti-bounce-back);
//   2. lambda_k(x) = (dCollide/dS)^T mu*(x): the forward node update is
//      recomputed in FP64 from the stored state and differentiated in
//      reverse order, line by line;
//   3. the parameter derivatives (dCollide/dtheta)^T mu*(x) are accumulated
//      in FP64: per cell for log10(Da), per workgroup (fixed slot, fixed
//      order) for ln nu0, n (direct) and the thermal rate s_g.
// The local viscosity is an implicit function (the fixed point of Eq. (21)
// with Eqs. (15), (22), (23)); its derivative is taken with the implicit
// function theorem on G(y; A, B, log2 nu0, n) = 0, y = log2 nu, or on the
// clamp (nu = bound * nu0) when the bound is active.
#include "pm_device.h"

namespace pm {
namespace {

using namespace pm::dev;

constexpr double LN2 = 0.693147180559945309417232121458176568;
constexpr double LN10 = 2.302585092994045684017991454684364208;

// sqrt(x) and 1 / sqrt(x), x >= 0, to about an ulp: the hardware estimate and
// Goldschmidt's iteration twice (10 instructions; the library's square root and
// a division take 30).  At x = 0 (a cell without porous resistance) and at
// infinity (one whose resistance, squared, overflows) the iteration is 0 * inf:
// there the root is x, and its reciprocal the estimate.
struct Root {
  double sqrt, rsqrt;
};
__device__ __forceinline__ Root root(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  double g = x * y, h = 0.5 * y;
  double r = __builtin_fma(-h, g, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  r = __builtin_fma(-h, g, 0.5);
  g = __builtin_fma(g, r, g);
  h = __builtin_fma(h, r, h);
  g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
  constexpr int ZERO_OR_INF = 0x260;  // -0, +0 and +inf
  const bool edge = __builtin_amdgcn_class(x, ZERO_OR_INF);
  return Root{edge ? x : g, edge ? y : 2.0 * h};
}

// Viscosity of one node in FP64 with the data the adjoint needs.
struct NuSol {
  double nu, y, s, g2;
  int branch;  // 0: power law (root of G), 1: at nu_min, 2: at nu_max
};

__device__ __forceinline__ NuSol nu_fp64(const AdjParams& a, double A, double B) {
  NuSol r;
  if (!a.pow) {  // Newtonian: nu = nu0 (the bounds bracket 1), G = y - log2 nu0
    r.y = a.log2nu0;
    r.nu = a.nu0;
    r.s = frcp<double>(3.0 * r.nu + 0.5);
    r.g2 = A + B * r.s * r.s;
    r.branch = 0;
    return r;
  }
  const double hn = 0.5 * a.nm1;
  // Start: the closed-form root for A << B s^2, 3 nu >> 1/2, refined by a few
  // FP32 Newton steps on the hardware exp2 / log2 / reciprocal (about 1e-6 in
  // y), so that the FP64 Newton steps below converge in two or three.
  float yf;
  {
    const float lo = (float)a.y_lo, hi = (float)a.y_hi, lc0 = (float)a.lc0, nm1 = (float)a.nm1;
    const float Af = (float)A, Bf = (float)B;
    // log2(0) = -inf (no shear, or B below the FP32 range) lands on a bound
    yf = (lc0 + nm1 * (0.5f * __builtin_amdgcn_logf(Bf) - 1.5849625007f)) * (float)a.inv_n;
    yf = fminf(fmaxf(yf, lo), hi);
    for (int it = 0; it < NU_FP32_STEPS; ++it) {
      const float nu = __builtin_amdgcn_exp2f(yf);
      const float sf = __builtin_amdgcn_rcpf(3.0f * nu + 0.5f);
      const float g2 = Af + Bf * sf * sf;
      if (!(g2 > 0.0f)) break;  // no shear in FP32: leave it to the FP64 steps
      const float G = (yf - lc0) - 0.5f * nm1 * __builtin_amdgcn_logf(g2);
      const float dG = 1.0f + 3.0f * nm1 * Bf * sf * sf * sf * nu * __builtin_amdgcn_rcpf(g2);
      yf = fminf(fmaxf(yf - G * __builtin_amdgcn_rcpf(dG), lo), hi);
    }
  }
  double y = fmin(fmax((double)yf, a.y_lo), a.y_hi);
  if (!(y == y)) y = a.y_hi;  // NaN start (no shear at all): the FP64 steps decide
  // Newton converges quadratically here: G' lies between min(n, 1) and
  // max(n, 1) and G'' is of order |n - 1|, so a step of size d leaves an
  // error of order d^2.  A step below 1e-9 therefore ends the iteration
  // (the error left is below 1e-17) without a further step to confirm it;
  // from the FP32 start that is two FP64 steps.  nu after the last step is
  // 2^y of the iterate before times 2^d = 1 + t + t^2/2 (t = d ln 2, the
  // next term below 1e-28), and s = 1 / (3 nu + 1/2) to first order.
  // The steps between are small as well, since the start is good to 1e-6: up to
  // 2^-13 they take 2^d and log2(g2 / g2_old) from their series (the terms left
  // out are below 1e-19) instead of calling exp2 and log2 again.
  double nu = exp2(y);
  double s = frcp<double>(3.0 * nu + 0.5);
  double g2 = A + B * s * s;
  double L = log2(g2);
  for (int it = 0; it < 60; ++it) {
    // 1 / g2 overflows where g2 is subnormal (ahead of the front of a flow that
    // sets in from rest the shear falls by a tenth of a decade per node)
    const bool weak = g2 < 0x1p-1000;
    const double rg = 1.0 / g2, x = 3.0 * a.nm1 * B * s * s * s * nu;
    const double G = (y - a.lc0) - hn * L;
    const double dG = 1.0 + (weak ? x / g2 : x * rg);
    double yn = y - G * frcp<double>(dG);
    if (!(g2 > 0.0)) yn = G < 0.0 ? a.y_hi : a.y_lo;
    yn = fmin(fmax(yn, a.y_lo), a.y_hi);
    const double d = yn - y, t = d * LN2;
    y = yn;
    if (fabs(d) <= 1e-9) {
      const double dnu = nu * (t * (1.0 + 0.5 * t));
      nu += dnu;
      s -= 3.0 * dnu * s * s;
      break;
    }
    if (fabs(d) < 0x1p-13 && !weak) {
      nu *= 1.0 + t * (1.0 + t * (0.5 + t * (1.0 / 6.0 + t * (1.0 / 24.0))));
      s = frcp<double>(3.0 * nu + 0.5);
      const double g2n = A + B * s * s, e = (g2n - g2) * rg;
      L += (1.0 / LN2) * e * (1.0 - e * (0.5 - e * (1.0 / 3.0 - e * (0.25 - e * 0.2))));
      g2 = g2n;
    } else {
      nu = exp2(y);
      s = frcp<double>(3.0 * nu + 0.5);
      g2 = A + B * s * s;
      L = log2(g2);
    }
  }
  r.y = y;
  r.nu = nu;
  r.s = s;
  r.g2 = A + B * s * s;
  r.branch = (y <= a.y_lo) ? 1 : ((y >= a.y_hi) ? 2 : 0);
  return r;
}

// Reverse-mode derivative of the node update (Steps 2-9) at the state
// (df, dg) (shifted populations, FP64), seeded with mu = dJ/d(post-collision).
__device__ __forceinline__ void vjp_node(const AdjParams& a, const double df[9], const double dg[5],
                                         double logda, const double mf[9], const double mg[5],
                                         double lf[9], double lg[5], double& g_ld, double& g_lnnu0,
                                         double& g_n, double& g_sg) {
  const double eps = a.eps, ie = a.inv_eps;
  // ---------------- forward recompute ----------------
  const double drho = (df[0] + ((df[1] + df[2]) + (df[3] + df[4]))) + ((df[5] + df[6]) + (df[7] + df[8]));
  const double rho = 1.0 + drho;
  const double jx = ((df[1] - df[3]) + (df[5] - df[6])) - (df[7] - df[8]);
  const double jy = ((df[2] - df[4]) + (df[5] + df[6])) - (df[7] + df[8]);
  const double dT = dg[0] + ((dg[1] + dg[2]) + (dg[3] + dg[4]));
  const double Gx = a.gx;
  const double Gy = a.gy + a.gbeta * (dT - a.dTm);
  const double irho = frcp<double>(rho);
  const double vx = jx * irho + 0.5 * eps * Gx;
  const double vy = jy * irho + 0.5 * eps * Gy;
  const double s14 = (df[1] + df[2]) + (df[3] + df[4]);
  const double s58 = (df[5] + df[6]) + (df[7] + df[8]);
  const double m1 = (-4.0 * df[0] - s14) + 2.0 * s58;
  const double m7 = (df[1] - df[2]) + (df[3] - df[4]);
  const double m8 = (df[5] - df[6]) + (df[7] - df[8]);
  const double vxx = vx * vx, vyy = vy * vy;
  const double en = (m1 + 2.0 * drho) - 3.0 * rho * (vxx + vyy) * ie;
  const double pn = m7 - rho * (vxx - vyy) * ie;
  const double qn = m8 - rho * vx * vy * ie;
  const double irho2 = irho * irho;
  const double A = 0.25 * a.s_e * a.s_e * en * en * irho2;
  const double B = 2.25 * (pn * pn + 4.0 * qn * qn) * irho2;
  const NuSol ns = nu_fp64(a, A, B);
  const double nu = ns.nu;
  double invK, invsK;
  if (a.has_logda) {
    invK = exp2(-3.321928094887362347870319429489390175864831 * logda) * a.inv_Kscale;
    invsK = root(invK).sqrt;
  } else {
    invK = a.invK;
    invsK = a.invsK;
  }
  const double c0 = 0.5 * (1.0 + 0.5 * eps * nu * invK);
  const double c1 = 0.5 * eps * a.Feps * invsK;
  // |v|, 1 / |v| (0 at rest) and from them |u| and the direction of both
  const double v2 = vxx + vyy;
  const bool moves = v2 > 1e-290;
  const Root rv = root(moves ? v2 : 1.0);
  const double vm = moves ? rv.sqrt : 0.0, ivm = moves ? rv.rsqrt : 0.0;
  const Root rq = root(c0 * c0 + c1 * vm);
  const double iden = frcp<double>(c0 + rq.sqrt);
  const double ux = vx * iden, uy = vy * iden;
  const double um = vm * iden;
  const double drag = eps * nu * invK + eps * a.Feps * invsK * um;
  const double Fx = eps * Gx - drag * ux;
  const double Fy = eps * Gy - drag * uy;
  const double uu = ux * ux + uy * uy;
  const double uF = ux * Fx + uy * Fy;
  const double snu = ns.s;
  const double hnu = 1.0 - 0.5 * snu;
  // (m2, m4, m6 enter the collision linearly: only their adjoints are needed)
  const double P7 = rho * (ux * ux - uy * uy) * ie, Q7 = 2.0 * rho * (ux * Fx - uy * Fy) * ie;
  const double P8 = rho * ux * uy * ie, Q8 = rho * (ux * Fy + uy * Fx) * ie;
  const double Tabs = a.T_ref + dT;
  const double n1 = dg[1] - dg[3], n2 = dg[2] - dg[4];

  // ---------------- reverse sweep ----------------
  // Step 9: g* = N^-1 (dT, ns1..ns4)
  const double bn0 = (mg[0] + mg[1] + mg[2] + mg[3] + mg[4]) * 0.2;
  const double bn1 = (mg[1] - mg[3]) * 0.5;
  const double bn2 = (mg[2] - mg[4]) * 0.5;
  const double bn3 = (-4.0 * mg[0] + mg[1] + mg[2] + mg[3] + mg[4]) * 0.05;
  const double bn4 = (mg[1] - mg[2] + mg[3] - mg[4]) * 0.25;
  double b_ux = 0.0, b_uy = 0.0, b_dT = 0.0, b_Tabs = 0.0, b_sg = 0.0;
  const double b_n1 = (1.0 - a.s_g) * bn1;
  b_ux += a.s_g * Tabs * bn1;
  b_Tabs += a.s_g * ux * bn1;
  b_sg += (ux * Tabs - n1) * bn1;
  const double b_n2 = (1.0 - a.s_g) * bn2;
  b_uy += a.s_g * Tabs * bn2;
  b_Tabs += a.s_g * uy * bn2;
  b_sg += (uy * Tabs - n2) * bn2;
  const double b_n3 = (1.0 - a.sT_e) * bn3;
  b_dT += -a.sT_e * (2.0 / 3.0) * bn3;
  const double b_n4 = (1.0 - a.sT_nu) * bn4;
  b_dT += bn0;
  b_dT += b_Tabs;

  // Step 8: f* = M^-1 ms
  const double sm58 = (mf[5] + mf[6]) + (mf[7] + mf[8]);
  const double sm14 = (mf[1] + mf[2]) + (mf[3] + mf[4]);
  // (the row norms 9, 36, 6, 12 of M as multiplications: FP64 division is a
  // long instruction sequence on this path)
  constexpr double i9 = 1.0 / 9.0, i36 = 1.0 / 36.0, i6 = 1.0 / 6.0, i12 = 1.0 / 12.0;
  const double bm0 = (mf[0] + sm14 + sm58) * i9;
  const double bm1 = (-4.0 * mf[0] - sm14 + 2.0 * sm58) * i36;
  const double bm2 = (4.0 * mf[0] - 2.0 * sm14 + sm58) * i36;
  const double bm3 = ((mf[1] - mf[3]) + (mf[5] - mf[6]) - (mf[7] - mf[8])) * i6;
  const double bm4 = (-2.0 * (mf[1] - mf[3]) + (mf[5] - mf[6]) - (mf[7] - mf[8])) * i12;
  const double bm5 = ((mf[2] - mf[4]) + (mf[5] + mf[6]) - (mf[7] + mf[8])) * i6;
  const double bm6 = (-2.0 * (mf[2] - mf[4]) + (mf[5] + mf[6]) - (mf[7] + mf[8])) * i12;
  const double bm7 = ((mf[1] - mf[2]) + (mf[3] - mf[4])) * 0.25;
  const double bm8 = ((mf[5] - mf[6]) + (mf[7] - mf[8])) * 0.25;
  double b_drho = bm0, b_rho = 0.0, b_Fx = 0.0, b_Fy = 0.0, b_snu = 0.0, b_hnu = 0.0;
  double b_m1 = 0.0, b_m7 = 0.0, b_m8 = 0.0;
  double b_ruu = 0.0, b_Fm1 = 0.0, b_rux = 0.0, b_ruy = 0.0;
  // ms1 = (1 - se) m1 + se (-2 drho + ruu) + (1 - se/2) Fm1
  b_m1 += (1.0 - a.s_e) * bm1;
  b_drho += -2.0 * a.s_e * bm1;
  b_ruu += a.s_e * bm1;
  b_Fm1 += (1.0 - 0.5 * a.s_e) * bm1;
  // ms2 = (1 - seps) m2 + seps (drho - ruu) - (1 - seps/2) Fm1
  const double b_m2 = (1.0 - a.s_eps) * bm2;
  b_drho += a.s_eps * bm2;
  b_ruu += -a.s_eps * bm2;
  b_Fm1 += -(1.0 - 0.5 * a.s_eps) * bm2;
  // ms3 = rux + rho Fx / 2
  b_rux += bm3;
  b_rho += 0.5 * Fx * bm3;
  b_Fx += 0.5 * rho * bm3;
  // ms4 = (1 - sq) m4 - sq rux - (1 - sq/2) rho Fx
  const double b_m4 = (1.0 - a.s_q) * bm4;
  b_rux += -a.s_q * bm4;
  b_rho += -(1.0 - 0.5 * a.s_q) * Fx * bm4;
  b_Fx += -(1.0 - 0.5 * a.s_q) * rho * bm4;
  // ms5, ms6
  b_ruy += bm5;
  b_rho += 0.5 * Fy * bm5;
  b_Fy += 0.5 * rho * bm5;
  const double b_m6 = (1.0 - a.s_q) * bm6;
  b_ruy += -a.s_q * bm6;
  b_rho += -(1.0 - 0.5 * a.s_q) * Fy * bm6;
  b_Fy += -(1.0 - 0.5 * a.s_q) * rho * bm6;
  // ms7 = (1 - snu) m7 + snu P7 + hnu Q7
  b_m7 += (1.0 - snu) * bm7;
  b_snu += (P7 - m7) * bm7;
  b_hnu += Q7 * bm7;
  double b_ux2 = 0.0, b_uy2 = 0.0;  // collected below into b_ux, b_uy
  {
    const double bP = snu * bm7, bQ = hnu * bm7;
    b_rho += (ux * ux - uy * uy) * ie * bP + 2.0 * (ux * Fx - uy * Fy) * ie * bQ;
    b_ux2 += 2.0 * rho * ux * ie * bP + 2.0 * rho * Fx * ie * bQ;
    b_uy2 += -2.0 * rho * uy * ie * bP - 2.0 * rho * Fy * ie * bQ;
    b_Fx += 2.0 * rho * ux * ie * bQ;
    b_Fy += -2.0 * rho * uy * ie * bQ;
  }
  // ms8 = (1 - snu) m8 + snu P8 + hnu Q8
  b_m8 += (1.0 - snu) * bm8;
  b_snu += (P8 - m8) * bm8;
  b_hnu += Q8 * bm8;
  {
    const double bP = snu * bm8, bQ = hnu * bm8;
    b_rho += ux * uy * ie * bP + (ux * Fy + uy * Fx) * ie * bQ;
    b_ux2 += rho * uy * ie * bP + rho * Fy * ie * bQ;
    b_uy2 += rho * ux * ie * bP + rho * Fx * ie * bQ;
    b_Fy += rho * ux * ie * bQ;
    b_Fx += rho * uy * ie * bQ;
  }
  b_ux += b_ux2;
  b_uy += b_uy2;
  b_snu += -0.5 * b_hnu;
  double b_nu = b_snu * (-3.0 * snu * snu);
  // Fm1 = 6 rho uF / eps
  b_rho += 6.0 * uF * ie * b_Fm1;
  const double b_uF = 6.0 * rho * ie * b_Fm1;
  b_ux += Fx * b_uF;
  b_uy += Fy * b_uF;
  b_Fx += ux * b_uF;
  b_Fy += uy * b_uF;
  // ruu = 3 rho uu / eps
  b_rho += 3.0 * uu * ie * b_ruu;
  const double b_uu = 3.0 * rho * ie * b_ruu;
  b_ux += 2.0 * ux * b_uu;
  b_uy += 2.0 * uy * b_uu;
  // rux = rho ux, ruy = rho uy
  b_rho += ux * b_rux + uy * b_ruy;
  b_ux += rho * b_rux;
  b_uy += rho * b_ruy;

  // Step 7: F = eps G - drag u, drag = eps nu invK + eps Feps invsK |u|
  double b_Gx = eps * b_Fx, b_Gy = eps * b_Fy;
  const double b_drag = -(ux * b_Fx + uy * b_Fy);
  b_ux += -drag * b_Fx;
  b_uy += -drag * b_Fy;
  b_nu += eps * invK * b_drag;
  double b_invK = eps * nu * b_drag;
  double b_invsK = eps * a.Feps * um * b_drag;
  const double b_um = eps * a.Feps * invsK * b_drag;
  const double ex = vx * ivm, ey = vy * ivm;
  b_ux += ex * b_um;
  b_uy += ey * b_um;

  // Step 6: u = v / (c0 + sqrt(c0^2 + c1 |v|))
  double b_vx = iden * b_ux, b_vy = iden * b_uy;
  const double b_iden = vx * b_ux + vy * b_uy;
  const double b_den = -iden * iden * b_iden;
  // (c0 >= 1/2: the root is not zero)
  const double b_rq = b_den * rq.rsqrt;
  const double b_c0 = b_den + c0 * b_rq;
  const double b_c1 = 0.5 * vm * b_rq;
  const double b_vm = 0.5 * c1 * b_rq;
  b_vx += ex * b_vm;
  b_vy += ey * b_vm;
  b_nu += 0.25 * eps * invK * b_c0;
  b_invK += 0.25 * eps * nu * b_c0;
  b_invsK += 0.5 * eps * a.Feps * b_c1;
  // invK = 10^-logDa / N^2, invsK = sqrt(invK)
  g_ld = a.has_logda ? (-LN10 * invK * b_invK - 0.5 * LN10 * invsK * b_invsK) : 0.0;

  // Step 5: nu from (A, B, log2 nu0, n) -- implicit function / clamp
  double b_A = 0.0, b_B = 0.0;
  g_lnnu0 = 0.0;
  g_n = 0.0;
  if (ns.branch != 0) {
    g_lnnu0 += nu * b_nu;  // nu = bound * nu0
  } else {
    const double b_y = b_nu * nu * LN2;  // nu = 2^y
    // dy = -(G_A dA + G_B dB + G_L0 dL0 + G_n dn) / G', with 1 / G' = g2 / (g2 + x)
    constexpr double ILN2 = 1.0 / LN2;
    const double x = a.pow ? 3.0 * a.nm1 * B * ns.s * ns.s * ns.s * ns.nu : 0.0;
    const double bg = b_y / (ns.g2 + x);
    const double w = a.pow ? bg * ns.g2 : b_y;
    g_lnnu0 += w * ILN2;  // L0 = log2 nu0, G_L0 = -1
    // At zero shear (possible only with n = 1, where no clamp is active) the
    // power law is singular in n and its one-sided limits sit on a clamp,
    // which does not depend on n at fixed nu0: no n or shear terms.
    if (ns.g2 > 0.0) {
      // G_n = -log2(gamma*).  At the root G = 0 gives log2(g2) = (y - lc0) / hn
      // (to the root's error over hn; the log is taken where hn is small).
      const double l2g2 = a.inv_hn != 0.0 ? (ns.y - a.lc0) * a.inv_hn : log2(ns.g2);
      g_n += w * (a.log2c + 0.5 * l2g2);
      if (ns.g2 > a.g2_floor) {
        const double wg = bg * 0.5 * a.nm1 * ILN2;
        b_A += wg;
        b_B += wg * ns.s * ns.s;
      }
    }
  }
  // A = se^2 en^2 irho2 / 4, B = 9 (pn^2 + 4 qn^2) irho2 / 4
  const double b_en = 0.5 * a.s_e * a.s_e * en * irho2 * b_A;
  const double b_pn = 4.5 * pn * irho2 * b_B;
  const double b_qn = 18.0 * qn * irho2 * b_B;
  const double b_irho2 = 0.25 * a.s_e * a.s_e * en * en * b_A + 2.25 * (pn * pn + 4.0 * qn * qn) * b_B;
  double b_irho = 2.0 * irho * b_irho2;
  // en, pn, qn
  b_m1 += b_en;
  b_drho += 2.0 * b_en;
  b_rho += -3.0 * (vxx + vyy) * ie * b_en - (vxx - vyy) * ie * b_pn - vx * vy * ie * b_qn;
  const double b_vxx = -3.0 * rho * ie * b_en - rho * ie * b_pn;
  const double b_vyy = -3.0 * rho * ie * b_en + rho * ie * b_pn;
  b_m7 += b_pn;
  b_m8 += b_qn;
  b_vx += 2.0 * vx * b_vxx - rho * vy * ie * b_qn;
  b_vy += 2.0 * vy * b_vyy - rho * vx * ie * b_qn;

  // Step 4: v = j / rho + eps G / 2
  const double b_jx = irho * b_vx, b_jy = irho * b_vy;
  b_irho += jx * b_vx + jy * b_vy;
  b_Gx += 0.5 * eps * b_vx;
  b_Gy += 0.5 * eps * b_vy;
  b_rho += -irho * irho * b_irho;
  // Step 3: Gy = gy + gbeta (dT - dTm)
  b_dT += a.gbeta * b_Gy;
  (void)b_Gx;
  // Step 2
  b_drho += b_rho;
  // populations: drho, jx, jy and the moments m1, m2, m4, m6, m7, m8 are
  // linear in df (rows of M)
  lf[0] = b_drho - 4.0 * b_m1 + 4.0 * b_m2;
  lf[1] = b_drho + b_jx - b_m1 - 2.0 * b_m2 - 2.0 * b_m4 + b_m7;
  lf[2] = b_drho + b_jy - b_m1 - 2.0 * b_m2 - 2.0 * b_m6 - b_m7;
  lf[3] = b_drho - b_jx - b_m1 - 2.0 * b_m2 + 2.0 * b_m4 + b_m7;
  lf[4] = b_drho - b_jy - b_m1 - 2.0 * b_m2 + 2.0 * b_m6 - b_m7;
  lf[5] = b_drho + b_jx + b_jy + 2.0 * b_m1 + b_m2 + b_m4 + b_m6 + b_m8;
  lf[6] = b_drho - b_jx + b_jy + 2.0 * b_m1 + b_m2 - b_m4 + b_m6 - b_m8;
  lf[7] = b_drho - b_jx - b_jy + 2.0 * b_m1 + b_m2 - b_m4 - b_m6 + b_m8;
  lf[8] = b_drho + b_jx - b_jy + 2.0 * b_m1 + b_m2 + b_m4 - b_m6 - b_m8;
  // thermal: dT, n1..n4 are linear in dg (rows of N)
  lg[0] = b_dT - 4.0 * b_n3;
  lg[1] = b_dT + b_n1 + b_n3 + b_n4;
  lg[2] = b_dT + b_n2 + b_n3 - b_n4;
  lg[3] = b_dT - b_n1 + b_n3 + b_n4;
  lg[4] = b_dT - b_n2 + b_n3 - b_n4;
  g_sg = b_sg;
}

// Adjoint of the streaming step: mu*_q(x) from lambda_{k+1} (natural layout).
// Each lambda value is read by at most two nodes of a launch (its pull
// neighbour, and the node itself at a wall) and written once, so the loads
// here and the stores in k_adjoint are non-temporal; measured 2-8% faster per
// launch from 256^2 to 4096^2 than cached accesses.
// The adjoint state is stored as L: double, or float for FP32 forward states
// (the arithmetic stays FP64; only the values kept between steps are
// rounded, to nearest).  gather_mu only loads; mu_signs then applies the
// anti-bounce-back sign of the Dirichlet walls, so that no arithmetic on a
// loaded value (and no wait for it) sits between the node's loads.
// Every address below is a select between two indices whose row parts are
// wave-uniform (j is the workgroup's row) and whose column part is the lane's,
// with the inside test as a bitwise and: no branches between the loads.
template <typename L>
__device__ __forceinline__ void gather_mu(const AdjParams& a, const L* __restrict__ lam, int i, int j,
                                          L rf[9], L rg[5]) {
  const int nx = a.nx, ny = a.ny;
  const int64_t nn = (int64_t)nx * ny, k = (int64_t)j * nx + i;
  const bool in_ip = i + 1 < nx, in_im = i >= 1, in_jp = j + 1 < ny, in_jm = j >= 1;
  const int64_t r0 = (int64_t)j * nx;
#pragma unroll
  for (int q = 0; q < 14; ++q) {
    const int d = q < 9 ? q : q - 9;  // direction within D2Q9 / D2Q5
    const int od = OPP[d] + (q < 9 ? 0 : 9);
    const bool in = (EXv[d] > 0 ? in_ip : (EXv[d] < 0 ? in_im : true)) &
                    (EYv[d] > 0 ? in_jp : (EYv[d] < 0 ? in_jm : true));
    const int64_t idx = in ? q * nn + r0 + EYv[d] * (int64_t)nx + (i + EXv[d]) : od * nn + k;
    const L v = __builtin_nontemporal_load(&lam[idx]);
    if (q < 9) rf[q] = v;
    else rg[q - 9] = v;
  }
}

template <typename L>
__device__ __forceinline__ void mu_signs(const AdjParams& a, int i, const L rf[9], const L rg[5], double mf[9],
                                         double mg[5]) {
#pragma unroll
  for (int q = 0; q < 9; ++q) mf[q] = (double)rf[q];
#pragma unroll
  for (int q = 0; q < 5; ++q) {
    const double v = (double)rg[q];
    const bool wall = (EXv[q] == 1 && i + 1 >= a.nx) || (EXv[q] == -1 && i == 0);
    mg[q] = wall ? -v : v;  // anti-bounce-back at the hot and cold walls
  }
}

// op over the 64 lanes of a wave (all active, values >= 0 or op a sum), in lane
// 63: rotations within the rows of 16, then the rows' results broadcast upwards.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp(double v) {
  const uint64_t w = __builtin_bit_cast(uint64_t, v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)w, CTRL, ROWS, 0xf, false);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(w >> 32), CTRL, ROWS, 0xf, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <typename Op>
__device__ __forceinline__ double wave_total(double v, Op op) {
  constexpr int ROW_ROR = 0x120, BCAST15 = 0x142, BCAST31 = 0x143;
  v = op(v, dpp<ROW_ROR + 8, 0xf>(v));
  v = op(v, dpp<ROW_ROR + 4, 0xf>(v));
  v = op(v, dpp<ROW_ROR + 2, 0xf>(v));
  v = op(v, dpp<ROW_ROR + 1, 0xf>(v));
  v = op(v, dpp<BCAST15, 0xa>(v));  // rows 1 and 3 take in rows 0 and 2
  return op(v, dpp<BCAST31, 0xc>(v));  // rows 2 and 3 take in row 1
}

// Each wave of a workgroup takes a segment of 64 nodes of a row, the segments of
// all rows numbered one after the other: no wave idles at the end of a row.  (With
// a workgroup of four waves per 256 nodes of one row a backward step at 300^2
// takes 17.1 us instead of 12.6.)
__host__ __device__ inline int64_t adj_groups(int nx, int ny) {
  return ((int64_t)((nx + 63) / 64) * ny + TILE / 64 - 1) / (TILE / 64);
}
__device__ __forceinline__ bool wave_segment(int nx, int ny, int blk, int& i0, int& j) {
  const int segs = (nx + 63) / 64;
  const int s = __builtin_amdgcn_readfirstlane(blk * (TILE / 64) + ((int)threadIdx.x >> 6));
  j = s / segs;
  i0 = (s - j * segs) * 64;
  return j < ny;
}

// What bounds it on small grids is one wave's chain of FP64 instructions (about
// 1300) between two memory round trips: 256^2 alone 6.3 us, 7.4 with library
// square roots, one division per quotient, exp2 and log2 in every Newton step
// and LDS permutes in the sums.  184 registers, two waves per SIMD; three spill
// (512^2 28.9 us per backward step against 25.3).
// ODD: the parity of the step whose state is read (a template parameter, so
// that each variant's loads are one straight-line sequence).
template <typename S, typename L, bool ODD>
__device__ __forceinline__ void adjoint_tile(const KParams<S>& st, const AdjParams& a, const L* __restrict__ lam_next,
                                             L* __restrict__ lam, double* __restrict__ g_logda,
                                             double* __restrict__ partial, int blk) {
  static_assert(TILE % 64 == 0, "whole waves per workgroup");
  constexpr int NW = TILE / 64;  // waves per workgroup
  __shared__ double red[ADJ_PART][NW];
  int i0, j;
  const bool some = wave_segment(a.nx, a.ny, blk, i0, j);
  const int i = i0 + ((int)threadIdx.x & 63);
  double c_lnnu0 = 0.0, c_n = 0.0, c_sg = 0.0, lmax = 0.0;
  // The workgroup's partials and the node's gradient are read, updated and
  // written back; their reads are issued with the node's loads, so that the
  // end of the wave does not wait on a load.
  double p_old = 0.0;
  if (threadIdx.x < ADJ_PART) p_old = partial[ADJ_PART * (int64_t)blk + threadIdx.x];
  if (some && i < a.nx) {
    // Loads in this order: lambda_{k+1}, the old gradient, the state (whose
    // wall conditions need their values), log10 Da.  Each wait then covers
    // loads that are all in flight already: one memory round trip.
    const int64_t k = (int64_t)j * a.nx + i, nn = (int64_t)a.nx * a.ny;
    L rf[9], rg[5];
    gather_mu(a, lam_next, i, j, rf, rg);
    const double gl_old = a.has_logda ? g_logda[k] : 0.0;
    S sf[9], sg[5];
    load_node_raw<S, ODD>(st, i, j, sf, sg);
    const double ld = a.has_logda ? (double)st.logda[k] : 0.0;
    if (ODD) pull_walls(st, i, sg);
    double df[9], dg[5], mf[9], mg[5], lf[9], lg[5];
#pragma unroll
    for (int q = 0; q < 9; ++q) df[q] = (double)sf[q];
#pragma unroll
    for (int q = 0; q < 5; ++q) dg[q] = (double)sg[q];
    mu_signs(a, i, rf, rg, mf, mg);
    double g_ld;
    vjp_node(a, df, dg, ld, mf, mg, lf, lg, g_ld, c_lnnu0, c_n, c_sg);
    double nan = 0.0;  // turns to NaN with a NaN or an infinity among the values: both count as unbounded
#pragma unroll
    for (int q = 0; q < 9; ++q) {
      __builtin_nontemporal_store((L)lf[q], &lam[q * nn + k]);
      lmax = fmax(lmax, fabs(lf[q]));
      nan = __builtin_fma(lf[q], 0.0, nan);
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) {
      __builtin_nontemporal_store((L)lg[q], &lam[(9 + q) * nn + k]);
      lmax = fmax(lmax, fabs(lg[q]));
      nan = __builtin_fma(lg[q], 0.0, nan);
    }
    if (nan != nan) lmax = INFINITY;
    if (a.has_logda) g_logda[k] = gl_old + g_ld;
  }
  // Workgroup sums (and the max): over the 64 lanes of each wave by DPP, then
  // the NW wave results in wave order, in one fixed order.
  c_lnnu0 = wave_total(c_lnnu0, [](double u, double v) { return u + v; });
  c_n = wave_total(c_n, [](double u, double v) { return u + v; });
  c_sg = wave_total(c_sg, [](double u, double v) { return u + v; });
  lmax = wave_total(lmax, [](double u, double v) { return fmax(u, v); });
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 63) {
    red[0][wv] = c_lnnu0;
    red[1][wv] = c_n;
    red[2][wv] = c_sg;
    red[3][wv] = lmax;
  }
  __syncthreads();
  if (threadIdx.x < ADJ_PART) {
    const int q = threadIdx.x;
    double v = red[q][0];
#pragma unroll
    for (int w = 1; w < NW; ++w) v = q < 3 ? v + red[q][w] : fmax(v, red[q][w]);
    partial[ADJ_PART * (int64_t)blk + q] = q < 3 ? p_old + v : fmax(p_old, v);
  }
}

template <typename S, typename L, bool ODD>
__global__ __launch_bounds__(TILE) void k_adjoint(KParams<S> st, AdjParams a, const L* __restrict__ lam_next,
                                                  L* __restrict__ lam, double* __restrict__ g_logda,
                                                  double* __restrict__ partial) {
  adjoint_tile<S, L, ODD>(st, a, lam_next, lam, g_logda, partial, blockIdx.x);
}

// The adjoint step and, in a second half of the grid (same tiles), one
// out-of-place forward step src -> dst of another state (src_odd: its parity):
// the replay of the segment that the adjoint reads next.  A small grid leaves
// the SIMDs one wave of the adjoint each, which waits most of the time; one
// launch per step pair instead of two also halves what the host has to submit.
// Backward, us per step, two launches on two streams / one (FP32 state): 100^2
// 8.5 / 7.1, 160^2 9.4 / 7.6, 256^2 9.5 / 8.7, 360^2 18.9 / 17.6, 420^2 22 / 22,
// 512^2 25.3 / 26.2; FP64 state: 100^2 8.4 / 7.2, 200^2 10.2 / 9.5, 256^2 10.1 ..
// 10.8 / 10.7, 300^2 14.2 / 15.4.
template <typename S, typename L, bool ODD, bool POW, bool LOGDA>
__global__ __launch_bounds__(TILE) void k_adjoint_replay(KParams<S> st, AdjParams a, const L* __restrict__ lam_next,
                                                         L* __restrict__ lam, double* __restrict__ g_logda,
                                                         double* __restrict__ partial, int nadj, KParams<S> src,
                                                         KParams<S> dst, int src_odd) {
  if ((int)blockIdx.x < nadj) {
    adjoint_tile<S, L, ODD>(st, a, lam_next, lam, g_logda, partial, blockIdx.x);
    return;
  }
  const int blk = (int)blockIdx.x - nadj;
  int i0, j;
  if (!wave_segment(a.nx, a.ny, blk, i0, j)) return;
  if constexpr (std::is_same<S, float>::value) {
    if (src.sr) {
      if (src_odd) step_tile<S, true, POW, LOGDA, true, true>(src, dst, i0, j, threadIdx.x & 63);
      else step_tile<S, false, POW, LOGDA, true, true>(src, dst, i0, j, threadIdx.x & 63);
      return;
    }
  }
  if (src_odd) step_tile<S, true, POW, LOGDA, false, true>(src, dst, i0, j, threadIdx.x & 63);
  else step_tile<S, false, POW, LOGDA, false, true>(src, dst, i0, j, threadIdx.x & 63);
}

// lambda_T = dJ/dS_T for J = Nu_bar (Eq. 24): only the thermal populations of
// the two hot-wall columns contribute.
template <typename L>
__global__ void k_adjoint_seed(int nx, int ny, double seed, L* __restrict__ lam) {
  const int64_t nn = (int64_t)nx * ny;
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < 14 * nn;
       t += (int64_t)gridDim.x * blockDim.x) {
    const int q = (int)(t / nn);
    const int64_t k = t - q * nn;
    const int i = (int)(k % nx);
    double v = 0.0;
    if (q >= 9) {
      if (i == 0) v = -3.0 * nx / (double)ny;
      else if (i == 1) v = nx / (3.0 * ny);
    }
    lam[t] = (L)(seed * v);
  }
}

__global__ __launch_bounds__(256) void k_fill_zero(double* __restrict__ a, int64_t n) {
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x)
    a[t] = 0.0;
}

// The per-workgroup adjoint partials reduced in workgroup order, as the host
// reduces them: out[q] = sum_b partial[b][q] for q < 3, out[3] = max_b
// partial[b][3] with a NaN turning it to +inf.  One thread per component, so
// the sums are added in exactly that order.
__global__ void k_adj_reduce(const double* __restrict__ partial, int nblocks, double* __restrict__ out) {
  const int q = threadIdx.x;
  if (q >= ADJ_PART) return;
  double acc = 0.0;
  for (int b = 0; b < nblocks; ++b) {
    const double m = partial[ADJ_PART * (int64_t)b + q];
    if (q < 3) acc += m;
    else acc = (m != m) ? INFINITY : (acc < m ? m : acc);
  }
  out[q] = acc;
}

}  // namespace

hipError_t launch_fill_zero(double* a, int64_t n, hipStream_t s) {
  int64_t b = (n + 255) / 256;
  if (b > 4096) b = 4096;
  if (b < 1) b = 1;
  hipLaunchKernelGGL(k_fill_zero, dim3((unsigned)b), dim3(256), 0, s, a, n);
  return hipGetLastError();
}

hipError_t launch_adj_reduce(const double* partial, int nblocks, double* out, hipStream_t s) {
  hipLaunchKernelGGL(k_adj_reduce, dim3(1), dim3(64), 0, s, partial, nblocks, out);
  return hipGetLastError();
}

template <typename S, typename L>
hipError_t launch_adjoint(const KParams<S>& st, const AdjParams& a, int parity, const L* lam_next, L* lam,
                          double* g_logda, double* partial, hipStream_t s, const Replay<S>* rp) {
  const int n = (int)adj_groups(a.nx, a.ny);
  if (rp) {
#define PM_R(ODD, POW, LOG)                                                                                         \
  hipLaunchKernelGGL((k_adjoint_replay<S, L, ODD, POW, LOG>), dim3(2 * n), dim3(TILE), 0, s, st, a, lam_next, lam,   \
                     g_logda, partial, n, rp->src, rp->dst, rp->parity)
#define PM_R_ALL(ODD)                                                                      \
  if (a.pow) { if (a.has_logda) PM_R(ODD, true, true); else PM_R(ODD, true, false); }       \
  else { if (a.has_logda) PM_R(ODD, false, true); else PM_R(ODD, false, false); }
    if (parity) { PM_R_ALL(true) } else { PM_R_ALL(false) }
#undef PM_R_ALL
#undef PM_R
    return hipGetLastError();
  }
  if (parity)
    hipLaunchKernelGGL((k_adjoint<S, L, true>), dim3(n), dim3(TILE), 0, s, st, a, lam_next, lam,
                       g_logda, partial);
  else
    hipLaunchKernelGGL((k_adjoint<S, L, false>), dim3(n), dim3(TILE), 0, s, st, a, lam_next, lam,
                       g_logda, partial);
  return hipGetLastError();
}

template <typename L>
hipError_t launch_adjoint_seed(int nx, int ny, double seed, L* lam, hipStream_t s) {
  const int64_t n = 14 * (int64_t)nx * ny;
  int64_t b = (n + 255) / 256;
  if (b > 65536) b = 65536;
  hipLaunchKernelGGL((k_adjoint_seed<L>), dim3((unsigned)b), dim3(256), 0, s, nx, ny, seed, lam);
  return hipGetLastError();
}

template hipError_t launch_adjoint<float, double>(const KParams<float>&, const AdjParams&, int, const double*,
                                                  double*, double*, double*, hipStream_t, const Replay<float>*);
template hipError_t launch_adjoint<float, float>(const KParams<float>&, const AdjParams&, int, const float*,
                                                 float*, double*, double*, hipStream_t, const Replay<float>*);
template hipError_t launch_adjoint<double, double>(const KParams<double>&, const AdjParams&, int, const double*,
                                                   double*, double*, double*, hipStream_t, const Replay<double>*);
template hipError_t launch_adjoint_seed<double>(int, int, double, double*, hipStream_t);
template hipError_t launch_adjoint_seed<float>(int, int, double, float*, hipStream_t);

}  // namespace pm
