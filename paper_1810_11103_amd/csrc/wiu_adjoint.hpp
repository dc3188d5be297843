// Hand-written reverse mode (vector-Jacobian products) of the device building
// blocks in wiu_device.hpp, metrics held fixed.  Each routine recomputes the
// forward quantities it needs in registers and then applies the chain rule
// backwards; "bar" variables are adjoints.  Non-smooth points: the mappings
// are C^1 at w = C (both pieces have zero slope there); |x| uses sign(0) = 0.
#pragma once

#include "wiu_device.hpp"

namespace wiu {

// ---------------------------------------------------------------------------
// WENO r = 3 (inputs a, b, d, e around the zero centre) -- see weno5, whose
// quantities are used throughout: with p_k the candidates times 8 c_k, E_k =
// eps + IS_k and D_k = E_k^2, P_k the products of the other two D, S_P =
// sum c_k P_k, r = 1/S_P, x_k = 16 P_k r - 1, g_k = 1 + K_k x_k^3 (in units of
// C_k), S = sum c_k g_k, N = sum g_k p_k, the value is out = N / (8 S).  Returns
// out; v[] enters as the inputs and leaves as out's derivatives by them.
// ---------------------------------------------------------------------------
template <bool PPM> WIU_DEV double weno5_grad(double v[4], double eps) {
  const double a = v[0], b = v[1], d = v[2], e = v[3];
  const double c[3] = {1.0, 10.0, 5.0};
  const double KL[3] = {WIU_M3L0 / 256.0, WIU_M3L1 * (0.625 * 0.625), WIU_M3L2 * (0.3125 * 0.3125)};
  const double KH[3] = {WIU_M3H0 / 256.0, WIU_M3H1 * (0.625 * 0.625), WIU_M3H2 * (0.3125 * 0.3125)};
  const double b10 = 10.0 * b, d30 = 30.0 * d;
  const double p[3] = {fma(3.0, a, -b10), d30 - b10, fma(-5.0, e, d30)};
  const double t[3] = {fma(-2.0, b, a), b + d, fma(-2.0, d, e)};
  const double u[3] = {fma(-0.5, a, t[0]), fma(0.5, t[1], -d), fma(-0.5, e, t[2])};
  double E[3], D[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    E[k] = fma(13.0 / 12.0, t[k] * t[k], fma(u[k], u[k], eps));
    D[k] = E[k] * E[k];
  }
  const double P[3] = {D[1] * D[2], D[0] * D[2], D[0] * D[1]};
  const double r = rcp_w(fma(10.0, P[1], fma(5.0, P[2], P[0])));
  const double r16 = 16.0 * r;
  double x[3], g[3], gx[3];  // gx = dg/dx / 3
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    x[k] = fma(P[k], r16, -1.0);
    if (PPM) {
      gx[k] = x[k] * kd(x[k], KL[k], KH[k]);
      g[k] = fma(x[k], gx[k], 1.0);
    } else {
      gx[k] = 1.0 / 3.0;
      g[k] = x[k] + 1.0;
    }
  }
  const double rs = rcp_w(fma(10.0, g[1], fma(5.0, g[2], g[0])));
  const double N = g[0] * p[0] + g[1] * p[1] + g[2] * p[2];
  const double Nb = 0.125 * rs;
  const double out = Nb * N;
  const double Sb = -(out * rs);
  double pb[3], z[3], T = 0.0;  // z = adjoint of x / 3
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    pb[k] = Nb * g[k];
    z[k] = fma(c[k], Sb, Nb * p[k]) * gx[k];
    T = fma(x[k] + 1.0, z[k], T);
  }
  // x_k = 16 P_k / S_P - 1, then P_k of the D and D_k = E_k^2
  const double q = 3.0 * r, q16 = 16.0 * q, SPb = -(q * T);
  double Pb[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) Pb[k] = fma(q16, z[k], c[k] * SPb);
  const double Db[3] = {fma(Pb[1], D[2], Pb[2] * D[1]), fma(Pb[0], D[2], Pb[2] * D[0]),
                        fma(Pb[0], D[1], Pb[1] * D[0])};
  double tb[3], sb[3];  // by t, and by s = 2 u (a - 4 b, b - d, e - 4 d)
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const double f = E[k] * Db[k];
    tb[k] = (13.0 / 3.0 * f) * t[k];
    sb[k] = (2.0 * f) * u[k];
  }
  const double p01 = pb[0] + pb[1], p12 = pb[1] + pb[2];
  v[0] = fma(3.0, pb[0], tb[0] + sb[0]);
  v[1] = fma(-10.0, p01, fma(-2.0, tb[0], fma(-4.0, sb[0], tb[1] + sb[1])));
  v[2] = fma(30.0, p12, fma(-2.0, tb[2], fma(-4.0, sb[2], tb[1] - sb[1])));
  v[3] = fma(-5.0, pb[2], tb[2] + sb[2]);
  return out;
}

// WENO r = 2 (inputs a, b, d around the zero centre) -- see weno3: p = (-b, d),
// P = (D_1, D_0), x_k = 4 P_k r - 1, g_k = 1 + K_k x_k^2 (in units of C_k), S =
// g_0 + 3 g_1, out = (3 g_1 d - g_0 b) / (2 S).
template <bool PPM> WIU_DEV double weno3_grad(double v[3], double eps) {
  const double a = v[0], b = v[1], d = v[2];
  const double KL[2] = {WIU_M2L0 * 0.25, WIU_M2L1 * 0.75};
  const double KH[2] = {WIU_M2H0 * 0.25, WIU_M2H1 * 0.75};
  const double t[2] = {fma(-2.0, b, a), b + d}, u[2] = {fma(-0.5, a, t[0]), fma(0.5, t[1], -d)};
  double E[2], D[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    E[k] = fma(13.0 / 12.0, t[k] * t[k], fma(u[k], u[k], eps));
    D[k] = E[k] * E[k];
  }
  const double r = rcp_w(fma(3.0, D[0], D[1])), r4 = 4.0 * r;
  double x[2], g[2], gx[2];  // gx = dg/dx / 2
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    x[k] = fma(D[1 - k], r4, -1.0);
    if (PPM) {
      gx[k] = kd(x[k], KL[k], KH[k]);
      g[k] = fma(x[k], gx[k], 1.0);
    } else {
      gx[k] = 0.5;
      g[k] = x[k] + 1.0;
    }
  }
  const double g1 = 3.0 * g[1];
  const double rs = rcp_w(g[0] + g1);
  const double Nb = 0.5 * rs;
  const double out = Nb * (g1 * d - g[0] * b);
  const double Sb = -(out * rs);
  const double z0 = (Sb - Nb * b) * gx[0], z1 = 3.0 * ((Nb * d + Sb) * gx[1]);
  const double T = fma(x[0], z0, z0) + fma(x[1], z1, z1);
  const double q = 2.0 * r, q4 = 4.0 * q, SPb = -(q * T);
  // P_0 = D_1, P_1 = D_0 with weights 1 and 3 in S_P; dD = 2 E dE; s = 2 u
  const double f1 = E[1] * fma(q4, z0, SPb), f0 = E[0] * fma(q4, z1, 3.0 * SPb);
  const double tb0 = (13.0 / 3.0 * f0) * t[0], sb0 = (2.0 * f0) * u[0];
  const double tb1 = (13.0 / 3.0 * f1) * t[1], sb1 = (2.0 * f1) * u[1];
  v[0] = tb0 + sb0;
  v[1] = fma(-2.0, tb0, fma(-4.0, sb0, tb1 + sb1)) - Nb * g[0];
  v[2] = (tb1 - sb1) + Nb * g1;
  return out;
}

// Orders two independent computations: what follows from b starts when a is done,
// so that the four fields' reverses are not interleaved (their temporaries at once
// are more than the register file holds).
template <int N> WIU_DEV void one_after(double* a, double* b) {
#pragma unroll
  for (int j = 0; j < N; ++j) asm volatile("" : "+v"(a[j]), "+v"(b[j]));
}

// ---------------------------------------------------------------------------
// Reverse of side_flux for one side: given Fb = adjoint of F^{+-}_{k+1/2},
// accumulate the adjoints of the states k-2 .. k+3 and of the line
// eigenvalue.  The states are read through q(m, c) and the adjoints added
// through qb(m, c, value), so both can live in LDS.  The sixteen characteristic
// values are projected once; each field's interpolation replaces its own by the
// derivatives that the reverse needs.
// ---------------------------------------------------------------------------
template <bool FIFTH, bool PPM, class QF, class QBF>
WIU_DEV void side_flux_vjp(QF q, int side, double nx_, double ny_, double mx, double my, double lam, double gam,
                           double eps, const double Fb[4], QBF qb, double& lamb) {
  const int mr = 2 + side;
  const double Qr[4] = {q(mr, 0), q(mr, 1), q(mr, 2), q(mr, 3)};
  const double gm1 = gam - 1.0;
  // ---- forward recompute
  const double rr = rcp(Qr[0]);
  const double u = Qr[1] * rr, v = Qr[2] * rr;
  const double q2 = u * u + v * v;
  const double p = gm1 * (Qr[3] - 0.5 * Qr[0] * q2);
  const double c2 = gam * p * rr;
  const double rc = rsqrt_(c2);
  const double c = c2 * rc;
  const double H = (Qr[3] + p) * rr;
  const double qn = u * nx_ + v * ny_;
  const double qt = v * nx_ - u * ny_;
  const double b1 = gm1 * (rc * rc);
  const double b2 = 0.5 * b1 * q2;
  const double b1h = 0.5 * b1, b2h = 0.5 * b2, rch = 0.5 * rc;
  // stencil entry j = 0..NV-1 <-> state m (left-biased order for side 0,
  // mirrored for 1); the reference node, between entries 1 and 2, has none
  constexpr int NV = FIFTH ? 4 : 3;
  auto mof = [&](int j) { const int s_ = j < 2 ? j : j + 1; return side == 0 ? s_ : 5 - s_; };
  double w[4][NV];
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int m = mof(j);
    const double dr = q(m, 0) - Qr[0], dm = q(m, 1) - Qr[1], dn = q(m, 2) - Qr[2], de = q(m, 3) - Qr[3];
    const double A = b2h * dr - b1h * (u * dm + v * dn - de);  // halves of A and B
    const double B = rch * (qn * dr - nx_ * dm - ny_ * dn);
    w[0][j] = A + B;
    w[1][j] = fma(-2.0, A, dr);
    w[2][j] = nx_ * dn - ny_ * dm - qt * dr;
    w[3][j] = A - B;
  }
  // WENO per characteristic component, one after the other: its value, and in
  // place of its inputs their derivatives (an adjoint is linear in Wb, so one
  // evaluation serves both passes)
  double W[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    if (k) one_after<NV>(w[k - 1], w[k]);
    if constexpr (FIFTH) W[k] = weno5_grad<PPM>(w[k], eps);
    else W[k] = weno3_grad<PPM>(w[k], eps);
  }
  const double s03 = W[0] + W[3], d30 = W[3] - W[0];
  const double sum = s03 + W[1];
  const double r0 = Qr[0] + sum;
  const double r1 = Qr[1] + (u * sum + c * nx_ * d30 - ny_ * W[2]);
  const double r2 = Qr[2] + (v * sum + c * ny_ * d30 + nx_ * W[2]);
  const double r3 = Qr[3] + (H * s03 + c * qn * d30 + 0.5 * q2 * W[1] + qt * W[2]);
  const double ri = rcp(r0);
  const double ul = r1 * ri, vl = r2 * ri;
  const double pl = gm1 * (r3 - 0.5 * (r1 * ul + r2 * vl));
  const double Ul = mx * ul + my * vl;
  const double sl = side == 0 ? lam : -lam;
  // ---- reverse: F = (r Ul + (0, mx pl, my pl, pl Ul) + sl r) / 2
  double r0b = 0.5 * Fb[0] * (Ul + sl);
  double r1b = 0.5 * Fb[1] * (Ul + sl);
  double r2b = 0.5 * Fb[2] * (Ul + sl);
  double r3b = 0.5 * Fb[3] * (Ul + sl);
  const double Ulb = 0.5 * (Fb[0] * r0 + Fb[1] * r1 + Fb[2] * r2 + Fb[3] * (r3 + pl));
  const double plb = 0.5 * (Fb[1] * mx + Fb[2] * my + Fb[3] * Ul);
  const double slb = 0.5 * (Fb[0] * r0 + Fb[1] * r1 + Fb[2] * r2 + Fb[3] * r3);
  lamb += side == 0 ? slb : -slb;
  double ulb = Ulb * mx, vlb = Ulb * my;
  r3b += gm1 * plb;
  r1b -= 0.5 * gm1 * plb * ul;
  ulb -= 0.5 * gm1 * plb * r1;
  r2b -= 0.5 * gm1 * plb * vl;
  vlb -= 0.5 * gm1 * plb * r2;
  r1b += ulb * ri;
  r2b += vlb * ri;
  r0b -= (ulb * r1 + vlb * r2) * ri * ri;
  // r = Qr + R W
  double Qrb[4] = {r0b, r1b, r2b, r3b};
  const double sumb = r0b + u * r1b + v * r2b;
  double ub = r1b * sum, vb = r2b * sum;
  const double d30b = c * (nx_ * r1b + ny_ * r2b + qn * r3b);
  const double cb = d30 * (nx_ * r1b + ny_ * r2b + qn * r3b);
  const double Wb2 = -ny_ * r1b + nx_ * r2b + qt * r3b;
  const double s03b = H * r3b + sumb;
  const double Hb = s03 * r3b;
  double qnb = c * d30 * r3b;
  double q2b = 0.5 * W[1] * r3b;
  const double Wb1 = 0.5 * q2 * r3b + sumb;
  double qtb = W[2] * r3b;
  const double Wb[4] = {s03b - d30b, Wb1, Wb2, s03b + d30b};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
#pragma unroll
    for (int j = 0; j < NV; ++j) w[k][j] *= Wb[k];
  }
  // projection of the deviations: per slot, adjoints of A, B and of the
  // deviation itself, then onto the slot's state and the reference state
  // (A = b2 dr - b1 (u dm + v dn - de), B = rc (qn dr - nx dm - ny dn)); the
  // coefficients' adjoints need only the sums of Ab, Bb and Wb_2 over the
  // deviations
  double Ar = 0.0, Am = 0.0, An = 0.0, Ae = 0.0, Br = 0.0, Bm = 0.0, Bn = 0.0, Tr = 0.0;
  const double rcq = rc * qn;
#pragma unroll
  for (int s_ = 0; s_ < NV; ++s_) {
    const int m = mof(s_);
    const double dr = q(m, 0) - Qr[0], dm = q(m, 1) - Qr[1], dn = q(m, 2) - Qr[2], de = q(m, 3) - Qr[3];
    const double Ab = fma(0.5, w[0][s_] + w[3][s_], -w[1][s_]);
    const double Bb = 0.5 * (w[0][s_] - w[3][s_]);
    const double Tb = w[2][s_];
    Ar = fma(Ab, dr, Ar);
    Am = fma(Ab, dm, Am);
    An = fma(Ab, dn, An);
    Ae = fma(Ab, de, Ae);
    Br = fma(Bb, dr, Br);
    Bm = fma(Bb, dm, Bm);
    Bn = fma(Bb, dn, Bn);
    Tr = fma(Tb, dr, Tr);
    const double deb = b1 * Ab, Bc = rc * Bb;
    const double drb = fma(rcq, Bb, fma(b2, Ab, fma(-qt, Tb, w[1][s_])));
    const double dmb = -fma(nx_, Bc, fma(u, deb, ny_ * Tb));
    const double dnb = fma(nx_, Tb, -fma(ny_, Bc, v * deb));
    // deviation = q[m] - Qr
    qb(m, 0, drb); qb(m, 1, dmb); qb(m, 2, dnb); qb(m, 3, deb);
    Qrb[0] -= drb; Qrb[1] -= dmb; Qrb[2] -= dnb; Qrb[3] -= deb;
  }
  const double b2b = Ar;
  double b1b = Ae - fma(u, Am, v * An);
  double rcb = fma(qn, Br, -fma(nx_, Bm, ny_ * Bn));
  ub = fma(-b1, Am, ub);
  vb = fma(-b1, An, vb);
  qnb = fma(rc, Br, qnb);
  qtb -= Tr;
  // reference state
  b1b += 0.5 * q2 * b2b;
  q2b += 0.5 * b1 * b2b;
  rcb += 2.0 * gm1 * rc * b1b;
  vb += nx_ * qtb;
  ub -= ny_ * qtb;
  ub += nx_ * qnb;
  vb += ny_ * qnb;
  Qrb[3] += Hb * rr;
  double pb = Hb * rr;
  double rrb = Hb * (Qr[3] + p);
  double c2b = cb * rc;
  rcb += cb * c2;
  c2b -= 0.5 * rcb * rc * rc * rc;
  pb += c2b * gam * rr;
  rrb += c2b * gam * p;
  Qrb[3] += gm1 * pb;
  Qrb[0] -= 0.5 * gm1 * q2 * pb;
  q2b -= 0.5 * gm1 * Qr[0] * pb;
  ub += 2.0 * u * q2b;
  vb += 2.0 * v * q2b;
  Qrb[1] += ub * rr;
  rrb += ub * Qr[1];
  Qrb[2] += vb * rr;
  rrb += vb * Qr[2];
  Qrb[0] -= rrb * rr * rr;
#pragma unroll
  for (int cc = 0; cc < 4; ++cc) qb(mr, cc, Qrb[cc]);
}

// Reverse of nodal_split: fpb, fmb = adjoints of f^+-; accumulates Qb, lamb.
WIU_DEV void nodal_split_vjp(const double Q[4], double kx, double ky, double lam, double gam, const double fpb[4],
                             const double fmb[4], double Qb[4], double& lamb) {
  const double gm1 = gam - 1.0;
  const double ri = rcp(Q[0]);
  const double u = Q[1] * ri, v = Q[2] * ri;
  const double p = gm1 * (Q[3] - 0.5 * (Q[1] * u + Q[2] * v));
  const double U = kx * u + ky * v;
  double Eb[4], db[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    Eb[c] = 0.5 * (fpb[c] + fmb[c]);
    db[c] = 0.5 * (fpb[c] - fmb[c]);
    Qb[c] += lam * db[c];
    lamb += Q[c] * db[c];
  }
  // E = (rho U, m U + kx p, n U + ky p, (e + p) U)
  const double Ub = Eb[0] * Q[0] + Eb[1] * Q[1] + Eb[2] * Q[2] + Eb[3] * (Q[3] + p);
  const double pb = Eb[1] * kx + Eb[2] * ky + Eb[3] * U;
  Qb[0] += Eb[0] * U;
  Qb[1] += Eb[1] * U;
  Qb[2] += Eb[2] * U;
  Qb[3] += Eb[3] * U;
  double ub = Ub * kx, vb = Ub * ky;
  // p = gm1 (e - (m u + n v)/2)
  Qb[3] += gm1 * pb;
  Qb[1] -= 0.5 * gm1 * pb * u;
  ub -= 0.5 * gm1 * pb * Q[1];
  Qb[2] -= 0.5 * gm1 * pb * v;
  vb -= 0.5 * gm1 * pb * Q[2];
  Qb[1] += ub * ri;
  Qb[2] += vb * ri;
  const double rib = ub * Q[1] + vb * Q[2];
  Qb[0] -= rib * ri * ri;
}

// Reverse of the wave speed |k . u| + sqrt(c^2 |k|^2) (c^2 = gam p / rho).
WIU_DEV void wave_speed_vjp(const double Q[4], double kx, double ky, double gam, double sb, double Qb[4]) {
  const double gm1 = gam - 1.0;
  const double ri = 1.0 / Q[0];
  const double u = Q[1] * ri, v = Q[2] * ri;
  const double p = gm1 * (Q[3] - 0.5 * (Q[1] * u + Q[2] * v));
  const double U = kx * u + ky * v;
  const double K2 = kx * kx + ky * ky;
  const double sc = sqrt(gam * p * ri * K2);
  const double sgn = U > 0.0 ? 1.0 : (U < 0.0 ? -1.0 : 0.0);
  const double Ub = sb * sgn;
  // c^2 = gam p ri, d sqrt(c^2 K2) / d c^2 = K2 / (2 sqrt(c^2 K2))
  const double c2b = sb * K2 / (2.0 * sc);
  const double pb = c2b * gam * ri;
  double rib = c2b * gam * p;
  double ub = Ub * kx, vb = Ub * ky;
  Qb[3] += gm1 * pb;
  Qb[1] -= 0.5 * gm1 * pb * u;
  ub -= 0.5 * gm1 * pb * Q[1];
  Qb[2] -= 0.5 * gm1 * pb * v;
  vb -= 0.5 * gm1 * pb * Q[2];
  Qb[1] += ub * ri;
  Qb[2] += vb * ri;
  rib += ub * Q[1] + vb * Q[2];
  Qb[0] -= rib * ri * ri;
}

// Adjoint of the flux combination: coefficients of H_{i+1/2} on the split
// fluxes (Eqs. 3.4, 3.8, 3.16, 3.20 and their mirror images).  H(i) =
//   sum_m NP[m] f+(i+m) + MP[m] F+(i+m) + NM[m] f-(i+m) + MM[m] F-(i+m),
// m = -2 .. 3 (index m + 2); F(k) is the value at k + 1/2.
template <int SC> struct HCoef;
template <> struct HCoef<0> {
  static constexpr double NP[6] = {0, -1.0 / 24, 2.0 / 24, -1.0 / 24, 0, 0};
  static constexpr double MP[6] = {0, 0, 1.0, 0, 0, 0};
  static constexpr double NM[6] = {0, 0, -1.0 / 24, 2.0 / 24, -1.0 / 24, 0};
  static constexpr double MM[6] = {0, 0, 1.0, 0, 0, 0};
};
template <> struct HCoef<1> {
  static constexpr double NP[6] = {0, 0, 2.0 / 6, 0, 0, 0};
  static constexpr double MP[6] = {0, -1.0 / 6, 5.0 / 6, 0, 0, 0};
  static constexpr double NM[6] = {0, 0, 0, 2.0 / 6, 0, 0};
  static constexpr double MM[6] = {0, 0, 5.0 / 6, -1.0 / 6, 0, 0};
};
template <> struct HCoef<2> {
  static constexpr double NP[6] = {19.0 / 1920, -116.0 / 1920, 154.0 / 1920, -36.0 / 1920, -21.0 / 1920, 0};
  static constexpr double MP[6] = {0, 0, 1.0, 0, 0, 0};
  static constexpr double NM[6] = {0, -21.0 / 1920, -36.0 / 1920, 154.0 / 1920, -116.0 / 1920, 19.0 / 1920};
  static constexpr double MM[6] = {0, 0, 1.0, 0, 0, 0};
};
template <> struct HCoef<3> {
  static constexpr double NP[6] = {0, 1.0 / 30, 1.0 / 30, -4.0 / 30, 0, 0};
  static constexpr double MP[6] = {0, -4.0 / 30, 36.0 / 30, 0, 0, 0};
  static constexpr double NM[6] = {0, 0, -4.0 / 30, 1.0 / 30, 1.0 / 30, 0};
  static constexpr double MM[6] = {0, 0, 36.0 / 30, -4.0 / 30, 0, 0};
};

}  // namespace wiu
