// One RK stage (or residual) of a small tile of nodes, both directions at once.
//
// The sweeps of wiu_sweep.hpp take one direction a launch and one item a lane:
// on grids that do not fill the chip each launch costs its slowest wave, and a
// lane computes both side fluxes of its midpoint one after the other.  Here a
// workgroup owns TX x TY output nodes, stages their states with the halo of
// both directions, and gives every side flux F^+ or F^- of every midpoint of
// either direction to a lane of its own, so a stage is one launch and a lane's
// work is half as long.  The price is recomputed halo work (5-2MP, 8 x 8: 5.5
// side fluxes a node where the method has 4; the sweeps compute 4.35), which is
// why larger grids keep the sweeps (use_stage_tiles).
#pragma once

#include "wiu_sweep.hpp"

namespace wiu {

template <int SC, int TX, int TY, bool OPT> struct StageLds {
  using T = Traits<SC>;
  static constexpr int QL = Range<SC>::QL;
  // states -SLO .. out - 1 + SHI along either direction
  static constexpr int SLO = QL - T::MLO > -T::NLO ? QL - T::MLO : -T::NLO;
  static constexpr int SHI = T::MHI + QL + 1 > T::NHI ? T::MHI + QL + 1 : T::NHI;
  static constexpr int BW = TX + SLO + SHI, BH = TY + SLO + SHI;
  // per line: nodes with a flux, midpoints with side fluxes, midpoints with an H
  static constexpr int NDX = TX + T::NHI - T::NLO, NDY = TY + T::NHI - T::NLO;
  static constexpr int MDX = TX + T::MHI - T::MLO, MDY = TY + T::MHI - T::MLO;
  static constexpr int ND = NDX * TY + TX * NDY;  // xi items first, then eta items
  static constexpr int MD = MDX * TY + TX * MDY;
  static constexpr int HD = (TX + 1) * TY + TX * (TY + 1);
  double sq[4][BH * BW];
  double e[4][ND];
  double f[2][4][MD];
  double d[OPT ? 2 : 1][OPT ? 4 : 1][OPT ? MD : 1];  // another midpoint split's difference
  double h[4][HD];
  double lam[TX + TY];               // eigenvalues of the tile's eta lines, then of its xi lines
  // operands of the output nodes: J^{-1}, U0 (4), nodal metrics (4)
  static constexpr int NOP = 9;
  double op[NOP][TX * TY];
  unsigned long long red[16];
};

// State at node (i, j) of the grid or beyond one of its sides (rules as in
// sweep_tile; a single grid has no interfaces): out of range in at most one direction.
WIU_DEV void stage_state(const SweepArgs& s, int i, int j, double Q[4]) {
  const Dims& d = s.d;
  const bool ox = i < 0 || i >= d.nx, oy = j < 0 || j >= d.ny;
  if (ox || oy) {
    const int k = ox ? i : j, n = ox ? d.nx : d.ny, bc = ox ? d.bcx : d.bcy;
    const int sd = (ox ? 0 : 2) + (k < 0 ? 0 : 1);
    const int rule = bc != 0 ? s.side[sd] : 0;
    if (rule == 2) {
#pragma unroll
      for (int c = 0; c < 4; ++c) Q[c] = s.fixed[sd][c];
      return;
    }
    const int kb = k < 0 ? 0 : n - 1;
    const int kk = rule == 1 ? min(max(2 * kb - k, 0), n - 1) : bc_index(k, n, bc);
    const long long o = ox ? (long long)j * d.nx + kk : (long long)kk * d.nx + i;
#pragma unroll
    for (int c = 0; c < 4; ++c) Q[c] = s.U[c * d.np + o];
    if (rule == 1) {
      const double* Mk = s.M + (ox ? 0 : 2) * d.mplane;
      const long long mb = (long long)((ox ? j : kb) + GHOST) * d.mpitch + ((ox ? kb : i) + GHOST);
      const double bx = Mk[mb], by = Mk[d.mplane + mb];
      const double rn = rsqrt_(bx * bx + by * by);
      const double nbx = bx * rn, nby = by * rn;
      const double mn = Q[1] * nbx + Q[2] * nby;
      Q[1] -= 2.0 * mn * nbx;
      Q[2] -= 2.0 * mn * nby;
    }
    return;
  }
  const long long o = (long long)j * d.nx + i;
#pragma unroll
  for (int c = 0; c < 4; ++c) Q[c] = s.U[c * d.np + o];
}

// Tile (bx, by); a block of NT threads, all of which call it, once.  Workgroup 0 writes
// the step size; clearing is shared by workgroup `wg` of `nwg`.
template <int SC, int TX, int TY, int NT, bool OPT, bool PPM>
WIU_DEV void stage_tile(const StageArgs& a, int bx, int by, int wg, int nwg, StageLds<SC, TX, TY, OPT>& L) {
  using T = Traits<SC>;
  using LT = StageLds<SC, TX, TY, OPT>;
  constexpr int SLO = LT::SLO, BW = LT::BW, BH = LT::BH, MDX = LT::MDX, NDX = LT::NDX;
  constexpr int MX = MDX * TY, NX = NDX * TY, HX = (TX + 1) * TY;  // xi items of each kind
  const SweepArgs& s = a.s;
  const Dims& d = s.d;
  const int tid = threadIdx.x;
  const int i0 = bx * TX, j0 = by * TY;
  const int ow = min(TX, d.nx - i0), oh = min(TY, d.ny - j0);
  const double ah = OPT ? s.ah : 1.0;
  const bool alt = OPT && s.split != 0;
  const int ppm = OPT ? (s.weights != 0 ? 2 : s.ppm) : PPM;
  const double gam = s.gamma;

  // Task t < 2 MD is a side flux (midpoint t % MD, side t / MD), then come the
  // ND nodal fluxes.  Its direction, line and position k along it, and whether
  // it is needed; the metrics of its node or midpoint.
  struct Task {
    bool act, mid, eta;
    int side, line, k, item;
    double kx0, ky0, kx1, ky1, mx, my;
  };
  auto task = [&](int t) {
    Task q;
    q.mid = t < 2 * LT::MD;
    q.side = q.mid && t >= LT::MD;
    q.item = q.mid ? t - q.side * LT::MD : t - 2 * LT::MD;
    const int nx = q.mid ? MX : NX, w = q.mid ? MDX : NDX, lo = q.mid ? T::MLO : T::NLO;
    q.eta = q.item >= nx;
    const int r = q.eta ? q.item - nx : q.item;
    // xi: positions along a row first; eta: columns first
    q.line = q.eta ? r % TX : r / w;
    q.k = (q.eta ? r / TX : r % w) + lo;
    const int out = q.eta ? oh : ow, hi = q.mid ? T::MHI : T::NHI;
    q.act = t < 2 * LT::MD + LT::ND && q.line < (q.eta ? ow : oh) && q.k < out + hi;
    if (q.act) {
      const int gi = i0 + (q.eta ? q.line : q.k), gj = j0 + (q.eta ? q.k : q.line);
      const long long mo = (long long)(gj + GHOST) * d.mpitch + (gi + GHOST);
      const long long st = q.eta ? d.mpitch : 1;
      const double* Mk = s.M + (q.eta ? 2 : 0) * d.mplane + mo;
      q.kx0 = Mk[0]; q.ky0 = Mk[d.mplane];
      if (q.mid) {
        const double* Mm = s.M + (q.eta ? 7 : 5) * d.mplane + mo;
        q.kx1 = Mk[st]; q.ky1 = Mk[d.mplane + st];
        q.mx = Mm[0]; q.my = Mm[d.mplane];
      }
    }
    return q;
  };

  constexpr int NTASK = 2 * LT::MD + LT::ND;
  constexpr int NR = (NTASK + NT - 1) / NT;
  static_assert(NR <= 4, "rounds of tasks");
  const bool next = s.mode == 2 && s.nlam_xi;

  // Everything the tile reads from global memory is loaded here, in one
  // latency: the metrics of this lane's tasks, states, line eigenvalues,
  // operands of the output nodes, the step size.
  Task tasks[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) tasks[r] = task(tid + r * NT);
  double dt = s.mode == 2 && !a.cflw ? s.dt[0] : 0.0;
  const double* tag = s.M + 9 * d.mplane;
  const bool other = tag[0] != TAG_MAGIC || tag[1] != (double)SC || tag[2] != (double)d.nx ||
                     tag[3] != (double)d.ny || tag[6] != ah;

  // states: the tile's rows with their xi halo, then the eta halo of its columns
  constexpr int NSX = BW * TY, NS = NSX + TX * (BH - TY);
  constexpr int NSR = (NS + NT - 1) / NT;
  double qv[NSR][4];
  bool qa[NSR];
#pragma unroll
  for (int r_ = 0; r_ < NSR; ++r_) {
    const int e = r_ * NT + tid;
    qa[r_] = false;
    if (e < NS) {
      const bool row = e < NSX;
      const int r = e - NSX;
      const int x = row ? e % BW : r % TX + SLO;
      int y = row ? e / BW + SLO : r / TX;
      if (!row && y >= SLO) y += TY;
      const int i = i0 + x - SLO, j = j0 + y - SLO;
      // the tile's rows and columns up to its own halo (a ragged tile's is
      // nearer): out of the grid in one direction at most
      const bool in_row = j >= j0 && j < j0 + oh, in_col = i >= i0 && i < i0 + ow;
      qa[r_] = (in_row && i < i0 + ow + LT::SHI) || (in_col && j < j0 + oh + LT::SHI);
      if (qa[r_]) stage_state(s, i, j, qv[r_]);
    }
  }
  // the lanes that stage no state (if there are enough) take the rest; the
  // last lanes come first
  constexpr int NO = TX * TY;
#pragma unroll
  for (int e0 = 0; e0 < NO; e0 += NT) {
    const int e = e0 + NT - 1 - tid;
    const int ti = e % TX, tj = e / TX;
    if (e < NO && ti < ow && tj < oh) {
      const long long mo = (long long)(j0 + tj + GHOST) * d.mpitch + (i0 + ti + GHOST);
      const long long o = (long long)(j0 + tj) * d.nx + (i0 + ti);
      double v[LT::NOP];
      v[0] = s.M[4 * d.mplane + mo];
      const bool base = s.mode == 2 && s.ca != 0.0;
#pragma unroll
      for (int c = 0; c < 4; ++c) v[1 + c] = base ? s.U0[c * d.np + o] : 0.0;
#pragma unroll
      for (int c = 0; c < 4; ++c) v[5 + c] = next ? s.M[c * d.mplane + mo] : 0.0;
#pragma unroll
      for (int c = 0; c < LT::NOP; ++c) L.op[c][e] = v[c];
    }
  }
  if (tid >= NT - 64 * ((TX + TY + 63) / 64)) {
    const int e = NT - 1 - tid;
    const bool eta = e < TX;
    const int ln = eta ? i0 + e : j0 + e - TX;
    if (e < TX + TY && ln < (eta ? d.nx : d.ny))
      L.lam[e] = s.alpha * __longlong_as_double((long long)(eta ? s.lam_eta : s.lam_xi)[ln]);
  }
#pragma unroll
  for (int r_ = 0; r_ < NSR; ++r_) {
    const int e = r_ * NT + tid;
    if (qa[r_]) {
      const bool row = e < NSX;
      const int r = e - NSX;
      const int x = row ? e % BW : r % TX + SLO;
      int y = row ? e / BW + SLO : r / TX;
      if (!row && y >= SLO) y += TY;
#pragma unroll
      for (int c = 0; c < 4; ++c) L.sq[c][y * BW + x] = qv[r_][c];
    }
  }
  // step size from the CFL maxima
  if (a.cflw) {
    unsigned long long m = 0;
    for (int k = tid; k < a.ncflw; k += NT) m = max(m, a.cflw[k]);
    for (int off = 32; off > 0; off >>= 1) m = max(m, (unsigned long long)__shfl_xor(m, off, 64));
    if ((tid & 63) == 0) L.red[tid >> 6] = m;
  }
  if (a.clear)
    for (long long k = (long long)wg * NT + tid; k < a.nclear; k += (long long)nwg * NT) a.clear[k] = 0ull;
  __syncthreads();
  auto step_size = [&]() {
    unsigned long long m = L.red[0];
#pragma unroll
    for (int k = 1; k < NT / 64; ++k) m = max(m, L.red[k]);
    return a.cfl / __longlong_as_double((long long)m);
  };
  if (a.cflw && wg == 0 && tid == 0) a.dt_out[0] = step_size();
  if (other) {  // metrics built for another scheme or grid: flag and do nothing (block-uniform)
    if (tid == 0) atomicOr(s.status, ST_SCHEME);
    return;
  }

  // side fluxes and nodal fluxes.  F^- is F^+ of the mirrored stencil with the
  // eigenvalue's sign reversed, so both sides run the same code: reference
  // node `ref`, one step along the stencil `st` slots (negative for F^-).
#pragma unroll
  for (int rd = 0; rd < NR; ++rd) {
    const Task& q = tasks[rd];
    if (q.act) {
      const int c0 = q.eta ? (q.k + SLO) * BW + q.line + SLO : (q.line + SLO) * BW + q.k + SLO;
      const int S = q.eta ? BW : 1;
      // rounds past the side fluxes carry no code for them
      if (rd * NT < 2 * LT::MD && q.mid) {
        const int ref = q.side ? c0 + S : c0, st = q.side ? -S : S;
        const double lq = L.lam[q.eta ? q.line : TX + q.line], lam = q.side ? -lq : lq;
        const double nbx = 0.5 * (q.kx0 + q.kx1), nby = 0.5 * (q.ky0 + q.ky1);
        const double rn = rsqrt_(nbx * nbx + nby * nby);
        const double nx_ = nbx * rn, ny_ = nby * rn;
        double F[4], D[4] = {0.0, 0.0, 0.0, 0.0};
        const int split = alt ? s.split : 0;
        auto w = [&](int m, int c) { return L.sq[c][ref + (m - LT::QL) * st]; };
        if (OPT && s.vars != 0)
          side_flux_comp<T::R, OPT>(w, 0, s.vars, q.mx, q.my, lam, gam, s.eps, ppm, F, split, D, q.side);
        else if constexpr (T::R == 4)
          side_flux7<OPT>(w, 0, nx_, ny_, q.mx, q.my, lam, gam, s.eps, ppm, F, split, D, q.side);
        else
          side_flux<T::fifth, OPT>(w, 0, nx_, ny_, q.mx, q.my, lam, gam, s.eps, ppm, F, split, D, q.side);
#pragma unroll
        for (int c = 0; c < 4; ++c) L.f[q.side][c][q.item] = F[c];
        if constexpr (OPT) {
#pragma unroll
          for (int c = 0; c < 4; ++c) L.d[q.side][c][q.item] = D[c];
        }
      } else {
        const double Qk[4] = {L.sq[0][c0], L.sq[1][c0], L.sq[2][c0], L.sq[3][c0]};
        double E[4];
        nodal_flux(Qk, q.kx0, q.ky0, gam, E);
#pragma unroll
        for (int c = 0; c < 4; ++c) L.e[c][q.item] = E[c];
      }
    }
  }
  __syncthreads();

  // H of every midpoint of the tile's nodes
  for (int t = tid; t < LT::HD; t += NT) {
    const bool eta = t >= HX;
    const int r = eta ? t - HX : t;
    const int line = eta ? r % TX : r / (TX + 1);
    const int k = (eta ? r / TX : r % (TX + 1)) - 1;
    if (line < (eta ? ow : oh) && k < (eta ? oh : ow)) {
      // slots of node k, midpoint k + 1/2 and state k, and their strides
      const int en = eta ? NX + (k - T::NLO) * TX + line : line * NDX + k - T::NLO, se = eta ? TX : 1;
      const int fn = eta ? MX + (k - T::MLO) * TX + line : line * MDX + k - T::MLO, sf = se;
      const int qn = eta ? (k + SLO) * BW + line + SLO : (line + SLO) * BW + k + SLO, sqs = eta ? BW : 1;
      const double lam = L.lam[eta ? line : TX + line];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double* e = &L.e[c][en];
        const double* u = &L.sq[c][qn];
        const double* gp = &L.f[0][c][fn];
        const double* gm = &L.f[1][c][fn];
        double H;
        if constexpr (SC == 3) {
          H = hsum52(lam, [&](int m) { return e[m * se]; }, [&](int m) { return u[m * sqs]; },
                     [&](int m) { return gp[m * sf]; }, [&](int m) { return gm[m * sf]; });
        } else {
          auto fp = [&](int kk) { return 0.5 * (e[(kk - k) * se] + lam * u[(kk - k) * sqs]); };
          auto fm = [&](int kk) { return 0.5 * (e[(kk - k) * se] - lam * u[(kk - k) * sqs]); };
          auto Fp = [&](int kk) { return gp[(kk - k) * sf]; };
          auto Fm = [&](int kk) { return gm[(kk - k) * sf]; };
          H = hflux<SC>(k, ah, fp, fm, Fp, Fm);
        }
        if constexpr (OPT) {
          if (alt) H += L.d[0][c][fn] + L.d[1][c][fn];
        }
        L.h[c][t] = H;
      }
    }
  }
  __syncthreads();
  if (tid >= (TX * TY + 63) / 64 * 64) return;  // whole waves take part in the reductions below

  const int ti = tid % TX, tj = tid / TX;
  const bool act = tid < TX * TY && ti < ow && tj < oh;
  const int ii = i0 + ti, jj = j0 + tj;
  const long long o = (long long)jj * d.nx + ii;
  if (a.cflw) dt = step_size();
  double sx = 0.0, se = 0.0, cf = 0.0;
  bool bad = false;
  if (act) {
    const int hx = tj * (TX + 1) + ti + 1, hy = HX + (tj + 1) * TX + ti;
    const double jinv = L.op[0][tid], rj = -rcp(jinv);
    double Qn[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double Rx = L.h[c][hx] - L.h[c][hx - 1], Re = L.h[c][hy] - L.h[c][hy - TX];
      if (s.mode == 1) {
        Qn[c] = (Rx + Re) * rj;
      } else {
        const double us = L.sq[c][(tj + SLO) * BW + ti + SLO];
        const double un = s.cb * (us + dt * (Rx * rj));
        Qn[c] = (s.ca == 0.0 ? un : s.ca * L.op[1 + c][tid] + un) + s.cb * (dt * (Re * rj));
      }
      s.out[c * d.np + o] = Qn[c];
    }
    if (next) {
      const WaveState w = wave_state(Qn, gam);
      const double sxr = wave_speed_dir(w, L.op[5][tid], L.op[6][tid]);
      const double ser = wave_speed_dir(w, L.op[7][tid], L.op[8][tid]);
      bad = w.bad || !(sxr < 1.0e300) || !(ser < 1.0e300);
      sx = fmax(0.0, sxr);
      se = fmax(0.0, ser);
      if (s.ncfl) cf = fmax(0.0, (sx + ser) / jinv);
    }
  }
  if (!next) return;
  // line maxima of the new state, as fused_stage_out forms them: a wave holds
  // 64 / TX rows of the tile
  static_assert(64 % TX == 0, "a wave holds whole tile rows");
  if (bad) atomicOr(s.status, ST_NONPHYS);
  for (int off = 1; off < TX; off <<= 1) sx = fmax(sx, __shfl_xor(sx, off, 64));
  for (int off = TX; off < 64; off <<= 1) se = fmax(se, __shfl_xor(se, off, 64));
  const bool col = (tid & 63) < TX && ti < ow && tj < oh;
  if (ti == 0 && act) atomicMax(&s.nlam_xi[jj], (unsigned long long)__double_as_longlong(sx));
  if (col) atomicMax(&s.nlam_eta[ii], (unsigned long long)__double_as_longlong(se));
  if (s.ncfl) {
    for (int off = 1; off < 64; off <<= 1) cf = fmax(cf, __shfl_xor(cf, off, 64));
    if ((tid & 63) == 0) atomicMax(&s.ncfl[wg % min(d.nx, CFL_SLOTS)], (unsigned long long)__double_as_longlong(cf));
  }
}

}  // namespace wiu
