// The cell's collision with its rounding stated, for the ideal, Euler, Navier-Cauchy and
// 13-component models in the kernels that have to agree with one another, below
// (vlbm_physics.h defines the method and serves the rest).
//
// The populations of these models advance in kernels of several forms: in place, with and
// without the exchange between lanes, by rows and flat, injecting, and several steps in a
// pass (vlbm_rows.hip).  Left to fuse products and sums where it finds both in one basic
// block, the compiler rounds each form in its own way, and the split of a run into calls, a
// restart, or memory for the passes would show in the last bit.  Here contraction is on:
// a product and a sum fuse if and only if they stand in one expression, the left operand's
// product first, and a product with a name is rounded.  Every kernel then gives the same
// bits.  The expressions are those the compiler makes of vlbm_physics.h in the sweeps whose
// lanes exchange nothing.  It costs no time (FP32 190 x 113 x 77, 40 steps 4.82 -> 4.72 ms;
// 2D sweeps and tiles within 1 %; the nine-variable 64^2, bound by its launches, 2.13 -> 2.20
// us a step in FP32).
#pragma once

#include "vlbm_physics.h"

namespace vlbm {

// Where the rounding has to be stated: periodic lattices without a body (the others have one
// step of one form) of the models above (the 26-component model and the Guo and Chai sources
// have kernels of one form), in FP32; in FP64 where there are passes (2D) or an injecting
// sweep (the ideal model); and in the flat 16-bit sweeps (FLAT), which then give the bits of
// the injecting sweep that takes the same lattices by rows, so that a corrected run that
// corrects nothing is the plain run.  On rows that the workgroups tile, 16-bit storage keeps
// the rounding its kernels have always had.
template <int ST, int D, int MODEL, int SRC, bool FLAT>
inline constexpr bool kFixedRounding =
    MODEL != 1 && SRC == 0 && (ST == 1 || (ST == 0 ? D == 2 || MODEL == 0 : FLAT));

namespace fixed {

// Flux P[k][a] = Phi[k][a], not scaled, source S[k], div B estimate and total pressure:
// flux_source (vlbm_physics.h), which says what they are.
template <typename R, int D, int MODEL>
__device__ __forceinline__ void flux(const R* Q, const R* Jb, const Phys& ph, R (*P)[3], R* S, R& dlat, R& pt) {
#pragma clang fp contract(on)
#pragma unroll
  for (int k = 0; k < kNVars<MODEL>; ++k) S[k] = R(0);
  dlat = R(0);
  if constexpr (MODEL == 3) {
    (void)Jb;
    const R ir0 = R(ph.inv_rho0);
    const R v[3] = {Q[0] * ir0, Q[1] * ir0, Q[2] * ir0};
    const R lam = R(ph.lame_lambda), mu = R(ph.lame_mu);
    pt = R(0);
#pragma unroll
    for (int a = 0; a < D; ++a) {
#pragma unroll
      for (int b = 0; b < 3; ++b) P[b][a] = -Q[sigma_index(b, a)];
#pragma unroll
      for (int b = 0; b < 3; ++b)
#pragma unroll
        for (int c = b; c < 3; ++c) {
          if (b == c)
            P[sigma_index(b, c)][a] = a == b ? -(lam * v[a] + mu * (v[a] + v[a])) : -(lam * v[a] + R(0));
          else
            P[sigma_index(b, c)][a] = a == b ? -(R(0) + mu * v[c]) : (a == c ? -(R(0) + mu * v[b]) : -R(0));
        }
    }
  } else if constexpr (MODEL == 2) {
    (void)Jb;
    const R ir = R(1) / Q[0];
    const R m[3] = {Q[1], Q[2], Q[3]};
    const R E = Q[4];
    const R u[3] = {m[0] * ir, m[1] * ir, m[2] * ir};
    const R ein = E - R(0.5) * (m[0] * u[0] + m[1] * u[1] + m[2] * u[2]);  // internal energy
    const R pres = R(ph.gm1) * ein;
    const R Ep = E + R(ph.gm1) * ein;
    pt = pres;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      P[0][a] = m[a];
#pragma unroll
      for (int b = 0; b < 3; ++b) P[1 + b][a] = m[b] * u[a] + (a == b ? pres : R(0));
      P[4][a] = Ep * u[a];
    }
  } else if constexpr (MODEL == 4) {
    static_assert(D == 2, "the 13-component system is two-dimensional");
    const R ir = R(1) / Q[0];
    const R E = Q[3];
    const R u[2] = {Q[1] * ir, Q[2] * ir}, B[2] = {Q[4], Q[5]};
    const R uu = u[0] * Q[1] + u[1] * Q[2];  // rho |u|^2
    const R bb = B[0] * B[0] + B[1] * B[1];
    const R ub = u[0] * B[0] + u[1] * B[1];
    const R ein = E - R(0.5) * uu - R(0.5) * bb;  // internal energy
    const R hbb = R(0.5) * bb;
    pt = R(ph.gm1) * ein + hbb;
    const R Ept = E + pt;
    const R itm = R(ph.inv_tauM), ith = R(ph.inv_tauH), muv = R(ph.mu);
    const R dB[2][2] = {{Q[9] * itm, Q[10] * itm}, {Q[11] * itm, Q[12] * itm}};
    const R tv[2][2] = {{Q[6] * ith, Q[7] * ith}, {Q[7] * ith, Q[8] * ith}};
    const R j = Q[10] * itm - dB[1][0];
    R eta = R(ph.eta0);
    if (ph.inv_jc2 > 0.0) eta = eta * (R(1) + j * j * R(ph.inv_jc2));
    const R jxb[2] = {-j * B[1], j * B[0]};
    const R b01 = B[0] * B[1], e01 = u[0] * B[1];
    const R BB[2][2] = {{B[0] * B[0], b01}, {b01, B[1] * B[1]}};
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      P[0][c] = Q[1 + c];
      R utv = R(0);
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        P[1 + a][c] = Q[1 + a] * u[c] - BB[a][c] - Q[6 + a + c] * ith + (a == c ? pt : R(0));
        utv += u[a] * tv[a][c];
        const R own = u[a] * B[a];
        const R e = a == c ? own - own : (c == 1 ? u[1] * B[0] - e01 : e01 - B[0] * u[1]);
        P[4 + a][c] = e - eta * dB[c][a];
      }
      P[3][c] = Ept * u[c] - B[c] * ub - utv + eta * jxb[c];
      P[6][c] = Q[6] * u[c] - muv * (c == 0 ? R(2) * u[0] : R(0));  // xx
      P[7][c] = Q[7] * u[c] - muv * (c == 0 ? u[1] : u[0]);         // xy
      P[8][c] = Q[8] * u[c] - muv * (c == 1 ? R(2) * u[1] : R(0));  // yy
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) P[9 + 2 * a + b][c] = Q[9 + 2 * a + b] * u[c] - (a == c ? B[b] : R(0));
    }
    const R sh = R(-ph.dt_over_tauH), sg = R(-ph.dt_over_tauM);
#pragma unroll
    for (int q = 0; q < 3; ++q) S[6 + q] = Q[6 + q] * sh;
#pragma unroll
    for (int q = 0; q < 4; ++q) S[9 + q] = Q[9 + q] * sg;
    if (ph.divb_mode == 1)
      dlat = (dB[0][0] + dB[1][1]) * R(ph.divb_scale);
    else
      dlat = -(Jb[0] * R(ph.inv_tauB[0]) + Jb[1] * R(ph.inv_tauB[1])) * R(ph.inv_cs2);
    if (ph.powell) {
      const R cp = -R(ph.s) * dlat;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        S[1 + b] += cp * B[b];
        S[4 + b] += cp * u[b];
      }
      S[3] += cp * ub;
    }
  } else {
    static_assert(MODEL == 0, "ideal, Euler, Navier-Cauchy, 13 components");
    const R ir = R(1) / Q[0];
    const R m[3] = {Q[1], Q[2], Q[3]}, B[3] = {Q[5], Q[6], Q[7]};
    const R E = Q[4];
    const R u[3] = {m[0] * ir, m[1] * ir, m[2] * ir};
    const R mu = m[0] * u[0] + m[1] * u[1] + m[2] * u[2];  // rho |u|^2
    const R bb = B[0] * B[0] + B[1] * B[1] + B[2] * B[2];
    const R ub = u[0] * B[0] + u[1] * B[1] + u[2] * B[2];
    const R ein = E - R(0.5) * mu - R(0.5) * bb;  // internal energy
    const R hbb = R(0.5) * bb;
    pt = R(ph.gm1) * ein + hbb;
    const R Ept = E + pt;
    const R b01 = B[0] * B[1], b02 = B[0] * B[2], b12 = B[1] * B[2];
    const R BB[3][3] = {{B[0] * B[0], b01, b02}, {b01, B[1] * B[1], b12}, {b02, b12, B[2] * B[2]}};
#pragma unroll
    for (int a = 0; a < D; ++a) {
      P[0][a] = m[a];
#pragma unroll
      for (int b = 0; b < 3; ++b) P[1 + b][a] = m[b] * u[a] - BB[a][b] + (a == b ? pt : R(0));
      P[4][a] = Ept * u[a] - B[a] * ub;
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        if (b >= D) {
          P[5 + b][a] = u[a] * B[b] - B[a] * u[b];
        } else {
          // the flux of B_b along a is exactly minus that of B_a along b: of the products they
          // share, u_lower B_upper is the one rounded before the difference
          const R e = u[a < b ? a : b] * B[a < b ? b : a];
          P[5 + b][a] = a == b ? e - e : (a > b ? u[a] * B[b] - e : e - B[a] * u[b]);
        }
      }
    }
    R acc = R(0);
#pragma unroll
    for (int a = 0; a < D; ++a) acc += Jb[a] * R(ph.inv_tauB[a]);
    dlat = -acc * R(ph.inv_cs2);
    if (ph.powell) {
      const R cp = -R(ph.s) * dlat;
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        S[1 + b] += cp * B[b];
        S[5 + b] += cp * u[b];
      }
      S[4] += cp * ub;
    }
  }
}

// vlbm::collide with the direct source
template <typename R, int D, int MODEL, int COLL, typename Tgt>
__device__ __forceinline__ void collide(R (*f)[2 * D + 1], const Phys& ph, R& dlat, R (&Q)[kNVars<MODEL>], R& pt,
                                        const Tgt& tgt) {
#pragma clang fp contract(on)
  constexpr int K = kNVars<MODEL>;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    R acc = f[k][0];
#pragma unroll
    for (int a = 0; a < D; ++a) acc += f[k][2 * a + 1] + f[k][2 * a + 2];
    Q[k] = acc;
  }
  R Jb[3] = {R(0), R(0), R(0)};
  if constexpr (MODEL == 0 || MODEL == 4) {
    constexpr int bx = kBx<MODEL>;
#pragma unroll
    for (int a = 0; a < D; ++a) Jb[a] = f[bx + a][2 * a + 1] - f[bx + a][2 * a + 2];
  }
  R Qt[K], P[K][3], S[K];
#pragma unroll
  for (int k = 0; k < K; ++k) Qt[k] = Q[k];
  tgt(Qt);
  fixed::flux<R, D, MODEL>(Qt, Jb, ph, P, S, dlat, pt);
  const R c = R(ph.s * ph.inv_cs2);  // to c_i . Phi / c_s^2, the units of the equilibrium
  const R wi = R(ph.wi);
  const R w0 = rest_weight<R, D>(wi);
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const R sw0 = w0 * S[k];
    const bool linear = MODEL == 4 && k >= 6;  // the source of a transported gradient
    if constexpr (COLL == 0) {
      const R om = R(ph.omega[k]);
      const R swi = wi * S[k];
      const R d0 = w0 * Qt[k] - f[k][0];
      f[k][0] += linear ? w0 * S[k] + om * d0 : om * d0 + sw0;
      // one operation of all directions after the other, not one direction after the other: in
      // that order neighbouring instructions do not wait for each other
      R r[2 * D];
#pragma unroll
      for (int i = 0; i < 2 * D; ++i) r[i] = i & 1 ? Qt[k] - P[k][i / 2] * c : Qt[k] + P[k][i / 2] * c;
#pragma unroll
      for (int i = 0; i < 2 * D; ++i) r[i] = wi * r[i] - f[k][i + 1];
#pragma unroll
      for (int i = 0; i < 2 * D; ++i) r[i] = om * r[i] + swi;
#pragma unroll
      for (int i = 0; i < 2 * D; ++i) f[k][i + 1] += r[i];
    } else {
      const R oa = R(ph.omega[k]), os = R(ph.omega_s[k]), od = R(ph.omega_d[k]);
      const R d0 = w0 * Qt[k] - f[k][0];
      f[k][0] += linear ? w0 * S[k] + os * d0 : os * d0 + sw0;
      R h[D], sum = R(0);
#pragma unroll
      for (int a = 0; a < D; ++a) {
        h[a] = R(0.5) * (f[k][2 * a + 1] + f[k][2 * a + 2]) - wi * Qt[k];
        sum += h[a];
      }
      const R mean = sum * R(1.0 / D);
      const R trace = os * mean;
#pragma unroll
      for (int a = 0; a < D; ++a) {
        const R fp = f[k][2 * a + 1], fm = f[k][2 * a + 2];
        const R even = trace + od * (h[a] - sum * R(1.0 / D));
        const R p = P[k][a] * c;
        const R odd = R(0.5) * (fp - fm) - wi * p;
        f[k][2 * a + 1] = fp - even - oa * odd + wi * S[k];
        f[k][2 * a + 2] = fm - even + oa * odd + wi * S[k];
      }
    }
  }
}

}  // namespace fixed

// One collision of a cell, its rounding stated (FIXED) or the compiler's.
template <bool FIXED, typename R, int D, int MODEL, int COLL = 0, typename Tgt = NoTarget, int SRC = 0>
__device__ __forceinline__ void collide_cell(R (*f)[2 * D + 1], const Phys& ph, R& dlat, R (&Q)[kNVars<MODEL>], R& pt,
                                             const Tgt& tgt = Tgt{}, R* sp = nullptr) {
  if constexpr (FIXED)
    fixed::collide<R, D, MODEL, COLL>(f, ph, dlat, Q, pt, tgt);
  else
    collide<R, D, MODEL, COLL, Tgt, SRC>(f, ph, dlat, Q, pt, tgt, sp);
}
template <bool FIXED, typename R, int D, int MODEL, int COLL = 0>
__device__ __forceinline__ void collide_cell(R (*f)[2 * D + 1], const Phys& ph, R& dlat) {
  R Q[kNVars<MODEL>];
  R pt;
  collide_cell<FIXED, R, D, MODEL, COLL>(f, ph, dlat, Q, pt);
}

}  // namespace vlbm
