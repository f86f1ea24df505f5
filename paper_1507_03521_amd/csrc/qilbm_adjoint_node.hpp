// Node-local part of the adjoint step, shared by its kernels: the transpose
// of the collision at one node and the f cotangents it leaves.
#pragma once

#include "qilbm_device.hpp"

namespace qilbm {

// Planes of a step record.
enum RecPlane : int { R_PHI = 0, R_MU, R_P, R_S, R_JX, R_JY, R_NPLANES };

// The f cotangents of the pre-collision state: the direct part fd_i plus the
// moment transposes Sbar + c_i.jbar, handed to store(i, value).
template <int I = 0, typename T, typename St>
__device__ __forceinline__ void fbar_out(const St& store, const T fd[9], T bS, T bjx, T bjy) {
  if constexpr (I < 9) {
    T v = fd[I] + bS;
    if constexpr (I != 0) v += cdot<CXS(I), CYS(I)>(bjx, bjy);
    store(I, v);
    fbar_out<I + 1>(store, fd, bS, bjx, bjy);
  }
}

// Transpose of collide_node at one node. Inputs: forward node state m,
// grad p, the populations' post-collision cotangents fh, gh. Outputs: the
// direct cotangents of the pre-collision populations (in fh, gh) and the
// cotangents of the node quantities the collision read.
template <typename T>
struct NodeBar {
  T p, rho, ux, uy, Fx, Fy, drx, dry, D, phi, mu, dpx, dpy, alpha;
};

// The collision in the form the forward kernels evaluate it (per node:
// u.F, u.(grad rho / 3), u.(grad p - F); per direction: s, A = (c-u).F,
// B = (c-u).grad rho / 3, Q = (c-u).(grad p - F), X = A + s (A + B),
// Y = Q + s Q;
//   f* = (1 - 1/tau_f) f + (1/tau_f) w (p + rho s / 3) + kf w (X + src1),
//   g* = (1 - 1/tau_g) g + (1/tau_g) (H + w phi s) + kg w K Y,
// src1 = -rho gamma D / 3, K = -3 phi / rho), transposed. With the weighted
// cotangents a = w fbar*, b = w gbar*:
//   sbar = a (rho/(3 tau_f) + kf (A + B)) + b (phi/tau_g + kg K Q),
//   Abar = kf a (1 + s), Bbar = kf a s, Qbar = kg K b (1 + s),
//   (c.u)bar = sbar (3 + 9 c.u), (1.5 u^2)bar = -sbar,
// and Abar, Bbar, Qbar go to F, grad rho, grad p - F through c - u. The
// sums over directions are carried per node and turned into the node
// cotangents once.
template <int I = 0, typename T>
__device__ __forceinline__ void coll_T_dirs(T fh[9], T gh[9], const CollNode<T>& n, T rp, T pp,
                                            T Kk, T kf, T af, T ag, T (&acc)[17]) {
  if constexpr (I < 9) {
    const T w = T(WGT(I));
    const T a = w * fh[I], b = w * gh[I];
    fh[I] = af * fh[I];
    gh[I] = ag * gh[I];
    T s, cu, A, B, Q;
    if constexpr (I == 0) {
      s = -n.usq15;
      cu = T(0);
      A = -n.uF;
      B = -n.ud;
      Q = -n.uq;
    } else {
      constexpr int cx = CXS(I), cy = CYS(I);
      cu = cdot<cx, cy>(n.ux, n.uy);
      s = fmad(cu, fmad(T(4.5), cu, T(3)), -n.usq15);
      A = cdot<cx, cy>(n.Fx, n.Fy) - n.uF;
      B = cdot<cx, cy>(n.dx, n.dy) - n.ud;
      Q = cdot<cx, cy>(n.qx, n.qy) - n.uq;
    }
    const T sbar = fmad(a, fmad(kf, A + B, rp), b * fmad(Kk, Q, pp));
    acc[0] += a;                       // sum a
    acc[1] = fmad(s, a, acc[1]);       // sum s a
    acc[2] = fmad(s, b, acc[2]);       // sum s b
    if constexpr (I != 0) acc[3] += b; // sum over i > 0 of b
    acc[4] = fmad(fmad(s, Q, Q), b, acc[4]);   // sum Y b
    const T Au = fmad(s, a, a), Bu = s * a, Qu = fmad(s, b, b);
    acc[5] += Au;
    acc[8] += Bu;
    acc[11] += Qu;
    if constexpr (I != 0) {
      constexpr int cx = CXS(I), cy = CYS(I);
      if constexpr (cx != 0) {
        acc[6] = cx > 0 ? acc[6] + Au : acc[6] - Au;
        acc[9] = cx > 0 ? acc[9] + Bu : acc[9] - Bu;
        acc[12] = cx > 0 ? acc[12] + Qu : acc[12] - Qu;
      }
      if constexpr (cy != 0) {
        acc[7] = cy > 0 ? acc[7] + Au : acc[7] - Au;
        acc[10] = cy > 0 ? acc[10] + Bu : acc[10] - Bu;
        acc[13] = cy > 0 ? acc[13] + Qu : acc[13] - Qu;
      }
      const T cbar = sbar * fmad(T(9), cu, T(3));
      if constexpr (cx != 0) acc[14] = cx > 0 ? acc[14] + cbar : acc[14] - cbar;
      if constexpr (cy != 0) acc[15] = cy > 0 ? acc[15] + cbar : acc[15] - cbar;
    }
    acc[16] += sbar;
    coll_T_dirs<I + 1>(fh, gh, n, rp, pp, Kk, kf, af, ag, acc);
  }
}

template <typename T>
__device__ __forceinline__ void collide_node_T(T fh[9], T gh[9], const Macro<T>& m, T dpx, T dpy,
                                               const Coef<T>& c, NodeBar<T>& nb) {
  const CollNode<T> n = coll_node(m, dpx, dpy);
  const T itf = c.inv_tau_f, itg = c.inv_tau_g;
  const T rinv = recip(m.rho);
  const T K = -T(3) * m.phi * rinv;
  const T Kk = K * c.kg;
  const T rp = m.rho * (itf * T(1.0 / 3.0));
  const T pp = m.phi * itg;
  const T b0 = gh[0];
  T acc[17];
#pragma unroll
  for (int j = 0; j < 17; ++j) acc[j] = T(0);
  coll_T_dirs(fh, gh, n, rp, pp, Kk, c.kf, T(1) - itf, T(1) - itg, acc);
  const T src1_bar = c.kf * acc[0];
  const T K_bar = c.kg * acc[4];
  // A, B, Q cotangents through c - u
  const T uF_bar = -c.kf * acc[5], ud_bar = -c.kf * acc[8], uq_bar = -Kk * acc[11];
  const T qx_bar = fmad(uq_bar, n.ux, Kk * acc[12]);
  const T qy_bar = fmad(uq_bar, n.uy, Kk * acc[13]);
  const T dx_bar = fmad(ud_bar, n.ux, c.kf * acc[9]);
  const T dy_bar = fmad(ud_bar, n.uy, c.kf * acc[10]);
  const T usq_bar = -acc[16];     // cotangent of 1.5 |u|^2
  nb.p = itf * acc[0];
  nb.rho = fmad(itf * T(1.0 / 3.0), acc[1],
                fmad(src1_bar, -c.gamma * m.D * T(1.0 / 3.0), K_bar * (T(3) * m.phi) * rinv * rinv));
  nb.D = -src1_bar * m.rho * c.gamma * T(1.0 / 3.0);
  nb.drx = dx_bar * T(1.0 / 3.0);
  nb.dry = dy_bar * T(1.0 / 3.0);
  // H_0 = phi - (1 - w_0) alpha mu, H_i = w_i alpha mu: (alpha mu)bar
  const T amu_bar = itg * fmad(-T(1.0 - 4.0 / 9.0), b0, acc[3]);
  nb.mu = c.alpha * amu_bar;
  nb.alpha = m.mu * amu_bar;
  nb.phi = fmad(itg, acc[2] + b0, -T(3) * K_bar * rinv);
  nb.dpx = qx_bar;
  nb.dpy = qy_bar;
  nb.Fx = fmad(uF_bar, n.ux, c.kf * acc[6]) - qx_bar;
  nb.Fy = fmad(uF_bar, n.uy, c.kf * acc[7]) - qy_bar;
  nb.ux = fmad(T(3) * n.ux, usq_bar,
               fmad(uq_bar, n.qx, fmad(ud_bar, n.dx, fmad(uF_bar, n.Fx, acc[14]))));
  nb.uy = fmad(T(3) * n.uy, usq_bar,
               fmad(uq_bar, n.qy, fmad(ud_bar, n.dy, fmad(uF_bar, n.Fy, acc[15]))));
}

}  // namespace qilbm
