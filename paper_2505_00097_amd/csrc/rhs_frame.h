// rhs_frame.h -- the algebra of the right-hand sides in the orthonormal frame
// of the reference metric.
//
// The rescaled variables are the components of their tensors in the frame
// e_k = (1/S_k) d_k (Sec. 2.2 of arXiv:2505.00097: h_ij = eps_ij/(S_i S_j),
// lambda^i = S_i Lambdabar^i, ...). There gammahat_ij = delta_ij and
// gammabar_ij = delta_ij + h_ij, no product of scale factors appears, and the
// reference connection is a rotation: with sigma_kl = e_k ln S_l,
//   Dhat_k V = e_k V + A_k V,   Dhat_k T = e_k T + A_k T + (A_k T)^T,
//   (A_k)_kj = sigma_jk, (A_k)_jk = -sigma_jk (j != k), all other entries 0.
// Spherical families: A_theta = a J_01, A_phi = a J_02 + b J_12 with a = 1/r,
// b = cot(theta)/r; cylindrical: A_phi = a J_01 with a = 1/rho, where J_PQ is
// the generator with (J)_QP = 1, (J)_PQ = -1. The only other entries of sigma
// are sigma_00 and, on cylindrical grids, sigma_22 (the sinh maps).
// f_k below is e_k f = d_k f / S_k and f_kl is d_k d_l f / (S_k S_l), so
// e_k e_l f = f_kl - sigma_kl f_l. Everything else (Delta, Ricci, the
// equations) follows the paper's covariant forms with frame components.
//
// In coordinate components the same right-hand side takes about twice the
// operations (products with S_i S_j and their derivatives, derivatives of the
// reference Christoffel symbols, both of which cancel).
#pragma once

#include "rhs_common.h"

namespace bhah {

// the frame at a point: 1/S_k, sigma_00, sigma_22 (cylindrical), a, b
struct Frame {
  double iS[3], s0, s2, a, b;
};

template <int C>
__device__ __forceinline__ Frame load_frame(const GridDev& G, int i0, int i1, int i2) {
  Frame F;
  const double* t0 = G.tab0 + i0 * TAB_W;
  F.iS[0] = t0[5];
  F.iS[1] = t0[4];
  F.s0 = C == BHAH_SPHERICAL ? 0.0 : t0[2] * (t0[5] * t0[5]);
  F.a = t0[4];
  if constexpr (C == BHAH_SINH_CYLINDRICAL) {
    const double* t2 = G.tab2 + i2 * TAB_W;
    F.iS[2] = t2[5];
    F.s2 = t2[2] * (t2[5] * t2[5]);
    F.b = 0.0;
  } else {
    const double* t1 = G.tab1 + i1 * TAB_W;
    F.iS[2] = t0[4] * t1[2];
    F.s2 = 0.0;
    F.b = (t1[1] * t1[2]) * t0[4];
  }
  return F;
}

// o += c (J_PQ T + (J_PQ T)^T) for a symmetric T, P < Q
template <int P, int Q>
__device__ __forceinline__ void add_rot(double (&o)[6], const double (&T)[6], double c) {
  constexpr int R = 3 - P - Q;
  const double c2 = c + c;
  o[sy(P, P)] = fma(-c2, T[sy(P, Q)], o[sy(P, P)]);
  o[sy(Q, Q)] = fma(c2, T[sy(P, Q)], o[sy(Q, Q)]);
  o[sy(P, Q)] = fma(c, T[sy(P, P)] - T[sy(Q, Q)], o[sy(P, Q)]);
  o[sy(P, R)] = fma(-c, T[sy(Q, R)], o[sy(P, R)]);
  o[sy(Q, R)] = fma(c, T[sy(P, R)], o[sy(Q, R)]);
}
// o += c J_PQ V
template <int P, int Q>
__device__ __forceinline__ void add_rotv(double (&o)[3], const double (&V)[3], double c) {
  o[P] = fma(-c, V[Q], o[P]);
  o[Q] = fma(c, V[P], o[Q]);
}
// o += A_k X for a symmetric tensor (both indices) or a vector X
template <int C, int K>
__device__ __forceinline__ void add_conn(const Frame& F, double (&o)[6], const double (&X)[6]) {
  if constexpr (K == 1) add_rot<0, 1>(o, X, F.a);
  if constexpr (K == 2 && C != BHAH_SINH_CYLINDRICAL) {
    add_rot<0, 2>(o, X, F.a);
    add_rot<1, 2>(o, X, F.b);
  }
}
template <int C, int K>
__device__ __forceinline__ void add_conn(const Frame& F, double (&o)[3], const double (&X)[3]) {
  if constexpr (K == 1) add_rotv<0, 1>(o, X, F.a);
  if constexpr (K == 2 && C != BHAH_SINH_CYLINDRICAL) {
    add_rotv<0, 2>(o, X, F.a);
    add_rotv<1, 2>(o, X, F.b);
  }
}
// Dhat_k X from X_k = e_k X, all k (N components: 6 symmetric or 3 vector)
template <int C, int N>
__device__ __forceinline__ void cov_deriv(const Frame& F, const double (&X)[N], const double (&Xk)[3][N],
                                          double (&D)[3][N]) {
#pragma unroll
  for (int k = 0; k < 3; k++)
#pragma unroll
    for (int c = 0; c < N; c++) D[k][c] = Xk[k][c];
  add_conn<C, 1>(F, D[1], X);
  add_conn<C, 2>(F, D[2], X);
}

// gammabar^ij of gammabar_ij = delta_ij + h_ij
__device__ __forceinline__ void metric_inverse(const double (&h)[6], double (&gU)[6]) {
  const double g[6] = {1.0 + h[0], h[1], h[2], 1.0 + h[3], h[4], 1.0 + h[5]};
  sym_inverse(g, gU);
}

// Coefficients of gammabar^kl Dhat_k Dhat_l X below second order:
//   gammabar^kl Dhat_k Dhat_l X = gammabar^kl X_kl + sum_m n_m X_m + B X
//                                + sum_l A_l sum_k gammabar^kl (X_k + Dhat_k X),
// n_m X_m being the scalar part (for a scalar X all of it), B the rotation
// with coefficients b01, b02, b12 of J_01, J_02, J_12.
struct Lower {
  double n[3], b01, b02, b12;
};
template <int C>
__device__ __forceinline__ Lower lower_terms(const Frame& F, const double (&gU)[6]) {
  Lower L;
  const double a = F.a, b = F.b;
  if constexpr (C == BHAH_SINH_CYLINDRICAL) {
    const double t1 = -a * gU[1];
    L.n[0] = fma(a, gU[3], -(gU[0] * F.s0));
    L.n[1] = t1 + t1;
    L.n[2] = -(gU[5] * F.s2);
    L.b01 = fma(t1, a, t1 * a);
    L.b02 = L.b12 = 0.0;
  } else {
    const double t1 = fma(b, gU[5], -(a * gU[1])), t2 = -fma(a, gU[2], b * gU[4]);
    L.n[0] = fma(a, gU[3] + gU[5], -(gU[0] * F.s0));
    L.n[1] = fma(-a, gU[1], t1);
    L.n[2] = t2 + t2;
    L.b01 = a * fma(-a, gU[1], t1);
    L.b02 = a * fma(-a, gU[2], t2);
    L.b12 = fma(t2, b, -fma(a * b, gU[2], fma(a, a, b * b) * gU[4]));
  }
  return L;
}
// the terms above added to o, which holds gammabar^kl X_kl (N: 6 or 3)
template <int C, int N>
__device__ __forceinline__ void add_lower(const Frame& F, const Lower& L, const double (&gU)[6], const double (&X)[N],
                                          const double (&Xk)[3][N], const double (&D)[3][N], double (&o)[N]) {
#pragma unroll
  for (int c = 0; c < N; c++)
    o[c] = fma(L.n[2], Xk[2][c], fma(L.n[1], Xk[1][c], fma(L.n[0], Xk[0][c], o[c])));
  if constexpr (N == 6) {
    add_rot<0, 1>(o, X, L.b01);
    if constexpr (C != BHAH_SINH_CYLINDRICAL) {
      add_rot<0, 2>(o, X, L.b02);
      add_rot<1, 2>(o, X, L.b12);
    }
  } else {
    add_rotv<0, 1>(o, X, L.b01);
    if constexpr (C != BHAH_SINH_CYLINDRICAL) {
      add_rotv<0, 2>(o, X, L.b02);
      add_rotv<1, 2>(o, X, L.b12);
    }
  }
  auto z = [&](int l, double (&Z)[N]) {
#pragma unroll
    for (int c = 0; c < N; c++) {
      double s = gU[sy(0, l)] * (Xk[0][c] + D[0][c]);
      s = fma(gU[sy(1, l)], Xk[1][c] + D[1][c], s);
      Z[c] = fma(gU[sy(2, l)], Xk[2][c] + D[2][c], s);
    }
  };
  double Z[N];
  z(1, Z);
  add_conn<C, 1>(F, o, Z);
  if constexpr (C != BHAH_SINH_CYLINDRICAL) {
    z(2, Z);
    add_conn<C, 2>(F, o, Z);
  }
}

// Dhat_i Dhat_j f - f_ij of a scalar with derivatives f_k, added to o
template <int C>
__device__ __forceinline__ void add_hessian_lower(const Frame& F, const double (&f)[3], double (&o)[6]) {
  o[0] = fma(-F.s0, f[0], o[0]);
  o[1] = fma(-F.a, f[1], o[1]);
  if constexpr (C == BHAH_SINH_CYLINDRICAL) {
    o[3] = fma(F.a, f[0], o[3]);
    o[5] = fma(-F.s2, f[2], o[5]);
  } else {
    o[2] = fma(-F.a, f[2], o[2]);
    o[3] = fma(F.a, f[0], o[3]);
    o[4] = fma(-F.b, f[2], o[4]);
    o[5] = fma(F.b, f[1], fma(F.a, f[0], o[5]));
  }
}

// Delta_l,ij = (Dhat_i h_lj + Dhat_j h_il - Dhat_l h_ij)/2 (Eq. 4, index
// lowered) for one l, from D[k][ij] = Dhat_k h_ij
__device__ __forceinline__ void delta_lower(const double (&D)[3][6], int l, double (&low)[6]) {
#pragma unroll
  for (int i = 0; i < 3; i++)
#pragma unroll
    for (int j = i; j < 3; j++) {
      if (i == j) low[sy(i, j)] = i == l ? 0.5 * D[l][sy(l, l)] : fma(-0.5, D[l][sy(i, i)], D[i][sy(l, i)]);
      else if (i == l) low[sy(i, j)] = 0.5 * D[j][sy(l, l)];
      else if (j == l) low[sy(i, j)] = 0.5 * D[i][sy(l, l)];
      else low[sy(i, j)] = 0.5 * ((D[i][sy(l, j)] + D[j][sy(i, l)]) - D[l][sy(i, j)]);
    }
}

// full contraction of two symmetric tensors given by six components; w holds
// one of them with its off-diagonal components doubled
__device__ __forceinline__ double dot6(const double (&w)[6], const double (&T)[6]) {
  double s = w[0] * T[0];
#pragma unroll
  for (int c = 1; c < 6; c++) s = fma(w[c], T[c], s);
  return s;
}
__device__ __forceinline__ void doubled(const double (&T)[6], double (&w)[6]) {
  w[0] = T[0]; w[3] = T[3]; w[5] = T[5];
  w[1] = T[1] + T[1]; w[2] = T[2] + T[2]; w[4] = T[4] + T[4];
}
// T^i_j = gammabar^ik T_kj
__device__ __forceinline__ void raise_first(const double (&gU)[6], const double (&T)[6], double (&M)[3][3]) {
#pragma unroll
  for (int i = 0; i < 3; i++)
#pragma unroll
    for (int j = 0; j < 3; j++)
      M[i][j] = fma(gU[sy(i, 2)], T[sy(2, j)], fma(gU[sy(i, 1)], T[sy(1, j)], gU[sy(i, 0)] * T[sy(0, j)]));
}
// T^ij = T^i_k gammabar^kj
__device__ __forceinline__ void raise_second(const double (&gU)[6], const double (&M)[3][3], double (&T)[6]) {
#pragma unroll
  for (int i = 0; i < 3; i++)
#pragma unroll
    for (int j = i; j < 3; j++)
      T[sy(i, j)] = fma(M[i][2], gU[sy(2, j)], fma(M[i][1], gU[sy(1, j)], M[i][0] * gU[sy(0, j)]));
}

// L_i^k of beta^k d_k T_ij + T_kj d_i beta^k + T_ik d_j beta^k
// = (advection of the components) + L_i^k T_kj + L_j^k T_ik, in frame
// components, from v_i = e_i v and D_i v = Dhat_i v: L[i][k]
template <int C>
__device__ __forceinline__ void lie_matrix(const Frame& F, const double (&v)[3], const double (&vk)[3][3],
                                           const double (&Dv)[3][3], double (&L)[3][3]) {
#pragma unroll
  for (int i = 0; i < 3; i++)
#pragma unroll
    for (int k = 0; k < 3; k++) L[i][k] = i == k ? Dv[i][i] : vk[i][k];
  L[0][1] = fma(-F.a, v[1], L[0][1]);
  if constexpr (C != BHAH_SINH_CYLINDRICAL) {
    L[0][2] = fma(-F.a, v[2], L[0][2]);
    L[1][2] = fma(-F.b, v[2], L[1][2]);
  }
}
// L_i^k T_kj + L_j^k T_ik added to o
__device__ __forceinline__ void add_lie(const double (&L)[3][3], const double (&T)[6], int i, int j, double& o) {
#pragma unroll
  for (int k = 0; k < 3; k++) o = fma(L[i][k], T[sy(k, j)], o);
#pragma unroll
  for (int k = 0; k < 3; k++) o = fma(L[j][k], T[sy(i, k)], o);
}

// Ricci tensor (Eq. 12) without its second-derivative part and its Lambdabar
// part: 1/2 Delta^k Dhat_k h_ij (= Delta^k Delta_(ij)k) and
// gammabar^kl (2 Delta^m_k(i Delta_j)ml + Delta^m_ik Delta_mjl), added to Rc;
// Del(k, ij) is Delta^k_ij. One lowered index p at a time, so that few of the
// 27 values gammabar^kl Delta_pml live together.
template <class DEL>
__device__ __forceinline__ void add_ricci_delta(const double (&gU)[6], const double (&D)[3][6], const double (&DU)[3],
                                                const DEL& Del, double (&Rc)[6]) {
#pragma unroll
  for (int c = 0; c < 6; c++)
#pragma unroll
    for (int k = 0; k < 3; k++) Rc[c] = fma(0.5 * DU[k], D[k][c], Rc[c]);
#pragma unroll
  for (int p = 0; p < 3; p++) {
    double low[6], E[3][3];  // E[m][k] = gammabar^kl Delta_pml
    delta_lower(D, p, low);
#pragma unroll
    for (int m = 0; m < 3; m++)
#pragma unroll
      for (int k = 0; k < 3; k++)
        E[m][k] = fma(gU[sy(k, 2)], low[sy(m, 2)], fma(gU[sy(k, 1)], low[sy(m, 1)], gU[sy(k, 0)] * low[sy(m, 0)]));
    // Delta^m_ki E_p,m^k goes to (i, p) and (p, i): twice to the diagonal
#pragma unroll
    for (int i = 0; i < 3; i++) {
      double u = 0.0;
#pragma unroll
      for (int m = 0; m < 3; m++)
#pragma unroll
        for (int k = 0; k < 3; k++) u = fma(Del(m, sy(k, i)), E[m][k], u);
      Rc[sy(i, p)] = i == p ? fma(2.0, u, Rc[sy(i, p)]) : Rc[sy(i, p)] + u;
    }
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
      for (int j = i; j < 3; j++)
#pragma unroll
        for (int k = 0; k < 3; k++) Rc[sy(i, j)] = fma(Del(p, sy(i, k)), E[j][k], Rc[sy(i, j)]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// gammabar_k(i Dhat_j) Lambdabar^k added to Rc, from Dl[j][k] = Dhat_j lambda^k
__device__ __forceinline__ void add_ricci_lambda(const double (&h)[6], const double (&Dl)[3][3], double (&Rc)[6]) {
#pragma unroll
  for (int i = 0; i < 3; i++)
#pragma unroll
    for (int j = i; j < 3; j++) {
      double s = Dl[j][i] + Dl[i][j];
#pragma unroll
      for (int k = 0; k < 3; k++) s = fma(h[sy(k, i)], Dl[j][k], fma(h[sy(k, j)], Dl[i][k], s));
      Rc[sy(i, j)] = fma(0.5, s, Rc[sy(i, j)]);
    }
}

}  // namespace bhah
