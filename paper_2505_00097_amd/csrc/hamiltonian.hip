// hamiltonian.hip -- the constraints: Hamiltonian (Eq. 16 of arXiv:2505.00097),
// momentum (Eq. 17) and C^i, at every interior point, centred differences of
// the grid's order (4th with 3 ghost layers, 8th with 5).
//
// Frame components (rhs_frame.h), with Delta_d = gammabar_dk Delta^k,
// psi_d = Delta^k_kd and W_k = -2 W phi_k:
//   H   = 2/3 K^2 - Abar_ij Abar^ij + W^2 Rbar
//         + 4 W gammabar^ij Dbar_i Dbar_j W - 6 gammabar^ij W_i W_j
//   M^i = W^2 gammabar^ia (gammabar^jb Dhat_j a_ab - 1/2 Abar^jk Dhat_a h_jk - 2/3 K_a)
//         - Abar^id (3 W W_d + W^2 Delta_d)
//   C^i = lambda^i - Delta^i
// (the derivatives of gammabar^ij in Dhat_j Abar^ij and the Delta terms of
// Eq. 17 partly cancel; the components of lambda^i, M^i and C^i are the
// rescaled ones).
//
// Two waves per 16 x 4 tile, as the right-hand side and through the same
// stencil stage: one takes h_ij, the Ricci tensor and H, the other W, lambda^i
// and, where M^i or C^i is asked for, a_ij, K and M^i. What bounds it: with
// two waves per SIMD the latency of the stage and the algebra; one thread per
// point with every stencil value read per lane (and 300 to 500 bytes of
// spills) took 34 us for H on the 128 x 2 x 256 grid and 244 us for all
// three on a spherical 128 x 64 x 32 one, now 7.6 and 38 us.
#include "rhs_stencil.h"

// The library builds this source in parts (one kernel variant each, as
// rhs_fused.hip); without a part everything is instantiated in one unit.
#ifndef BHAH_PART
#define BHAH_PART -1
#endif

namespace bhah {

// LDS slots per point (slot v of lane l at xs[v * 64 + l])
template <bool AX, int H>
struct ConSlots {
  static constexpr int SL = StageSize<AX, H>::SL;  // a wave's stencil stage
  static constexpr int HK = SL;                // 18 e_k h_ij at HK + 6 k + ij
  static constexpr int LK = HK + 18;           // 9  e_k lambda^i at LK + 3 k + i
  static constexpr int W1 = LK + 9;            // 3  e_k W
  static constexpr int S = W1 + 3;             // 1  H without W^2 Rbar and the Delta term of Dbar Dbar W
  static constexpr int AK = S + 1;             // 18 e_k a_ij (gauge wave only)
  static constexpr int GAUGE = AK + 18;        // the second wave's stage
  static constexpr int N = GAUGE + SL;
};

template <int C, bool AX, int H, bool MC>
__device__ __forceinline__ void constraints_tile(const GridDev& G, const TileMap& T, int w,
                                                 const double* __restrict__ y, double* __restrict__ Hc,
                                                 double* __restrict__ Mo, double* __restrict__ Co,
                                                 double* __restrict__ xs0) {
  constexpr int PD = C == BHAH_SINH_CYLINDRICAL ? 1 : 2;
  using CS = ConSlots<AX, H>;
  const int lane = (int)(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  TilePoint p;
  p.live = tile_point<H>(G, T, w, lane, p.t0, p.t1, p.t2, p.i0, p.i1, p.i2);
  p.q = (unsigned)(p.i0 + G.s1 * p.i1 + G.s2 * p.i2);
  double* xs = xs0 + lane;
  auto put = [&](int v, double x) { xs[v * 64] = x; };
  auto get = [&](int v) { return xs[v * 64]; };
  auto at = [&](int g) { return gf_ld(y, G.sgf, g, p.q * 8u, 0); };
  const auto S = make_source<C, AX, H>(y, G, p, lane, xs0 + (wave ? CS::GAUGE * 64 : 0));
  double gU[6], gd[6];
  {
    double h[6];
#pragma unroll
    for (int a = 0; a < 6; a++) h[a] = at(G_HDD00 + a);
    metric_inverse(h, gU);
    doubled(gU, gd);
  }
  Coefs<H> c;  // only the scales are used: the constraints have no advection
  double wg[6];
  {
    const Frame F = load_frame<C>(G, p.i0, p.i1, p.i2);
    const double v0[3] = {0.0, 0.0, 0.0};
    make_coefs<false, H>(G, Gauge{0.0, 0.0, 0.0}, F.iS, v0, c);
  }
#pragma unroll
  for (int k = 0; k < 3; k++)
#pragma unroll
    for (int l = k; l < 3; l++) wg[sy(k, l)] = gd[sy(k, l)] * c.sc(k, l);

  if (wave == 0) {
    double L6[6], h[6];
#pragma unroll
    for (int a = 0; a < 6; a++) L6[a] = 0.0;
    constexpr int list[6] = {G_HDD00, G_HDD00 + 1, G_HDD00 + 2, G_HDD00 + 3, G_HDD00 + 4, G_HDD00 + 5};
    run_stencils<C, AX, H, 0, 6, 6, false>(
        S, list, [&](int a, const AxisSums(&s)[3], const double(&dd)[6], double c0) BHAH_INLINE {
          h[a] = c0;
          pin(h[a]);
#pragma unroll
          for (int k = 0; k < 3; k++)
            if (!(AX && k == PD)) put(CS::HK + 6 * k + a, c.s1[k] * s[k].d1);
#pragma unroll
          for (int kl = 0; kl < 6; kl++) L6[a] = fma(wg[kl], dd[kl], L6[a]);
          pin(L6[a]);
        });
    BHAH_PHASE_BARRIER();
    double hk[3][6], D[3][6], Rc[6], DU[3], Del[3][6];
#pragma unroll
    for (int a = 0; a < 6; a++) {
#pragma unroll
      for (int k = 0; k < 3; k++) hk[k][a] = AX && k == PD ? 0.0 : get(CS::HK + 6 * k + a);
    }
    const Frame F = load_frame<C>(G, p.i0, p.i1, p.i2);
    const double W = at(G_CF);
    double lam[3];
#pragma unroll
    for (int i = 0; i < 3; i++) lam[i] = at(G_LAMU0 + i);
    cov_deriv<C, 6>(F, h, hk, D);
    {
      const Lower L = lower_terms<C>(F, gU);
      add_lower<C, 6>(F, L, gU, h, hk, D, L6);
#pragma unroll
      for (int a = 0; a < 6; a++) Rc[a] = -0.5 * L6[a];
    }
    BHAH_PHASE_BARRIER();
#pragma unroll
    for (int k = 0; k < 3; k++)
#pragma unroll
      for (int a = 0; a < 6; a++) Del[k][a] = 0.0;
#pragma unroll
    for (int l = 0; l < 3; l++) {
      double low[6];
      delta_lower(D, l, low);
#pragma unroll
      for (int k = 0; k < 3; k++)
#pragma unroll
        for (int a = 0; a < 6; a++) Del[k][a] = fma(gU[sy(k, l)], low[a], Del[k][a]);
    }
#pragma unroll
    for (int k = 0; k < 3; k++) DU[k] = dot6(gd, Del[k]);
    BHAH_PHASE_BARRIER();
    add_ricci_delta(gU, D, DU, [&](int k, int a) { return Del[k][a]; }, Rc);
    __syncthreads();
    double lk[3][3], Dl[3][3];
#pragma unroll
    for (int k = 0; k < 3; k++)
#pragma unroll
      for (int i = 0; i < 3; i++) lk[k][i] = AX && k == PD ? 0.0 : get(CS::LK + 3 * k + i);
    cov_deriv<C, 3>(F, lam, lk, Dl);
    add_ricci_lambda(h, Dl, Rc);
    double dw = 0.0;
#pragma unroll
    for (int k = 0; k < 3; k++)
      if (!(AX && k == PD)) dw = fma(DU[k], get(CS::W1 + k), dw);
    if (!p.live) return;
    if (Hc) Hc[p.q] = fma(W, fma(W, dot6(gd, Rc), -4.0 * dw), get(CS::S));
    if constexpr (MC) {
      if (Co) {
#pragma unroll
        for (int i = 0; i < 3; i++) Co[i * G.sgf + p.q] = lam[i] - DU[i];
      }
    }
  } else {
    double LW = 0.0, Wk[3], Kk[3];
    constexpr int N = MC ? 11 : 4;
    constexpr int full[11] = {G_CF, G_LAMU0, G_LAMU0 + 1, G_LAMU0 + 2, G_TRK, 0, 1, 2, 3, 4, 5};
    int list[N];
#pragma unroll
    for (int t = 0; t < N; t++) list[t] = full[t];
    run_stencils<C, AX, H, 0, 1, N, false>(
        S, list, [&](int t, const AxisSums(&s)[3], const double(&dd)[6], double) BHAH_INLINE {
          double d[3];
#pragma unroll
          for (int k = 0; k < 3; k++) d[k] = AX && k == PD ? 0.0 : c.s1[k] * s[k].d1;
          if (t == 0) {
#pragma unroll
            for (int k = 0; k < 3; k++) {
              Wk[k] = d[k];
              if (!(AX && k == PD)) put(CS::W1 + k, d[k]);
            }
#pragma unroll
            for (int kl = 0; kl < 6; kl++) LW = fma(wg[kl], dd[kl], LW);
            pin(LW);
          } else if (t < 4) {
#pragma unroll
            for (int k = 0; k < 3; k++)
              if (!(AX && k == PD)) put(CS::LK + 3 * k + t - 1, d[k]);
          } else if (t == 4) {
#pragma unroll
            for (int k = 0; k < 3; k++) Kk[k] = d[k];
          } else {
#pragma unroll
            for (int k = 0; k < 3; k++)
              if (!(AX && k == PD)) put(CS::AK + 6 * k + t - 5, d[k]);
          }
        });
    BHAH_PHASE_BARRIER();
    const Frame F = load_frame<C>(G, p.i0, p.i1, p.i2);
    const double W = at(G_CF), K = at(G_TRK);
    double a6[6], AUD[3][3], AUU[6], AUUd[6];
#pragma unroll
    for (int a = 0; a < 6; a++) a6[a] = at(G_ADD00 + a);
    raise_first(gU, a6, AUD);
    raise_second(gU, AUD, AUU);
    doubled(AUU, AUUd);
    {
      const Lower L = lower_terms<C>(F, gU);
      double g2 = 0.0;
#pragma unroll
      for (int i = 0; i < 3; i++) {
        LW = fma(L.n[i], Wk[i], LW);
        double u = gU[sy(i, 0)] * Wk[0];
        u = fma(gU[sy(i, 1)], Wk[1], u);
        u = fma(gU[sy(i, 2)], Wk[2], u);
        g2 = fma(u, Wk[i], g2);
      }
      const double s = fma((2.0 / 3.0) * K, K, -dot6(AUUd, a6));
      put(CS::S, fma(-6.0, g2, fma(4.0 * W, LW, s)));
    }
    __syncthreads();
    if constexpr (MC) {
      if (!Mo || !p.live) return;
      double h[6], hk[3][6], D[3][6], ak[3][6], Da[3][6], z[3], dl[3];
#pragma unroll
      for (int a = 0; a < 6; a++) {
        h[a] = at(G_HDD00 + a);
#pragma unroll
        for (int k = 0; k < 3; k++) {
          hk[k][a] = AX && k == PD ? 0.0 : get(CS::HK + 6 * k + a);
          ak[k][a] = AX && k == PD ? 0.0 : get(CS::AK + 6 * k + a);
        }
      }
      cov_deriv<C, 6>(F, h, hk, D);
      cov_deriv<C, 6>(F, a6, ak, Da);
#pragma unroll
      for (int a = 0; a < 3; a++) {
        // gammabar^jb Dhat_j (a_ab, h_ab); Delta_a = gammabar^jb Dhat_j h_ab - psi_a
        double s = fma(-0.5, dot6(AUUd, D[a]), -(2.0 / 3.0) * Kk[a]), d = -0.5 * dot6(gd, hk[a]);
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
          for (int b = 0; b < 3; b++) {
            s = fma(gU[sy(j, b)], Da[j][sy(a, b)], s);
            d = fma(gU[sy(j, b)], D[j][sy(a, b)], d);
          }
        z[a] = s;
        dl[a] = fma(W, d, 3.0 * Wk[a]);
      }
#pragma unroll
      for (int i = 0; i < 3; i++) {
        double s = 0.0, t = 0.0;
#pragma unroll
        for (int a = 0; a < 3; a++) {
          s = fma(gU[sy(i, a)], z[a], s);
          t = fma(AUU[sy(i, a)], dl[a], t);
        }
        Mo[i * G.sgf + p.q] = W * fma(W, s, -t);
      }
    }
  }
}

template <int C, bool AX, int H, bool MC>
__global__ void __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_constraints(GridDev G, TileMap T, const double* __restrict__ y, double* __restrict__ Hc, double* __restrict__ Mo,
              double* __restrict__ Co) {
  const int per = (T.ntiles + BHAH_NXCD - 1) / BHAH_NXCD;
  const int w = xcd_remap((int)blockIdx.x, per);
  if (w >= T.ntiles) return;
  __shared__ __attribute__((aligned(16))) double xs[ConSlots<AX, H>::N * 64];
  static_assert(sizeof(xs) <= 40960, "four blocks per CU");
  constraints_tile<C, AX, H, MC>(G, T, w, y, Hc, Mo, Co, xs);
}

using ConLaunch = void (*)(dim3, hipStream_t, const GridDev&, const TileMap&, const double*, double*, double*, double*);
template <int C, bool AX, int H, bool MC>
void launch_con_t(dim3 g, hipStream_t s, const GridDev& G, const TileMap& T, const double* y, double* Hc, double* Mo,
                  double* Co) {
  hipLaunchKernelGGL((k_constraints<C, AX, H, MC>), g, dim3(128), 0, s, G, T, y, Hc, Mo, Co);
}
// [M^i or C^i asked for], per variant (rhs_variant)
template <int V>
ConLaunch con_part(bool mc);
#define BHAH_DEFINE_PART(V)                                                                                     \
  template <>                                                                                                   \
  ConLaunch con_part<V>(bool mc) {                                                                              \
    return mc ? launch_con_t<(V) / 2 % 3, (V) % 2 == 1, (V) >= 6 ? 5 : 3, true>                                 \
              : launch_con_t<(V) / 2 % 3, (V) % 2 == 1, (V) >= 6 ? 5 : 3, false>;                               \
  }
#if BHAH_PART >= 0
BHAH_DEFINE_PART(BHAH_PART)
#else
BHAH_DEFINE_PART(0) BHAH_DEFINE_PART(1) BHAH_DEFINE_PART(2) BHAH_DEFINE_PART(3) BHAH_DEFINE_PART(4)
BHAH_DEFINE_PART(5) BHAH_DEFINE_PART(6) BHAH_DEFINE_PART(7) BHAH_DEFINE_PART(8) BHAH_DEFINE_PART(9)
BHAH_DEFINE_PART(10) BHAH_DEFINE_PART(11)
#endif

#if BHAH_PART <= 0
template <> ConLaunch con_part<1>(bool);
template <> ConLaunch con_part<2>(bool);
template <> ConLaunch con_part<3>(bool);
template <> ConLaunch con_part<4>(bool);
template <> ConLaunch con_part<5>(bool);
template <> ConLaunch con_part<6>(bool);
template <> ConLaunch con_part<7>(bool);
template <> ConLaunch con_part<8>(bool);
template <> ConLaunch con_part<9>(bool);
template <> ConLaunch con_part<10>(bool);
template <> ConLaunch con_part<11>(bool);

void launch_constraints(const GridDev& G, const double* y, double* Hc, double* Mo, double* Co, hipStream_t s) {
  using Get = ConLaunch (*)(bool);
  static const Get get[NVAR] = {con_part<0>, con_part<1>, con_part<2>, con_part<3>, con_part<4>,  con_part<5>,
                                con_part<6>, con_part<7>, con_part<8>, con_part<9>, con_part<10>, con_part<11>};
  const TileMap T = make_tilemap(G, BHAH_DEFAULT_BAND);
  const int per = (T.ntiles + BHAH_NXCD - 1) / BHAH_NXCD;
  get[rhs_variant(G.coord, G.N1, G.N2, G.ng)](Mo || Co)(dim3(per * BHAH_NXCD), s, G, T, y, Hc, Mo, Co);
}

void launch_hamiltonian(const GridDev& G, const double* y, double* H, hipStream_t s) {
  launch_constraints(G, y, H, nullptr, nullptr, s);
}
#endif

}  // namespace bhah
