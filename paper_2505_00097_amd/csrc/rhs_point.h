// rhs_point.h -- the full BSSN + gauge right-hand side (Eqs. 7-15 with the
// conformal Ricci tensor of Eq. 12, arXiv:2505.00097) of one 64-point tile by
// two cooperating waves of one block, with the Runge-Kutta stage combination
// as epilogue.
//
// Lane l of both waves holds the same point.
//   metric wave: the stencils of h_ij; the inverse metric, Delta, the Ricci
//     tensor and what d_k (Dbar_j beta^j) needs of gammabar; after the
//     barrier Eqs. 7 and 8. It stores h_ij and a_ij.
//   gauge wave: the stencils of W, alpha, vet^i, lambda^i and K and the
//     advection of B^i and a_ij; after the barrier Eqs. 9, 10, 11, 13, 14, 15.
//     It stores the other twelve.
// What bounds it: the latency of a wave's own loads, LDS reads and arithmetic,
// so the aim is two waves per SIMD, each within 256 registers and half of
// 40 KB of LDS (four blocks, eight waves, per CU). On large grids loads queue
// for the L2s as well (rhs_stencil.h): on the 256 x 128 x 64 grid a wave issues
// vector arithmetic in 18% of its cycles and waits for memory or LDS in 35%, at
// 8th order in 12% and 44%. The split keeps about 60 values per point in each
// wave; what the waves exchange and the stencil stages share 80 LDS slots per
// point (slot v of lane l at xs[v * 64 + l]). One wave per tile and SIMD with
// the algebra in coordinate components took 19.2 us for a right-hand side on the
// 128 x 2 x 256 head-on grid, 954 us on a 256 x 128 x 64 one and 2.44 ms there
// at 8th order with dissipation; this form takes 13.0 us, 641 us and 1.29 ms.
#pragma once

#include "rhs_stencil.h"

namespace bhah {

enum {
  // metric -> gauge
  X_DEL = 0,   // 18 Delta^k_ij at X_DEL + 6 k + sy(i, j)
  X_DU = 18,   // 3  Delta^k
  X_PSI = 21,  // 3  psi_m = 1/2 gammabar^ab e_m h_ab = Delta^k_km
  X_Q = 24,    // 3  v^m d_k d_m psi in frame scaling
  // gauge -> metric
  X_V = 27,    // 9  e_k vet^i at X_V + 3 k + i
  X_L = 36,    // 9  e_k lambda^i at X_L + 3 k + i
  X_Y = 45,    // 6  second-derivative terms of alpha and W in Eq. 8
  X_U = 51,    // 3  2 alpha phi_k + alpha_k
  X_A = 54,    // 6  advection (and dissipation) of a_ij
  X_LATE = 72,   // 8  a_ij, K, alpha: in the gauge wave's stencil stage, after its stencils
  X_PARK = 60,   // the metric wave's park during its stencils, below the gauge wave's stencil stage
  X_SLOTS = 80,
  // results (12 per wave) take slots that neither wave reads any more
  R_METRIC = X_V, R_GAUGE = X_PARK
};

// Stencil stages: the metric wave's takes slots 0.. (its exchange slots, which
// it writes only after its stencils), the gauge wave's the last ones. The
// metric wave parks e_k h_ij and the advection of h_ij in what is left.
template <bool AX, int H>
struct Stage : StageSize<AX, H> {
  using StageSize<AX, H>::SL;
  static constexpr int GAUGE = X_SLOTS - SL, LOW = X_V - SL;
  static constexpr int CAP = LOW + GAUGE - X_PARK;  // park slots
  static_assert(LOW >= 0 && GAUGE >= X_PARK && GAUGE <= X_LATE, "stages");
  static constexpr int park(int i) { return i < LOW ? SL + i : X_PARK + i - LOW; }
};

// ---- epilogue: the right-hand side or the Runge-Kutta stage combination -------
// of the wave's twelve gridfunctions list[], results in park[(i) * 64].
// Every base value is read before any result is stored. Within a stage the
// arrays never overlap but at the same point (RK4: y, A, B, C into A, B, C or
// y; SSPRK3 mixes y with A or B into B or y), but the compiler cannot know it
// and would otherwise put each load behind the stores before it.
// Row pairs: where all 64 lanes are live and lanes 2p, 2p+1 hold adjacent
// points of one row, lane l takes points 2p and 2p+1, p = l mod 32, of
// gridfunction list[2 i + l / 32], one 16-byte access for two gridfunctions
// and two points: half the vector memory instructions of the per-lane form.
typedef double bhah_d2 __attribute__((ext_vector_type(2)));

// a value of V from and to the caller's arrays, which are aligned to 8 bytes
// (an alignment given to a type is lost where the type is a template argument,
// so it stands at the access)
typedef double bhah_d2_8 __attribute__((ext_vector_type(2), aligned(8)));
template <class V>
__device__ __forceinline__ V load_v(const double* p) {
  if constexpr (std::is_same_v<V, double>) return *p;
  else return *(const bhah_d2_8*)p;
}
__device__ __forceinline__ void store_v(double* p, double v) { *p = v; }
__device__ __forceinline__ void store_v(double* p, bhah_d2 v) { *(bhah_d2_8*)p = v; }

// V: double (per lane, twelve results) or bhah_d2 (row pairs, six); e(i) is
// the element of result i, res(i) its place in the park (for row pairs an even
// one: aligned to 16 bytes). With keep the stored values replace the results
// there.
template <class V, int N, class E, class RES>
__device__ __forceinline__ void store_stage(const StageArgs& st, bool keep, const E& e, const RES& res) {
  auto each = [](const V& k, auto f) {
    if constexpr (std::is_same_v<V, double>) return f(k, 0);
    else return V{f(k.x, 0), f(k.y, 1)};
  };
  auto el = [](const V& v, int h) {
    if constexpr (std::is_same_v<V, double>) return v;
    else return h ? v.y : v.x;
  };
  auto ld = [&](const double* b, V(&x)[N]) {
#pragma unroll
    for (int i = 0; i < N; i++) x[i] = load_v<V>(b + e(i));
  };
  auto k = [&](int i) -> V& { return *(V*)res(i); };
  if (st.rhs) {
#pragma unroll
    for (int i = 0; i < N; i++) store_v(st.rhs + e(i), k(i));
    return;
  }
  V b1[N], o[N];
  ld(st.base1, b1);
  if (st.base4) {
    V b2[N], b3[N], b4[N];
    ld(st.base2, b2);
    ld(st.base3, b3);
    ld(st.base4, b4);
    BHAH_PHASE_BARRIER();
#pragma unroll
    for (int i = 0; i < N; i++)
      o[i] = each(k(i), [&](double x, int h) {
        return combine_rk4(st, x, el(b1[i], h), el(b2[i], h), el(b3[i], h), el(b4[i], h));
      });
  } else if (st.base2) {
    V b2[N];
    ld(st.base2, b2);
    BHAH_PHASE_BARRIER();
#pragma unroll
    for (int i = 0; i < N; i++)
      o[i] = each(k(i), [&](double x, int h) { return combine_mix(st, x, el(b1[i], h), el(b2[i], h)); });
  } else {
    BHAH_PHASE_BARRIER();
#pragma unroll
    for (int i = 0; i < N; i++) o[i] = each(k(i), [&](double x, int h) { return combine_plain(st, x, el(b1[i], h)); });
  }
#pragma unroll
  for (int i = 0; i < N; i++) store_v(st.out + e(i), o[i]);
  if (keep) {
#pragma unroll
    for (int i = 0; i < N; i++) k(i) = o[i];
  }
}

// Ghosts g0 .. g1 - 1 of the pushed list from the tile's stored values
// (val[i * 64 + lane] of gridfunction list[i]): the sum of weights times
// values in the order of the ghost lists, then the parity sign, as the ghost
// kernel forms them. A separate kernel for the few thousand ghosts of a stage
// takes 4.5 to 5 us, most of it launch and three dependent rounds of loads.
// (Fetching a tile's range and first records before the last phase, to hide
// their latency, costs 200 to 400 bytes of spills and 20% of the step.)
__device__ __forceinline__ void push_ghosts(const GridDev& G, const PushDev& P, int g0, int g1, double* out,
                                            const int (&list)[12], const double* val, int lane) {
  for (int t = g0 + lane; t < g1; t += 64) {
    const int4 r = ((const int4*)P.rec)[t];
    const int par = r.y & 7;
    double x[12];
    if (r.y & 32) {
      const int n = r.y >> 8;
#pragma unroll
      for (int i = 0; i < 12; i++) x[i] = 0.0;
      for (int k = 0; k < n; k++) {
        const int2 lw = ((const int2*)P.terms)[r.z + k];
#pragma unroll
        for (int i = 0; i < 12; i++) x[i] = fma((double)lw.y, val[i * 64 + lw.x], x[i]);
      }
    } else if ((r.y >> 3) == 1) {
#pragma unroll
      for (int i = 0; i < 12; i++) x[i] = val[i * 64 + (r.z & 63)];
    } else {
#pragma unroll
      for (int i = 0; i < 12; i++) x[i] = 0.0;
#pragma unroll
      for (int k = 0; k < 3; k++) {
        const double w = (double)(signed char)(r.w >> (8 * k));
        const double* v = val + ((r.z >> (6 * k)) & 63);
#pragma unroll
        for (int i = 0; i < 12; i++) x[i] = fma(w, v[i * 64], x[i]);
      }
    }
#pragma unroll
    for (int i = 0; i < 12; i++) out[list[i] * G.sgf + r.x] = gf_flip(list[i], par) ? -x[i] : x[i];
  }
}

template <int C, int H, bool PUSH>
__device__ __forceinline__ void stage_epilogue(const GridDev& G, const StageArgs& st, const PushDev& P,
                                               const TilePoint& p, const int (&list)[12], double* __restrict__ park,
                                               int lane) {
  const unsigned q = p.q;
  const bool live = p.live;
  int g0 = 0, g1 = 0;  // the tile's pushed ghosts
  if (PUSH && P.start) {
    const int n = patch_number<C, H>(P, p.t0, p.t1, p.t2);
    g0 = P.start[n];
    g1 = P.start[n + 1];
  }
  const bool push = g0 < g1;
  wave_fence();  // the row pairs take other lanes' results
  const int p2 = 2 * (lane & 31), gs = lane >> 5;
  const unsigned qa = (unsigned)__shfl((int)q, p2), qb = (unsigned)__shfl((int)q, p2 + 1);
  if (__all(live && qb == qa + 1u)) {
    double* pk = park - lane + p2 + gs * 64;  // result 2 i + gs of point p2 at pk[128 i]
    long long e[6];
#pragma unroll
    for (int i = 0; i < 6; i++) e[i] = (gs ? list[2 * i + 1] : list[2 * i]) * G.sgf + (long long)qa;
    store_stage<bhah_d2, 6>(st, push, [&](int i) { return e[i]; }, [&](int i) { return pk + 128 * i; });
  } else if (live) {
    store_stage<double, 12>(st, push, [&](int i) { return list[i] * G.sgf + q; }, [&](int i) { return park + i * 64; });
  }
  if (push) {
    wave_fence();
    push_ghosts(G, P, g0, g1, st.out, list, park - lane, lane);
  }
}

// ---- metric wave ---------------------------------------------------------------
template <int C, bool AX, bool KO, int H, bool PUSH>
__device__ __forceinline__ void metric_wave(const GridDev& G, const Gauge& ga, const double* __restrict__ y,
                                            const StageArgs& st, const PushDev& P, const TilePoint& p,
                                            double* __restrict__ aux, double* __restrict__ xs0, int lane) {
  constexpr int PD = C == BHAH_SINH_CYLINDRICAL ? 1 : 2;
  double* xs = xs0 + lane;
  auto put = [&](int v, double x) { xs[v * 64] = x; };
  auto get = [&](int v) { return xs[v * 64]; };
  auto at = [&](int g) { return gf_ld(y, G.sgf, g, p.q * 8u, 0); };
  const auto S = make_source<C, AX, H>(y, G, p, lane, xs0);
  using ST = Stage<AX, H>;
  // values at the point itself come from the stencil stage where the wave takes
  // the gridfunction through it, others are read once (late: what the park cannot take)
  double gU[6], Pc[6], ck[6], h[6], v[3], late[24];
  auto keep = [&](int i, double x) {
    if (i < ST::CAP) put(ST::park(i), x);
    else late[i] = x;
  };
  auto kept = [&](int i) { return i < ST::CAP ? get(ST::park(i)) : late[i]; };
  {
    Coefs<H> c;
    double w[6], gd[6];
    {
#pragma unroll
      for (int a = 0; a < 6; a++) h[a] = at(G_HDD00 + a);
#pragma unroll
      for (int i = 0; i < 3; i++) v[i] = at(G_VETU0 + i);
      const Frame F = load_frame<C>(G, p.i0, p.i1, p.i2);
      metric_inverse(h, gU);
      make_coefs<KO, H>(G, ga, F.iS, v, c);
    }
    doubled(gU, gd);
#pragma unroll
    for (int k = 0; k < 3; k++)
#pragma unroll
      for (int l = k; l < 3; l++) w[sy(k, l)] = gd[sy(k, l)] * c.sc(k, l);
#pragma unroll
    for (int a = 0; a < 6; a++) { Pc[a] = 0.0; ck[a] = 0.0; }
    constexpr int list[6] = {G_HDD00, G_HDD00 + 1, G_HDD00 + 2, G_HDD00 + 3, G_HDD00 + 4, G_HDD00 + 5};
    //   Pc_ij = gammabar^kl h_ij,kl,  ck_kl = gammabar^ab h_ab,kl (unscaled)
    run_stencils<C, AX, H, 0, 6, 6, true>(S, list, [&](int a, const AxisSums(&s)[3], const double(&dd)[6],
                                                       double c0) BHAH_INLINE {
      h[a] = c0;
      pin(h[a]);
#pragma unroll
      for (int k = 0; k < 3; k++)
        if (!(AX && k == PD)) keep(3 * a + k, c.s1[k] * s[k].d1);
      keep(18 + a, advect<H>(s, c.ch, c.q));
#pragma unroll
      for (int kl = 0; kl < 6; kl++) {
        Pc[a] = fma(w[kl], dd[kl], Pc[a]);
        ck[kl] = fma(gd[a], dd[kl], ck[kl]);
        if (!zero_pair<AX, PD>(kl)) pin(ck[kl]);
      }
      pin(Pc[a]);
    });
#pragma unroll
    for (int k = 0; k < 3; k++)
#pragma unroll
      for (int l = k; l < 3; l++) ck[sy(k, l)] *= c.sc(k, l);
  }
  BHAH_PHASE_BARRIER();
  double adv[6], hk[3][6];
#pragma unroll
  for (int a = 0; a < 6; a++) {
    adv[a] = kept(18 + a);
#pragma unroll
    for (int k = 0; k < 3; k++) hk[k][a] = AX && k == PD ? 0.0 : kept(3 * a + k);
  }
  const Frame F = load_frame<C>(G, p.i0, p.i1, p.i2);
  // for the last phase: fetched there, they would wait behind the loads and
  // stores of the other waves' epilogues
  double lam[3];
#pragma unroll
  for (int i = 0; i < 3; i++) lam[i] = at(G_LAMU0 + i);
  const double W = at(G_CF);
  BHAH_PHASE_BARRIER();
  // psi = 1/2 ln det(gammabar/gammahat): psi_m = 1/2 gammabar^ab h_ab,m and
  // v^m psi_km = 1/2 (v^m gammabar^ab h_ab,km - (gammabar^-1 v^m h_m gammabar^-1)^ab h_ab,k)
  {
    double gd[6], hb[6], M[3][3], N[6], Nd[6];
    doubled(gU, gd);
#pragma unroll
    for (int m = 0; m < 3; m++) put(X_PSI + m, 0.5 * dot6(gd, hk[m]));
#pragma unroll
    for (int c = 0; c < 6; c++) hb[c] = fma(v[2], hk[2][c], fma(v[1], hk[1][c], v[0] * hk[0][c]));
    raise_first(gU, hb, M);
    raise_second(gU, M, N);
    doubled(N, Nd);
#pragma unroll
    for (int k = 0; k < 3; k++) {
      double s = v[0] * ck[sy(k, 0)];
      s = fma(v[1], ck[sy(k, 1)], s);
      s = fma(v[2], ck[sy(k, 2)], s);
      put(X_Q + k, 0.5 * (s - dot6(Nd, hk[k])));
    }
  }
  BHAH_PHASE_BARRIER();
  double D[3][6];  // Dhat_k h_ij
  cov_deriv<C, 6>(F, h, hk, D);
  double Rc[6];
  {
    const Lower L = lower_terms<C>(F, gU);
    add_lower<C, 6>(F, L, gU, h, hk, D, Pc);
#pragma unroll
    for (int c = 0; c < 6; c++) Rc[c] = -0.5 * Pc[c];
  }
  BHAH_PHASE_BARRIER();
  double DU[3];
  {
    double gd[6];
    doubled(gU, gd);
#pragma unroll
    for (int k = 0; k < 3; k++) {
      double Dk[6];
#pragma unroll
      for (int c = 0; c < 6; c++) Dk[c] = 0.0;
#pragma unroll
      for (int l = 0; l < 3; l++) {
        double low[6];
        delta_lower(D, l, low);
#pragma unroll
        for (int c = 0; c < 6; c++) Dk[c] = fma(gU[sy(k, l)], low[c], Dk[c]);
      }
#pragma unroll
      for (int c = 0; c < 6; c++) put(X_DEL + 6 * k + c, Dk[c]);
      DU[k] = dot6(gd, Dk);
      put(X_DU + k, DU[k]);
    }
  }
  BHAH_PHASE_BARRIER();
  add_ricci_delta(gU, D, DU, [&](int k, int c) { return get(X_DEL + 6 * k + c); }, Rc);
  __syncthreads();

  // ---- Lambdabar part of the Ricci tensor, Eq. 8's X_ij -------------------
  {
    double lk[3][3], Dl[3][3];
#pragma unroll
    for (int k = 0; k < 3; k++)
#pragma unroll
      for (int i = 0; i < 3; i++) lk[k][i] = AX && k == PD ? 0.0 : get(X_L + 3 * k + i);
    cov_deriv<C, 3>(F, lam, lk, Dl);
    add_ricci_lambda(h, Dl, Rc);
  }
  if (aux && p.live) {
#pragma unroll
    for (int c = 0; c < 6; c++) aux[c * G.sgf + p.q] = Rc[c];
    // Q_k = (d_k Gammabar^j_jm) beta^m in logical coordinates: beta^m d_k d_m
    // of ln(S_0 S_1 S_2) + psi
    const double* t0 = G.tab0 + p.i0 * TAB_W;
    const double r1 = t0[1] * t0[4], l0 = t0[2] * t0[5];  // r'/r, r''/r'
    const double n = C == BHAH_SINH_CYLINDRICAL ? 1.0 : 2.0;
    double dl[3] = {t0[3] * t0[5] - l0 * l0 + n * (t0[2] * t0[4] - r1 * r1), 0.0, 0.0};
    if constexpr (C == BHAH_SINH_CYLINDRICAL) {
      const double* t2 = G.tab2 + p.i2 * TAB_W;
      const double l2 = t2[2] * t2[5];
      dl[2] = t2[3] * t2[5] - l2 * l2;
    } else {
      const double* t1 = G.tab1 + p.i1 * TAB_W;
      dl[1] = -(t1[2] * t1[2]);
    }
#pragma unroll
    for (int k = 0; k < 3; k++)
      aux[(6 + k) * G.sgf + p.q] = v[k] * F.iS[k] * dl[k] + get(X_Q + k) / F.iS[k];
  }
  BHAH_PHASE_BARRIER();
  double a6[6];
#pragma unroll
  for (int c = 0; c < 6; c++) a6[c] = get(X_LATE + c);
  const double K = get(X_LATE + 6), alpha = get(X_LATE + 7);
  double X[6], L[3][3], Dv[3][3], div = 0.0;
#pragma unroll
  for (int c = 0; c < 6; c++) X[c] = fma(alpha, Rc[c], get(X_Y + c));
#pragma unroll
  for (int k = 0; k < 3; k++) {
    const double u = get(X_U + k);
#pragma unroll
    for (int c = 0; c < 6; c++) X[c] = fma(get(X_DEL + 6 * k + c), u, X[c]);
  }
  {
    double vk[3][3];
#pragma unroll
    for (int k = 0; k < 3; k++)
#pragma unroll
      for (int i = 0; i < 3; i++) vk[k][i] = AX && k == PD ? 0.0 : get(X_V + 3 * k + i);
    cov_deriv<C, 3>(F, v, vk, Dv);
    lie_matrix<C>(F, v, vk, Dv, L);
#pragma unroll
    for (int k = 0; k < 3; k++) div = fma(get(X_PSI + k), v[k], div + Dv[k][k]);
  }
  double AUD[3][3], gd[6];
  raise_first(gU, a6, AUD);
  doubled(gU, gd);
  const double trX3 = (1.0 / 3.0) * dot6(gd, X), W2 = W * W;
  const double trA = AUD[0][0] + AUD[1][1] + AUD[2][2];
  const double fA = fma(alpha, K, -(2.0 / 3.0) * div), fh = (2.0 / 3.0) * fma(alpha, trA, -div);
  double ra[6], rh[6];
#pragma unroll
  for (int i = 0; i < 3; i++)
#pragma unroll
    for (int j = i; j < 3; j++) {
      const int c = sy(i, j);
      const double gb = i == j ? 1.0 + h[c] : h[c];
      // Eq. 8
      double AA = a6[sy(i, 0)] * AUD[0][j];
      AA = fma(a6[sy(i, 1)], AUD[1][j], AA);
      AA = fma(a6[sy(i, 2)], AUD[2][j], AA);
      double r = fma(fA, a6[c], get(X_A + c));
      r = fma(-2.0 * alpha, AA, r);
      r = fma(W2, fma(-gb, trX3, X[c]), r);
      add_lie(L, a6, i, j, r);
      ra[c] = r;
      // Eq. 7
      r = fma(fh, gb, adv[c]) + (Dv[i][j] + Dv[j][i]);
      r = fma(-2.0 * alpha, a6[c], r);
      add_lie(L, h, i, j, r);
      rh[c] = r;
    }
  BHAH_PHASE_BARRIER();
#pragma unroll
  for (int c = 0; c < 6; c++) {
    put(R_METRIC + c, ra[c]);
    put(R_METRIC + 6 + c, rh[c]);
  }
  constexpr int out[12] = {0, 1, 2, 3, 4, 5, G_HDD00, G_HDD00 + 1, G_HDD00 + 2, G_HDD00 + 3, G_HDD00 + 4, G_HDD00 + 5};
  stage_epilogue<C, H, PUSH>(G, st, P, p, out, xs + R_METRIC * 64, lane);
}

// ---- gauge wave ------------------------------------------------------------------
template <int C, bool AX, bool KO, int H, bool PUSH>
__device__ __forceinline__ void gauge_wave(const GridDev& G, const Gauge& ga, const double* __restrict__ y,
                                           const StageArgs& st, const PushDev& P, const TilePoint& p,
                                           double* __restrict__ xs0, int lane) {
  constexpr int PD = C == BHAH_SINH_CYLINDRICAL ? 1 : 2;
  double* xs = xs0 + lane;
  auto put = [&](int v, double x) { xs[v * 64] = x; };
  auto get = [&](int v) { return xs[v * 64]; };
  auto at = [&](int g) { return gf_ld(y, G.sgf, g, p.q * 8u, 0); };
  const auto S = make_source<C, AX, H>(y, G, p, lane, xs0 + Stage<AX, H>::GAUGE * 64);
  double gU[6], Y[6], Za = 0.0, Bv[3], Bd[3], ak[3], phi[3], Kk[3];
  double advW = 0.0, advAl = 0.0, advK = 0.0, advV[3], advL[3], advB[3], koL[3];
  double v[3], lam[3], bet[3], a6[6], K = 0.0;  // values at the point, from the stencil stage
#pragma unroll
  for (int i = 0; i < 3; i++) { Bv[i] = 0.0; Bd[i] = 0.0; koL[i] = 0.0; }
  const double alpha = at(G_ALPHA), W = at(G_CF);
  {
    Coefs<H> c;
    double w[6];
    {
      double h[6];
#pragma unroll
      for (int a = 0; a < 6; a++) h[a] = at(G_HDD00 + a);
#pragma unroll
      for (int i = 0; i < 3; i++) v[i] = at(G_VETU0 + i);
      const Frame F = load_frame<C>(G, p.i0, p.i1, p.i2);
      metric_inverse(h, gU);
      make_coefs<KO, H>(G, ga, F.iS, v, c);
    }
    doubled(gU, w);
#pragma unroll
    for (int k = 0; k < 3; k++)
#pragma unroll
      for (int l = k; l < 3; l++) w[sy(k, l)] *= c.sc(k, l);
    const double iW = 1.0 / W, aW = alpha * iW;
    // the gridfunctions with second derivatives come while few results wait in
    // registers, those whose values wait as well last
    constexpr int list[18] = {G_VETU0, G_VETU0 + 1, G_VETU0 + 2, G_CF, G_ALPHA, G_LAMU0, G_LAMU0 + 1, G_LAMU0 + 2,
                              G_TRK, G_BETU0, G_BETU0 + 1, G_BETU0 + 2, 0, 1, 2, 3, 4, 5};
    run_stencils<C, AX, H, 0, 5, 9, true>(S, list, [&](int t, const AxisSums(&s)[3], const double(&dd)[6],
                                                       double c0) BHAH_INLINE {
      const bool gauge = t < 3 || t == 4 || (t >= 9 && t < 12);
      const double adv = gauge ? advect<H>(s, c.ch, c.qg) : advect<H>(s, c.ch, c.q);
      double d[3];
#pragma unroll
      for (int k = 0; k < 3; k++) d[k] = AX && k == PD ? 0.0 : c.s1[k] * s[k].d1;
      if (t >= 12) {  // a_ij
        put(X_A + t - 12, adv);
        a6[t - 12] = c0;
        pin(a6[t - 12]);
      } else if (t < 3) {  // vet^i
        const int i = t;
        advV[i] = adv;
        v[i] = c0;
        pin(v[i]);
#pragma unroll
        for (int k = 0; k < 3; k++)
          if (!(AX && k == PD)) put(X_V + 3 * k + i, d[k]);
#pragma unroll
        for (int kl = 0; kl < 6; kl++) Bv[i] = fma(w[kl], dd[kl], Bv[i]);
#pragma unroll
        for (int k = 0; k < 3; k++) Bd[k] = fma(c.sc(k, i), dd[sy(k, i)], Bd[k]);
        pin(Bv[i]);
        pin(advV[i]);
        pin(Bd[0]);
        pin(Bd[3 - PD]);
      } else if (t == 3) {  // W
        advW = adv;
#pragma unroll
        for (int k = 0; k < 3; k++) phi[k] = (-0.5 * iW) * d[k];
#pragma unroll
        for (int kl = 0; kl < 6; kl++) {
          Y[kl] = aW * dd[kl];
          if (!zero_pair<AX, PD>(kl)) pin(Y[kl]);
        }
        pin(advW);
      } else if (t == 4) {  // alpha
        advAl = adv;
#pragma unroll
        for (int k = 0; k < 3; k++) {
          ak[k] = d[k];
#pragma unroll
          for (int l = k; l < 3; l++) {
            const int kl = sy(k, l);
            Y[kl] = (Y[kl] - dd[kl]) * c.sc(k, l);
            Za = fma(w[kl], dd[kl], Za);
            if (!zero_pair<AX, PD>(kl)) pin(Y[kl]);
          }
        }
        pin(Za);
        pin(advAl);
      } else if (t < 8) {  // lambda^i
        const int i = t - 5;
        advL[i] = adv;
        lam[i] = c0;
        pin(lam[i]);
#pragma unroll
        for (int k = 0; k < 3; k++)
          if (!(AX && k == PD)) put(X_L + 3 * k + i, d[k]);
        if constexpr (KO) {  // kept apart: B^i takes 3/4 of lambda^i's undissipated right-hand side
          double o = 0.0;
#pragma unroll
          for (int k = 0; k < 3; k++) o = fma(c.kw[k], s[k].K, o);
          koL[i] = ga.dm * o;
          pin(koL[i]);
        }
        pin(advL[i]);
      } else if (t == 8) {  // K
        advK = adv;
        K = c0;
        pin(K);
#pragma unroll
        for (int k = 0; k < 3; k++) Kk[k] = d[k];
        pin(advK);
      } else {  // B^i
        advB[t - 9] = adv;
        pin(advB[t - 9]);
        bet[t - 9] = c0;
        pin(bet[t - 9]);
      }
    });
  }
  BHAH_PHASE_BARRIER();
#pragma unroll
  for (int c = 0; c < 6; c++) put(X_LATE + c, a6[c]);
  put(X_LATE + 6, K);
  put(X_LATE + 7, alpha);
  const Frame F = load_frame<C>(G, p.i0, p.i1, p.i2);
  BHAH_PHASE_BARRIER();
  {
    // alpha W_ij/W - alpha_ij + its lower terms + 2 (alpha_i phi_j + alpha_j phi_i);
    // the terms alpha W_i W_j / W^2 and 4 alpha phi_i phi_j of Eq. 8 cancel
    double f[3];
#pragma unroll
    for (int k = 0; k < 3; k++) {
      const double u = fma(2.0 * alpha, phi[k], ak[k]);
      f[k] = -u;
      put(X_U + k, u);
    }
    add_hessian_lower<C>(F, f, Y);
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
      for (int j = i; j < 3; j++) put(X_Y + sy(i, j), fma(2.0, fma(ak[i], phi[j], ak[j] * phi[i]), Y[sy(i, j)]));
  }
  // gammabar^jk Dhat_j Dhat_k beta^i
  double vk[3][3], Dv[3][3];
#pragma unroll
  for (int k = 0; k < 3; k++)
#pragma unroll
    for (int i = 0; i < 3; i++) vk[k][i] = AX && k == PD ? 0.0 : get(X_V + 3 * k + i);
  cov_deriv<C, 3>(F, v, vk, Dv);
  const Lower Lw = lower_terms<C>(F, gU);
  add_lower<C, 3>(F, Lw, gU, v, vk, Dv, Bv);
  // d_k (Dhat_j beta^j)
  const double a = F.a, b = F.b;
  if constexpr (C == BHAH_SINH_CYLINDRICAL) {
    Bd[0] = fma(-a, vk[1][1], fma(-F.s0, vk[0][0], Bd[0]));
    Bd[2] = fma(-F.s2, vk[2][2], Bd[2]);
#pragma unroll
    for (int k = 0; k < 3; k++) Bd[k] = fma(a, vk[k][0], Bd[k]);
    Bd[0] = fma(-(a * a), v[0], Bd[0]);
  } else {
    Bd[0] = fma(-a, vk[1][1] + vk[2][2], fma(-F.s0, vk[0][0], Bd[0]));
    Bd[1] = fma(-b, vk[2][2], Bd[1]);
#pragma unroll
    for (int k = 0; k < 3; k++) Bd[k] = fma(b, vk[k][1], fma(a + a, vk[k][0], Bd[k]));
    Bd[0] = fma(-a, fma(a + a, v[0], b * v[1]), Bd[0]);
    Bd[1] = fma(-fma(a, a, b * b), v[1], Bd[1]);
  }
  __syncthreads();

  double L[3][3], psi[3], DU[3], div = 0.0;
  lie_matrix<C>(F, v, vk, Dv, L);
#pragma unroll
  for (int k = 0; k < 3; k++) {
    psi[k] = get(X_PSI + k);
    DU[k] = get(X_DU + k);
    div = fma(psi[k], v[k], div + Dv[k][k]);
  }
  double AUU[6], AA;
  {
    double AUD[3][3], w[6];
    raise_first(gU, a6, AUD);
    raise_second(gU, AUD, AUU);
    doubled(AUU, w);
    AA = dot6(w, a6);
  }
  double rl[3];
#pragma unroll
  for (int i = 0; i < 3; i++) {
    double t = 0.0;
#pragma unroll
    for (int j = 0; j < 3; j++)
#pragma unroll
      for (int k = j; k < 3; k++)
        t = fma((j == k ? 1.0 : 2.0) * AUU[sy(j, k)], get(X_DEL + 6 * i + sy(j, k)), t);
    rl[i] = fma(2.0 * alpha, t, Bv[i]);
  }
  double q[3];
#pragma unroll
  for (int k = 0; k < 3; k++) q[k] = get(X_Q + k);
  BHAH_PHASE_BARRIER();
  // Eq. 10 (K), Eq. 9 (W), Eq. 13 (alpha)
  double rK;
  {
    double lap = Za, dd = 0.0;
#pragma unroll
    for (int i = 0; i < 3; i++) {
      lap = fma(Lw.n[i] - DU[i], ak[i], lap);
      double u = gU[sy(i, 0)] * ak[0];
      u = fma(gU[sy(i, 1)], ak[1], u);
      u = fma(gU[sy(i, 2)], ak[2], u);
      dd = fma(u, phi[i], dd);
    }
    const double aK = alpha * K;
    rK = fma((1.0 / 3.0) * aK, K, advK);
    rK = fma(alpha, AA, rK);
    rK = fma(-(W * W), fma(2.0, dd, lap), rK);
    put(R_GAUGE + 8, rK);
    put(R_GAUGE + 4, fma(-(1.0 / 3.0) * W, div - aK, advW));
    put(R_GAUGE + 0, fma(-2.0, aK, advAl));
  }
  // Eq. 11 (Lambdabar), Eqs. 14-15 (shift, B)
  double z[3];  // 1/3 d_j (Dbar_k beta^k) - 4/3 alpha K_j, to be raised
#pragma unroll
  for (int k = 0; k < 3; k++) {
    // d_k (Dbar_j beta^j) = d_k (Dhat_j beta^j) + v^m psi_km + (v_k^m - sigma_km v^m) psi_m
    double s = Bd[k] + q[k];
#pragma unroll
    for (int m = 0; m < 3; m++) {
      double g = k == m ? vk[k][k] : L[k][m];
      if (k == m && k == 0) g = fma(-F.s0, v[0], g);
      if (C == BHAH_SINH_CYLINDRICAL && k == m && k == 2) g = fma(-F.s2, v[2], g);
      s = fma(g, psi[m], s);
    }
    z[k] = (1.0 / 3.0) * fma(-4.0 * alpha, Kk[k], s);
  }
  double bS[3];  // v^k e_k ln S_i
  bS[0] = v[0] * F.s0;
  bS[1] = v[0] * a;
  bS[2] = C == BHAH_SINH_CYLINDRICAL ? v[2] * F.s2 : fma(v[1], b, bS[1]);
#pragma unroll
  for (int i = 0; i < 3; i++) {
    double r = fma((2.0 / 3.0) * div, DU[i], rl[i]);
#pragma unroll
    for (int j = 0; j < 3; j++) {
      r = fma(gU[sy(i, j)], z[j], r);
      r = fma(-2.0 * AUU[sy(i, j)], fma(-6.0 * alpha, phi[j], ak[j]), r);
      r = fma(-lam[j], L[j][i], r);
    }
    r += advL[i];
    put(R_GAUGE + 5 + i, r);
    put(R_GAUGE + 1 + i, fma(0.75, KO ? r - koL[i] : r, advB[i]) - fma(bet[i], bS[i], ga.eta * bet[i]));
    put(R_GAUGE + 9 + i, fma(-v[i], bS[i], bet[i]) + advV[i]);
  }
  constexpr int out[12] = {G_ALPHA, G_BETU0, G_BETU0 + 1, G_BETU0 + 2, G_CF, G_LAMU0, G_LAMU0 + 1, G_LAMU0 + 2, G_TRK,
                           G_VETU0, G_VETU0 + 1, G_VETU0 + 2};
  stage_epilogue<C, H, PUSH>(G, st, P, p, out, xs + R_GAUGE * 64, lane);
}

// One tile by the block's two waves. Every lane takes part (lanes past the
// grid compute a point on it and store nothing). PUSH: with the tile's pushed
// ghosts.
template <int C, bool AX, bool KO, int H, bool PUSH>
__device__ __forceinline__ void rhs_tile(const GridDev& G, const TileMap& T, int w, const Gauge& ga,
                                         const double* __restrict__ y, const StageArgs& st, const PushDev& P,
                                         double* __restrict__ aux, double* __restrict__ xs) {
  const int lane = (int)(threadIdx.x & 63), wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  TilePoint p;
  p.live = tile_point<H>(G, T, w, lane, p.t0, p.t1, p.t2, p.i0, p.i1, p.i2);
  p.q = (unsigned)(p.i0 + G.s1 * p.i1 + G.s2 * p.i2);
  if (wave == 0) metric_wave<C, AX, KO, H, PUSH>(G, ga, y, st, P, p, aux, xs, lane);
  else gauge_wave<C, AX, KO, H, PUSH>(G, ga, y, st, P, p, xs, lane);
}

}  // namespace bhah
