// rhs_stencil.h -- the stencil side of the right-hand side (rhs_point.h) and
// the constraints (hamiltonian.hip): the stencil sums of one gridfunction,
// where its values come from (LDS patches of a tile, or per-lane loads), the
// loops over gridfunctions, and the tile walk.
#pragma once

#include <type_traits>
#include <utility>

#include "rhs_frame.h"

namespace bhah {

#define BHAH_PHASE_BARRIER() __builtin_amdgcn_sched_barrier(0)

// Keeps arithmetic where it is written: a scheduling barrier holds loads and
// stores, but arithmetic on loaded values would still sink to its last use
// and keep every operand in a register until there (at 8th order all 64
// values of a mixed pair). No instruction is emitted.
__device__ __forceinline__ void pin(double& x) { asm volatile("" : "+v"(x)); }

// Upwinded advection beta^k d_k f (Sec. 3: the centred stencil shifted one
// point upwind) as its antisymmetric and symmetric parts. With
// D_j = f_j - f_-j and S_j = (f_j - f_0) + (f_-j - f_0), for either sign of
// the shift component v,
//   den1 v U f = (v/2) sum_j ua[j] D_j + sk |v| sum_j ko[j] S_j,  j = 1..R+1,
// where sum_j ko[j] S_j is the difference of order 2R+2 that the
// Kreiss-Oliger term uses: its strength adds to sk |v|, so dissipation costs
// no stencil arithmetic of its own, and no value is selected by the sign of
// the shift. At 4th order (up = -3, -10, 18, -6, 1): D: 21, -6, 1 (halves),
// S: (f_3 + f_-3) - 6 (f_2 + f_-2) + 15 (f_1 + f_-1) - 20 f_0, sk = 1/2.
// D_j and S_j also give the first and second derivatives.
template <int R>
struct UpW;
template <>
struct UpW<2> {
  static constexpr double ua[4] = {0.0, 21.0, -6.0, 1.0}, sk = 0.5;
};
template <>
struct UpW<4> {
  static constexpr double ua[6] = {0.0, 1470.0, -480.0, 145.0, -30.0, 3.0}, sk = 1.5;
};

// f(0), f(1), .., f(N - 1) with the index as a compile-time constant (loops of
// this size are not always unrolled by the compiler, and a loop left over
// would index registers at run time)
template <class F, int... I>
__device__ __forceinline__ void static_for_(const F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(const F& f) {
  static_for_(f, std::make_integer_sequence<int, N>{});
}
#define BHAH_INLINE __attribute__((always_inline))

// raw sums of one gridfunction along one direction: den1 D f, den2 D2 f and
// the two parts of the upwinded sum (A: sum ua D_j, K: sum ko S_j)
struct AxisSums {
  double d1, d2, A, K;
};
// (first, second, ADV: whether d1, d2, and A and K are used at all)
template <bool ADV>
__device__ __forceinline__ void pin(AxisSums& s, bool first, bool second) {
  if (first) pin(s.d1);
  if (second) pin(s.d2);
  if constexpr (ADV) {
    pin(s.A);
    pin(s.K);
  }
}
template <int R>
__device__ __forceinline__ AxisSums axis_sums(const double (&v)[2 * R + 3]) {
  constexpr int H = R + 1;
  double D[H + 1], S[H + 1];
#pragma unroll
  for (int j = 1; j <= H; j++) {
    D[j] = v[H + j] - v[H - j];
    S[j] = (v[H + j] - v[H]) + (v[H - j] - v[H]);
  }
  AxisSums s;
  s.d1 = FdW<R>::d1[R] * D[R];
  s.d2 = FdW<R>::d2[R] * S[R];
#pragma unroll
  for (int j = R - 1; j >= 1; j--) {
    s.d1 = fma(FdW<R>::d1[j], D[j], s.d1);
    s.d2 = fma(FdW<R>::d2[j], S[j], s.d2);
  }
  s.A = UpW<R>::ua[H] * D[H];
  s.K = FdW<R>::ko[H] * S[H];
#pragma unroll
  for (int j = R; j >= 1; j--) {
    s.A = fma(UpW<R>::ua[j], D[j], s.A);
    s.K = fma(FdW<R>::ko[j], S[j], s.K);
  }
  return s;
}
// The same along phi on a grid with two phi planes: odd offsets land on the
// other plane (value o), even ones on the point's own (c), so D_j = 0 and the
// odd S_j are all 2 (o - c).
template <int R>
__device__ __forceinline__ AxisSums axis_sums_two_planes(double c, double o) {
  double kd2 = 0.0, kk = 0.0;
#pragma unroll
  for (int j = 1; j <= R; j += 2) kd2 += 2.0 * FdW<R>::d2[j];
#pragma unroll
  for (int j = 1; j <= R + 1; j += 2) kk += 2.0 * FdW<R>::ko[j];
  const double x = o - c;
  return AxisSums{0.0, kd2 * x, 0.0, kk * x};
}
// den1 D f from values v[R + m] = f(m), m = -R..R (v[R] is not used)
template <int R>
__device__ __forceinline__ double d1_sum(const double (&v)[2 * R + 1]) {
  double a = FdW<R>::d1[R] * (v[2 * R] - v[0]);
#pragma unroll
  for (int j = R - 1; j >= 1; j--) a = fma(FdW<R>::d1[j], v[R + j] - v[R - j], a);
  return a;
}

// ---- where stencil values come from ----------------------------------------
// A tile is a patch of EX points along i0 and EE along the other
// non-periodic direction e (i2 on SinhCylindrical grids, i1 otherwise) on one
// phi plane: 16 x 4. For one gridfunction at a time the wave brings the
// patch with its halo into LDS with 16-byte loads and takes every stencil
// value along i0 and e and of the mixed pair (0, e) from there. On grids with
// more than two phi planes the planes at phi offsets +-j follow in pairs, for
// the mixed pairs (0, phi) and (e, phi); values at phi offsets +-(R+1), and
// all phi offsets of gridfunctions without second derivatives, are read per
// lane. The CU's vector memory path takes about the same time for every load
// instruction whatever its width (16 cycles measured for 64 lanes), so what
// counts is the number of instructions: a 16 x 4 patch with its halo at 4th
// order is 22 x 10 values, two loads, where a row of 64 points would be 7 x
// 70, four, and per-lane gathers 30 to 70.
constexpr int TLX = PATCH_LX, TEX = PATCH_X, TEE = PATCH_E;
// row length and 16-byte pieces of the main patch (halo H) and of one pair of
// phi planes (halo R each)
template <int H>
struct Patch {
  static constexpr int R = H - 1;
  static constexpr int RL = TEX + 2 * H, RE = TEE + 2 * H, NP = RL * RE / 2, NR = (NP + 63) / 64;
  static constexpr int QL = TEX + 2 * R, QE = TEE + 2 * R, QN = QL * QE, QP = QN, QR = (QP + 63) / 64;
  static constexpr int MAIN = 2 * NP, PAIR = 2 * QN;  // doubles
};

// All accessors give f at offsets (d0, de) on the point's phi plane or on the
// plane at phi offset +-j, and the phi column of the point.
template <int H>
struct StagedSrc {
  static constexpr bool STG = true;
  using PG = Patch<H>;
  static constexpr int R = H - 1;
  const double* y;
  long long sgf;
  double* lds;         // the wave's stage: main patches, then a pair of phi planes
  unsigned voff[PG::NR], qoff[PG::QR];  // per-lane byte offsets of the lane's pieces
  int lane;
  unsigned vlane;      // per-lane byte offset of the point, phi index removed
  int sw[2 * H + 1];   // byte offsets of the (wrapped) phi planes at offsets -H..H, wave-uniform
  unsigned org;        // byte offset of the patch origin (halo H), phi index removed, wave-uniform
  int c0, q0;          // the point's place in the main patch and in a phi-plane patch

  // tile origin (it, et), point (i0, ie), phi index ip; sE, sP strides
  __device__ __forceinline__ void init(const double* y_, const GridDev& G, int pd, int it, int et, int i0, int ie,
                                       int ip, int lane_, double* lds_, bool two_planes) {
    y = y_;
    lane = lane_;
    sgf = G.sgf;
    lds = lds_;
    const int sP = pd == 1 ? G.s1 : G.s2, sE = pd == 1 ? G.s2 : G.s1, nP = pd == 1 ? G.N1 : G.N2;
    const int id = ip - H;
#pragma unroll
    for (int o = -H; o <= H; o++) {
      int x = id + o;
      if (two_planes) {
        x = (x + 2 * H) & 1;
      } else if constexpr (H == 3) {  // nP >= 2: two corrections each way suffice
        x += x < 0 ? nP : 0;
        x += x < 0 ? nP : 0;
        x -= x >= nP ? nP : 0;
        x -= x >= nP ? nP : 0;
      } else {
        x %= nP;
        x += x < 0 ? nP : 0;
      }
      sw[o + H] = (H + x) * sP * 8;
    }
    org = (unsigned)((it - H) + sE * (et - H)) * 8u;
    vlane = (unsigned)(i0 + sE * ie) * 8u;
#pragma unroll
    for (int r = 0; r < PG::NR; r++) {
      const int p = piece<PG::NP>(r), row = p / (PG::RL / 2), col = 2 * (p - row * (PG::RL / 2));
      voff[r] = (unsigned)(col + row * sE) * 8u;
    }
    if (!two_planes) {
#pragma unroll
      for (int r = 0; r < PG::QR; r++) {
        int p = piece<PG::QP>(r);
        if (far_plane(r)) p -= PG::QN / 2;
        const int row = p / (PG::QL / 2), col = 2 * (p - row * (PG::QL / 2));
        qoff[r] = (unsigned)((col + 1) + (row + 1) * sE) * 8u;  // halo R = H - 1
      }
    }
    c0 = (ie - et + H) * PG::RL + (i0 - it + H);
    q0 = (ie - et + R) * PG::QL + (i0 - it + R);
  }
  // the lane's r-th 16-byte piece of N; past the last one it repeats it, so
  // that every lane loads and stores in bounds
  template <int N>
  __device__ __forceinline__ int piece(int r) const {
    return (r + 1) * 64 <= N ? r * 64 + lane : min(r * 64 + lane, N - 1);
  }
  // whether it lies on the second plane (phi offset -j) of a pair
  __device__ __forceinline__ bool far_plane(int r) const {
    constexpr int half = PG::QN / 2;
    return (r + 1) * 64 <= half ? false : (r * 64 >= half ? true : r * 64 + lane >= half);
  }
  struct MainRegs {
    double lo[PG::NR], hi[PG::NR];
  };
  struct PairRegs {
    double lo[PG::QR], hi[PG::QR];
  };
  __device__ __forceinline__ void issue_main(int g, MainRegs& m) const {
#pragma unroll
    for (int r = 0; r < PG::NR; r++) gf_ld2(y, sgf, g, voff[r], (int)org + sw[H], m.lo[r], m.hi[r]);
  }
  __device__ __forceinline__ void commit_main(const MainRegs& m, int slot) const {
#pragma unroll
    for (int r = 0; r < PG::NR; r++) {
      lds[slot * PG::MAIN + 2 * piece<PG::NP>(r)] = m.lo[r];
      lds[slot * PG::MAIN + 2 * piece<PG::NP>(r) + 1] = m.hi[r];
    }
  }
  __device__ __forceinline__ void issue_pair(int g, int j, PairRegs& m) const {
#pragma unroll
    for (int r = 0; r < PG::QR; r++)
      gf_ld2(y, sgf, g, qoff[r] + (unsigned)(far_plane(r) ? sw[H - j] : sw[H + j]), (int)org, m.lo[r], m.hi[r]);
  }
  __device__ __forceinline__ void commit_pair(const PairRegs& m, int base) const {
#pragma unroll
    for (int r = 0; r < PG::QR; r++) {
      lds[base + 2 * piece<PG::QP>(r)] = m.lo[r];
      lds[base + 2 * piece<PG::QP>(r) + 1] = m.hi[r];
    }
  }
  __device__ __forceinline__ double main_at(int slot, int d0, int de) const {
    return lds[slot * PG::MAIN + c0 + de * PG::RL + d0];
  }
  __device__ __forceinline__ double pair_at(int base, int side, int d0, int de) const {
    return lds[base + side * PG::QN + q0 + de * PG::QL + d0];
  }
  // value in the point's phi column
  __device__ __forceinline__ double column(int g, int m) const { return gf_ld(y, sgf, g, vlane, sw[H + m]); }
};

// per-lane loads (tile shapes other than the staged patch)
template <int H>
struct GatherSrc {
  static constexpr bool STG = false;
  PtT<H> P;
  int pd;
  __device__ __forceinline__ double at(int g, int d0, int de, int dp) const {
    return pd == 1 ? P.at(g, d0, dp, de) : P.at(g, d0, de, dp);
  }
};

// Tiles: 64 points, 2^lx along i0 times 2^ly along i1 times 64 >> (lx + ly)
// along i2; the tile grid is walked in bands of `band` tile rows of i1, and
// within a band by i2, then i1, then i0 (fastest), so that tiles that share
// cache lines along i0 run at the same time. The hardware hands consecutive
// workgroup ids to the XCDs in turn; block ids are remapped so that every XCD
// works through one contiguous range of the walk (its L2 then holds a compact
// part of the grid). The lines matter more than the bytes: in columns of 64
// points the 3-D RK4 stage reads 2.4 GB instead of 4.2 GB through the L2s, but
// every column edge leaves lines that two tiles complete far apart in time
// (1.16x the write requests), and the step takes 3.90 ms instead of 3.66 ms
// (head-on 0.934 instead of 0.902 ms per 10 steps).
// (t0, t1, t2) is the tile's first point; (i0, i1, i2) the lane's, moved onto
// the grid where the tile runs past it (false is returned for such lanes).
template <int H>
__device__ __forceinline__ bool tile_point(const GridDev& G, const TileMap& T, int w, int lane, int& t0, int& t1,
                                           int& t2, int& i0, int& i1, int& i2) {
  const int full = T.band * T.tz * T.tx;  // tiles in one full band
  const int nb = (T.ty + T.band - 1) / T.band;
  int bi = w / full;
  if (bi > nb - 1) bi = nb - 1;
  const int start = bi * T.band;
  const int hgt = min(T.band, T.ty - start);
  const int idx = w - start * T.tz * T.tx;
  const int r = idx / T.tx;
  const int xt = idx - r * T.tx;
  const int j2 = r / hgt;
  const int j1 = start + (r - j2 * hgt);
  const int ex = 1 << T.lx, ey = 1 << T.ly;
  t0 = H + xt * ex;
  t1 = H + j1 * ey;
  t2 = H + (j2 << (6 - T.lx - T.ly));
  const int a = t0 + (lane & (ex - 1)), b = t1 + ((lane >> T.lx) & (ey - 1)), c = t2 + (lane >> (T.lx + T.ly));
  i0 = min(a, H + G.N0 - 1);
  i1 = min(b, H + G.N1 - 1);
  i2 = min(c, H + G.N2 - 1);
  return a == i0 && b == i1 && c == i2;
}

// logical position in the walk of the tile a block works on; with G_blocks a
// multiple of the XCD count, block b runs on XCD b % nxcd
__device__ __forceinline__ int xcd_remap(int b, int per) { return (b % BHAH_NXCD) * per + b / BHAH_NXCD; }

// a wave's stencil stage: PER main patches on grids with two phi planes (a
// batch of gridfunctions), else one main patch and a pair of phi planes
template <bool AX, int H>
struct StageSize {
  static constexpr int PER = AX && H == 3 ? 2 : 1;
  static constexpr int N = AX ? PER * Patch<H>::MAIN : Patch<H>::MAIN + Patch<H>::PAIR;  // doubles
  static constexpr int SL = (N + 63) / 64;                                              // slots of 64
};

// scales of the derivatives and upwind coefficients at a point
template <int H>
struct Coefs {
  double s1[3];  // e_k f = s1[k] * (den1 D f)
  double ch[3], q[3], qg[3];  // advection and dissipation: ch A + q K (metric strength), qg (gauge strength)
  double kw[3];
  // f_kl = sc(k, l) * raw second difference
  __device__ __forceinline__ double sc(int k, int l) const {
    constexpr double r = FdW<H - 1>::den1 * FdW<H - 1>::den1 / FdW<H - 1>::den2;
    return k == l ? s1[k] * s1[k] * r : s1[k] * s1[l];
  }
};
template <bool KO, int H>
__device__ __forceinline__ void make_coefs(const GridDev& G, const Gauge& ga, const double (&iS)[3],
                                           const double (&v)[3], Coefs<H>& c) {
  constexpr int R = H - 1;
  using W = FdW<R>;
#pragma unroll
  for (int k = 0; k < 3; k++) {
    c.s1[k] = iS[k] * (G.inv_dx[k] * (1.0 / W::den1));
    const double b = v[k] * c.s1[k];
    c.ch[k] = 0.5 * b;
    c.q[k] = c.qg[k] = UpW<R>::sk * fabs(b);
    if constexpr (KO) {
      c.kw[k] = G.inv_dx[k] * (1.0 / W::kden);
      c.qg[k] = fma(ga.dg, c.kw[k], c.q[k]);
      c.q[k] = fma(ga.dm, c.kw[k], c.q[k]);
    }
  }
}

template <int H>
__device__ __forceinline__ double advect(const AxisSums (&s)[3], const double (&ch)[3], const double (&q)[3]) {
  double a = 0.0;
#pragma unroll
  for (int k = 0; k < 3; k++) a = fma(ch[k], s[k].A, fma(q[k], s[k].K, a));
  return a;
}

// ---- stencil drivers ---------------------------------------------------------
// Runs over the gridfunctions list[0..N): for each, fn(t, axis sums
// along the three directions, raw second differences dd[sy(k, l)]); dd is
// formed for t in [F0, F1), first derivatives are used for t in [F0, F2), the
// upwinded sums where ADV.
// Identically vanishing phi derivatives of two-plane
// grids are literal zeros. The arithmetic is the same for both sources.
// whether d_k d_l, kl = sy(k, l), vanishes identically (mixed with phi on two planes)
template <bool AX, int PD>
__device__ __forceinline__ constexpr bool zero_pair(int kl) {
  return AX && (kl == sy(0, PD) || kl == sy(3 - PD, PD));
}
template <int R>
__device__ __forceinline__ double acc_pair(int j, double acc, double p, double m) {
  return j == 1 ? FdW<R>::d1[1] * (p - m) : fma(FdW<R>::d1[j], p - m, acc);
}

template <int C, bool AX, int H, int F0, int F1, int F2, bool ADV, int N, class FN>
__device__ __forceinline__ void run_stencils(const StagedSrc<H>& S, const int (&list)[N], const FN& fn) {
  constexpr int PD = C == BHAH_SINH_CYLINDRICAL ? 1 : 2, E = 3 - PD, R = H - 1;
  using SS_ = StagedSrc<H>;
  auto in_plane = [&](int slot, bool full, bool first, AxisSums(&s)[3], double (&dd)[6], double& c) BHAH_INLINE {
    double v0[2 * H + 1], vE[2 * H + 1];
#pragma unroll
    for (int m = -H; m <= H; m++) {
      v0[H + m] = S.main_at(slot, m, 0);
      vE[H + m] = m == 0 ? v0[H] : S.main_at(slot, 0, m);
    }
    c = v0[H];
    s[0] = axis_sums<R>(v0);
    s[E] = axis_sums<R>(vE);
    pin<ADV>(s[0], first, full);
    pin<ADV>(s[E], first, full);
    if (full) {
      if constexpr (H == 5) BHAH_PHASE_BARRIER();
      double e[2 * R + 1];
      e[R] = 0.0;
#pragma unroll
      for (int m = -R; m <= R; m++)
        if (m != 0) {
          double r[2 * R + 1];
          r[R] = 0.0;
#pragma unroll
          for (int n = -R; n <= R; n++)
            if (n != 0) r[R + n] = S.main_at(slot, n, m);
          e[R + m] = d1_sum<R>(r);
          pin(e[R + m]);
          if constexpr (H == 5) BHAH_PHASE_BARRIER();
        }
      dd[sy(0, E)] = d1_sum<R>(e);
      pin(dd[sy(0, E)]);
    }
  };
  if constexpr (AX) {
    constexpr int PER = StageSize<AX, H>::PER, NB = (N + PER - 1) / PER;
    typename SS_::MainRegs m[PER];
    double ph[PER];
    auto issue = [&](int b) {
#pragma unroll
      for (int t = 0; t < PER; t++)
        if (b * PER + t < N) {
          S.issue_main(list[b * PER + t], m[t]);
          ph[t] = S.column(list[b * PER + t], 1);
        }
    };
    issue(0);
    static_for<NB>([&](auto bc) BHAH_INLINE {
      constexpr int b = decltype(bc)::value;
      double o[PER];
#pragma unroll
      for (int t = 0; t < PER; t++)
        if (b * PER + t < N) {
          S.commit_main(m[t], t);
          o[t] = ph[t];
        }
      if constexpr (b + 1 < NB) issue(b + 1);
      BHAH_PHASE_BARRIER();
      static_for<PER>([&](auto tc) BHAH_INLINE {
        constexpr int t = decltype(tc)::value, tt = b * PER + t;
        if constexpr (tt < N) {
          AxisSums s[3];
          double dd[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, c;
          in_plane(t, tt >= F0 && tt < F1, tt >= F0 && tt < F2, s, dd, c);
          s[PD] = axis_sums_two_planes<R>(c, o[t]);
#pragma unroll
          for (int k = 0; k < 3; k++) dd[sy(k, k)] = s[k].d2;
          fn(tt, s, dd);
        }
      });
    });
  } else {
    constexpr int PB = SS_::PG::MAIN;  // the phi planes' place in the stage
    // Loads run one gridfunction ahead of their use. At 8th order, where a
    // gridfunction has four pairs of phi planes, one pair and then the next
    // main patch: more in flight spills (3-D production step 6.0 instead of
    // 5.2 ms); at 4th order deeper prefetch measures the same.
    constexpr int PS = H == 3 ? 2 : 1;
    typename SS_::MainRegs m;
    typename SS_::PairRegs pr[PS];
    double col[2 * H];  // phi offsets -H..-1, 1..H
    auto issue = [&](auto tc) BHAH_INLINE {
      constexpr int t = decltype(tc)::value;
      if constexpr (t < N) {
        S.issue_main(list[t], m);
#pragma unroll
        for (int o = 1; o <= H; o++)
          if (o == H ? ADV : !(t >= F0 && t < F1)) {
            col[H - o] = S.column(list[t], -o);
            col[H + o - 1] = S.column(list[t], o);
          }
      }
    };
    issue(std::integral_constant<int, 0>{});
    if constexpr (F0 == 0) {
#pragma unroll
      for (int j = 1; j <= PS; j++) S.issue_pair(list[0], j, pr[j - 1]);
    }
    static_for<N>([&](auto tc) BHAH_INLINE {
      constexpr int t = decltype(tc)::value;
      constexpr bool full = t >= F0 && t < F1;
      double vP[2 * H + 1];
      vP[0] = vP[2 * H] = 0.0;
      S.commit_main(m, 0);
#pragma unroll
      for (int o = 1; o <= H; o++)
        if (o == H ? ADV : !full) {
          vP[H - o] = col[H - o];
          vP[H + o] = col[H + o - 1];
        }
      if constexpr (H == 3 || !full) issue(std::integral_constant<int, t + 1>{});
      // the first pairs: a gridfunction early, at 8th order with their own main patch
      if constexpr (H == 3 ? t + 1 == F0 : full && t > 0) {
#pragma unroll
        for (int j = 1; j <= PS; j++) S.issue_pair(list[H == 3 ? F0 : t], j, pr[j - 1]);
      }
      BHAH_PHASE_BARRIER();
      AxisSums s[3];
      double dd[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, c;
      in_plane(0, full, t >= F0 && t < F2, s, dd, c);
      vP[H] = c;
      if constexpr (full) {
        double a0 = 0.0, aE = 0.0;
        static_for<R>([&](auto jc) BHAH_INLINE {
          constexpr int j = decltype(jc)::value + 1;
          S.commit_pair(pr[(j - 1) % PS], PB);
          if constexpr (j + PS <= R) S.issue_pair(list[t], j + PS, pr[(j - 1) % PS]);
          else if constexpr (H == 3 && t + 1 < F1) S.issue_pair(list[t + 1], j + PS - R, pr[(j - 1) % PS]);
          if constexpr (H == 5 && j == R) issue(std::integral_constant<int, t + 1>{});
          BHAH_PHASE_BARRIER();
          double e0[2], eE[2];
#pragma unroll
          for (int side = 0; side < 2; side++) {
            double r0[2 * R + 1], rE[2 * R + 1];
            r0[R] = rE[R] = 0.0;
#pragma unroll
            for (int n = -R; n <= R; n++)
              if (n != 0) {
                r0[R + n] = S.pair_at(PB, side, n, 0);
                rE[R + n] = S.pair_at(PB, side, 0, n);
              }
            e0[side] = d1_sum<R>(r0);
            eE[side] = d1_sum<R>(rE);
            vP[side ? H - j : H + j] = S.pair_at(PB, side, 0, 0);
          }
          a0 = acc_pair<R>(j, a0, e0[0], e0[1]);
          aE = acc_pair<R>(j, aE, eE[0], eE[1]);
          pin(a0);
          pin(aE);
          BHAH_PHASE_BARRIER();
        });
        dd[sy(0, PD)] = a0;
        dd[sy(E, PD)] = aE;
      }
      s[PD] = axis_sums<R>(vP);
      pin<ADV>(s[PD], t >= F0 && t < F2, full);
#pragma unroll
      for (int k = 0; k < 3; k++) dd[sy(k, k)] = s[k].d2;
      fn(t, s, dd);
    });
  }
}

template <int C, bool AX, int H, int F0, int F1, int F2, bool ADV, int N, class FN>
__device__ __forceinline__ void run_stencils(const GatherSrc<H>& S, const int (&list)[N], const FN& fn) {
  constexpr int PD = C == BHAH_SINH_CYLINDRICAL ? 1 : 2, E = 3 - PD, R = H - 1;
  static_for<N>([&](auto tc) BHAH_INLINE {
    constexpr int t = decltype(tc)::value;
    const int g = list[t];
    double v0[2 * H + 1], vE[2 * H + 1], vP[2 * H + 1];
#pragma unroll
    for (int m = -H; m <= H; m++) {
      v0[H + m] = S.at(g, m, 0, 0);
      vE[H + m] = m == 0 ? v0[H] : S.at(g, 0, m, 0);
      if constexpr (!AX) vP[H + m] = m == 0 ? v0[H] : S.at(g, 0, 0, m);
    }
    if constexpr (AX) vP[H + 1] = S.at(g, 0, 0, 1);
    AxisSums s[3];
    double dd[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (t >= F0 && t < F1) {
      double x[4 * R * R];  // f at (n, m) along (i0, e)
#pragma unroll
      for (int m = -R; m <= R; m++)
#pragma unroll
        for (int n = -R; n <= R; n++)
          if (m != 0 && n != 0) x[2 * R * xo<R>(m) + xo<R>(n)] = S.at(g, n, m, 0);
      BHAH_PHASE_BARRIER();
      double e[2 * R + 1];
      e[R] = 0.0;
#pragma unroll
      for (int m = -R; m <= R; m++)
        if (m != 0) {
          double r[2 * R + 1];
          r[R] = 0.0;
#pragma unroll
          for (int n = -R; n <= R; n++)
            if (n != 0) r[R + n] = x[2 * R * xo<R>(m) + xo<R>(n)];
          e[R + m] = d1_sum<R>(r);
        }
      dd[sy(0, E)] = d1_sum<R>(e);
      pin(dd[sy(0, E)]);
      if constexpr (!AX) {
        double a0 = 0.0, aE = 0.0;
#pragma unroll
        for (int j = 1; j <= R; j++) {
          double e0[2], eE[2];
#pragma unroll
          for (int side = 0; side < 2; side++) {
            double r0[2 * R + 1], rE[2 * R + 1];
            r0[R] = rE[R] = 0.0;
#pragma unroll
            for (int n = -R; n <= R; n++)
              if (n != 0) {
                r0[R + n] = S.at(g, n, 0, side ? -j : j);
                rE[R + n] = S.at(g, 0, n, side ? -j : j);
              }
            e0[side] = d1_sum<R>(r0);
            eE[side] = d1_sum<R>(rE);
          }
          a0 = acc_pair<R>(j, a0, e0[0], e0[1]);
          aE = acc_pair<R>(j, aE, eE[0], eE[1]);
          pin(a0);
          pin(aE);
        }
        dd[sy(0, PD)] = a0;
        dd[sy(E, PD)] = aE;
      }
    }
    BHAH_PHASE_BARRIER();
    s[0] = axis_sums<R>(v0);
    s[E] = axis_sums<R>(vE);
    if constexpr (AX) s[PD] = axis_sums_two_planes<R>(v0[H], vP[H + 1]);
    else s[PD] = axis_sums<R>(vP);
#pragma unroll
    for (int k = 0; k < 3; k++) dd[sy(k, k)] = s[k].d2;
    fn(t, s, dd);
    BHAH_PHASE_BARRIER();
  });
}

// the number of a staged tile as the pushed ghosts are grouped (PushDev)
template <int C, int H>
__device__ __forceinline__ int patch_number(const PushDev& P, int t0, int t1, int t2) {
  const int x = (t0 - H) >> TLX;
  if constexpr (C == BHAH_SINH_CYLINDRICAL) return ((t1 - H) * P.ne + (t2 - H) / TEE) * P.nx + x;
  else return ((t2 - H) * P.ne + (t1 - H) / TEE) * P.nx + x;
}

// the point of a lane and the tile it belongs to
struct TilePoint {
  int t0, t1, t2, i0, i1, i2;
  unsigned q;
  bool live;
};

template <class SRC, int C, bool AX, int H>
__device__ __forceinline__ SRC make_source(const double* y, const GridDev& G, const TilePoint& p, int lane,
                                           double* lds) {
  constexpr bool cyl = C == BHAH_SINH_CYLINDRICAL;
  if constexpr (SRC::STG) {
    SRC S;
    if (cyl) S.init(y, G, 1, p.t0, p.t2, p.i0, p.i2, p.t1, lane, lds, AX);
    else S.init(y, G, 2, p.t0, p.t1, p.i0, p.i1, p.t2, lane, lds, AX);
    return S;
  } else {
    return SRC{PtT<H>(y, G, C, p.i0, p.i1, p.i2), cyl ? 1 : 2};
  }
}

}  // namespace bhah
