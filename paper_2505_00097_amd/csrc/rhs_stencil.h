// rhs_stencil.h -- the stencil side of the right-hand side (rhs_point.h) and
// the constraints (hamiltonian.hip): the stencil sums of one gridfunction,
// the LDS patches its values come from, the loop over gridfunctions, and the
// tile walk.
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

// Between LDS accesses of a wave where one lane reads or overwrites what another
// lane of the wave stored or reads. The LDS serves a wave's accesses in the order
// of their issue, so no instruction is emitted; this holds the compiler to that
// order, which otherwise would rest on its not telling the addresses apart. The
// 72 x 12 x 24 RK4 step takes 63.5 us with it, 63.3 without.
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

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
// A tile is a patch of 16 points along i0 and 4 along the other non-periodic
// direction e (i2 on SinhCylindrical grids, i1 otherwise) on one phi plane.
// For one gridfunction at a time the wave brings the patch with its halo into
// LDS with 16-byte loads and takes every stencil value along i0 and e from
// there; values at other phi planes are read per lane. The CU's vector memory
// path takes about the same time for every load instruction whatever its width
// (16 cycles measured for 64 lanes), so what counts is the number of
// instructions: a 16 x 4 patch with its halo at 4th order is 22 x 10 values,
// two loads, where a row of 64 points would be 7 x 70, four, and per-lane
// gathers 30 to 70.
// Mixed derivatives are taken one direction at a time: every lane's D_e f
// (which its first derivative needs anyway) goes into a second LDS patch, with
// those of the halo columns, and D_0 of it is the mixed pair (0, e); the same
// with D_phi f and a halo in both directions for (0, phi) and (e, phi). On
// general grids this reads 16 values from LDS per gridfunction at 4th order
// and 32 at 8th where products of stencils read 52 and 192, and leaves
// registers free: a right-hand side of one 72 x 12 x 24 grid takes 12.6 us
// instead of 14.3, at 8th order with dissipation 1.32 ms instead of 1.53 on a
// 256 x 128 x 64 one.
constexpr int TLX = PATCH_LX, TEX = PATCH_X, TEE = PATCH_E;
template <int H, bool AX>
struct Patch {
  static constexpr int R = H - 1;
  // the main patch (halo H): row length, 16-byte pieces, loads, doubles
  static constexpr int RL = TEX + 2 * H, NP = RL * (TEE + 2 * H) / 2, NR = (NP + 63) / 64, MAIN = 2 * NP;
  // the derivative patches: of D_e with a halo R along i0, on general grids
  // of D_phi with one along e too
  static constexpr int GL = TEX + 2 * R, EN = GL * TEE, PN = AX ? 0 : GL * (TEE + 2 * R);
  // The phi planes at offsets -R..R, in pairs of points. 4th order (RAW): the
  // patch's rows with their halo along i0, then the rows of the halo along e,
  // D_phi of each formed in registers; the point's own values come from the
  // same loads through LDS (a raw patch of the four planes). Line requests from
  // the CUs to the L2s cost time on 3-D grids: the 256 x 128 x 64 right-hand side
  // took 716, 684 and 642 us with 92, 84 and 74 million of them, about 4 us per
  // million (and some 345 us that do not follow them), so no line is asked for
  // twice: with the halo alone in pairs and the point's own column loaded apart
  // it makes 92 instead of 83 million, 716 instead of 687 us. At 8th order
  // LDS has no room for the raw patch: halo (rows along e, then columns) and
  // own column there.
  static constexpr bool RAW = !AX && H == 3;
  static constexpr int IN = GL / 2 * TEE, HROWS = 2 * R * TEX / 2, HP = RAW ? IN + HROWS : HROWS + TEE * R;
  static constexpr int HR = (HP + 63) / 64;
  static constexpr int RAWP = GL * TEE, RN = RAW ? 2 * R * RAWP : 0, DUMP = RAW ? 2 * (64 - IN) : 0;
};

// a wave's stencil stage: PER gridfunctions at a time (main patch, D_e
// patch), then the D_phi patch
template <bool AX, int H>
struct StageSize {
  static constexpr int PER = AX && H == 3 ? 2 : 1;
  using PG = Patch<H, AX>;
  static constexpr int DN = PER * PG::EN + PG::PN;  // the derivative patches; the raw patch lies over them
  static constexpr int N = PER * PG::MAIN + (PG::RN > DN ? PG::RN : DN) + PG::DUMP;  // doubles
  static constexpr int SL = (N + 63) / 64;                                           // slots of 64
};

// All lanes work at their own place in the patch, also where it lies past the
// grid (their loads stay in the descriptors' bounds, their values reach no
// point on the grid).
template <int H, bool AX>
struct Source {
  using PG = Patch<H, AX>;
  static constexpr int R = H - 1, PER = StageSize<AX, H>::PER;
  static constexpr int EB = PER * PG::MAIN, PB = EB + PER * PG::EN;  // where the D_e and D_phi patches begin
  const double* y;
  long long sgf;
  double* lds;             // the wave's stage
  int lane;
  unsigned voff[PG::NR];   // per-lane byte offsets of the lane's pieces of the main patch
  unsigned hoff[PG::HR];   // ... of its pairs of the phi halo
  int hpos[PG::HR];        // their place in the D_phi patch
  int rpos, rstep;         // place of the first pairs in the raw patch, step from plane to plane
  unsigned vlane;          // byte offset of the point, phi index removed
  int sw[2 * H + 1];       // byte offsets of the (wrapped) phi planes at offsets -H..H, wave-uniform
  unsigned org;            // byte offset of the patch origin (halo H), phi index removed, wave-uniform
  int c0, g0;              // the point's place in the main and in a D_e patch
  int hc0, hg0;            // the same of the lane's halo column point

  // tile origin (it, et), phi index ip; pd: the phi direction
  __device__ __forceinline__ Source(const double* y_, const GridDev& G, int pd, int it, int et, int ip, int lane_,
                                    double* lds_)
      : y(y_), sgf(G.sgf), lds(lds_), lane(lane_) {
    const int sP = pd == 1 ? G.s1 : G.s2, sE = pd == 1 ? G.s2 : G.s1, nP = pd == 1 ? G.N1 : G.N2;
    const int id = ip - H;
#pragma unroll
    for (int o = -H; o <= H; o++) {
      int x = id + o;
      if (AX) {
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
    const int x = lane & (TEX - 1), e = lane >> TLX;
    vlane = org + (unsigned)((x + H) + sE * (e + H)) * 8u;
#pragma unroll
    for (int r = 0; r < PG::NR; r++) {
      const int p = piece<PG::NP>(r), row = p / (PG::RL / 2), col = 2 * (p - row * (PG::RL / 2));
      voff[r] = (unsigned)(col + row * sE) * 8u;
    }
    c0 = (e + H) * PG::RL + x + H;
    g0 = e * PG::GL + x + R;
    {  // 2R halo columns of TEE points; lanes beyond repeat them
      const int p = lane & (2 * R * TEE - 1), he = p / (2 * R), k = p & (2 * R - 1);
      const int hx = k < R ? k - R : TEX + k - R;
      hc0 = (he + H) * PG::RL + hx + H;
      hg0 = he * PG::GL + hx + R;
    }
    if constexpr (!AX) {
#pragma unroll
      for (int r = 0; r < PG::HR; r++) {
        int hx, he;
        const int p = piece<PG::HP>(r), q = p - (PG::RAW ? PG::IN : PG::HROWS);
        if (PG::RAW ? q >= 0 : q < 0) {
          const int row = PG::RAW ? q : p;
          he = row / (TEX / 2);
          hx = 2 * (row & (TEX / 2 - 1));
          he = he < R ? he - R : TEE + he - R;
        } else if (PG::RAW) {
          he = p / (PG::GL / 2);
          hx = 2 * (p - he * (PG::GL / 2)) - R;
        } else {
          he = q / R;
          hx = 2 * (q & (R - 1));
          hx = hx < R ? hx - R : TEX + hx - R;
        }
        hoff[r] = (unsigned)((hx + H) + (he + H) * sE) * 8u;
        hpos[r] = (he + R) * PG::GL + hx + R;
      }
      if constexpr (PG::RAW) {  // the pairs of other rows go to places that nobody reads
        rpos = EB + (lane < PG::IN ? 2 * lane : PG::RN + 2 * (lane - PG::IN));
        rstep = lane < PG::IN ? PG::RAWP : 0;
      }
    }
  }
  // the lane's r-th piece of N; past the last one it repeats it, so that every
  // lane loads and stores in bounds
  template <int N>
  __device__ __forceinline__ int piece(int r) const {
    return (r + 1) * 64 <= N ? r * 64 + lane : min(r * 64 + lane, N - 1);
  }
  // two values at an even place, in one 16-byte write (as two writes of 8
  // bytes neighbouring lanes' would conflict)
  __device__ __forceinline__ void put2(int at, double a, double b) const {
    typedef double d2 __attribute__((ext_vector_type(2)));
    *(d2*)(lds + at) = d2{a, b};
  }
  struct MainRegs {
    double lo[PG::NR], hi[PG::NR];
  };
  struct HaloRegs {
    double lo[2 * R + 1], hi[2 * R + 1];  // phi offsets -R..R (0 unused)
  };
  __device__ __forceinline__ void issue_main(int g, MainRegs& m) const {
#pragma unroll
    for (int r = 0; r < PG::NR; r++) gf_ld2(y, sgf, g, voff[r], (int)org + sw[H], m.lo[r], m.hi[r]);
  }
  __device__ __forceinline__ void commit_main(const MainRegs& m, int slot) const {
#pragma unroll
    for (int r = 0; r < PG::NR; r++) {
      put2(slot * PG::MAIN + 2 * piece<PG::NP>(r), m.lo[r], m.hi[r]);
    }
  }
  __device__ __forceinline__ void issue_halo(int g, int r, HaloRegs& h) const {
    h.lo[R] = h.hi[R] = 0.0;
#pragma unroll
    for (int m = -R; m <= R; m++)
      if (m != 0) gf_ld2(y, sgf, g, hoff[r], (int)org + sw[H + m], h.lo[R + m], h.hi[R + m]);
  }
  // the lane's first pair of every plane, into the raw patch
  __device__ __forceinline__ void commit_raw(const HaloRegs& h) const {
    int at = rpos;
#pragma unroll
    for (int m = -R; m <= R; m++)
      if (m != 0) {
        put2(at, h.lo[R + m], h.hi[R + m]);
        at += rstep;
      }
  }
  // the point's own values there (v[H + m])
  __device__ __forceinline__ void raw_column(double (&v)[2 * H + 1]) const {
#pragma unroll
    for (int m = -R; m <= R; m++)
      if (m != 0) v[H + m] = lds[EB + (m + R - (m > 0)) * PG::RAWP + g0];
  }
  // D_phi of the lane's r-th pair of points
  __device__ __forceinline__ void put_halo(int r, double lo, double hi) const {
    put2(PB + hpos[r], lo, hi);
  }
  __device__ __forceinline__ void commit_halo(const HaloRegs& h, int r) const {
    put_halo(r, d1_sum<R>(h.lo), d1_sum<R>(h.hi));
  }
  // the values along i0 and e around the point
  __device__ __forceinline__ void cross(int slot, double (&v0)[2 * H + 1], double (&vE)[2 * H + 1]) const {
    const double* p = lds + slot * PG::MAIN + c0;
#pragma unroll
    for (int m = -H; m <= H; m++) vE[H + m] = p[m * PG::RL];
#pragma unroll
    for (int m = -H; m <= H; m++) v0[H + m] = m == 0 ? vE[H] : p[m];
  }
  // the values along e around the lane's halo column point
  __device__ __forceinline__ void halo_column(int slot, double (&v)[2 * R + 1]) const {
    v[R] = 0.0;
#pragma unroll
    for (int m = -R; m <= R; m++)
      if (m != 0) v[R + m] = lds[slot * PG::MAIN + hc0 + m * PG::RL];
  }
  __device__ __forceinline__ void put_e(int slot, double own, double halo) const {
    lds[EB + slot * PG::EN + g0] = own;
    lds[EB + slot * PG::EN + hg0] = halo;
  }
  __device__ __forceinline__ void put_p(double own) const { lds[PB + R * PG::GL + g0] = own; }
  // values of a derivative patch around the point: D_e along i0, D_phi along i0 and e
  __device__ __forceinline__ void around(int at, int step, double (&v)[2 * R + 1]) const {
    v[R] = 0.0;
#pragma unroll
    for (int m = -R; m <= R; m++)
      if (m != 0) v[R + m] = lds[at + m * step];
  }
  __device__ __forceinline__ void e_along_0(int slot, double (&v)[2 * R + 1]) const {
    around(EB + slot * PG::EN + g0, 1, v);
  }
  __device__ __forceinline__ void p_along_0(double (&v)[2 * R + 1]) const { around(PB + R * PG::GL + g0, 1, v); }
  __device__ __forceinline__ void p_along_e(double (&v)[2 * R + 1]) const { around(PB + R * PG::GL + g0, PG::GL, v); }
  // value in the point's phi column
  __device__ __forceinline__ double column(int g, int m) const { return gf_ld(y, sgf, g, vlane, sw[H + m]); }
};

// Tiles: patches of 2^lx points along i0 times 2^ly along i1 times
// 64 >> (lx + ly) along i2 (16 along i0, 4 along e); the tile grid is walked in
// bands of `band` tile rows of i1, and within a band by i2, then i1, then i0
// (fastest), so that tiles that share cache lines along i0 run at the same time.
// The hardware hands consecutive workgroup ids to the XCDs in turn; block ids
// are remapped so that every XCD works through one contiguous range of the walk
// (its L2 then holds a compact part of the grid). Bands of 16, 4 and 1: a
// 256 x 128 x 64 RK4 step takes 3.33, 3.10 and 3.27 ms, an SSPRK3 step there at
// 8th order with dissipation 5.22, 4.23 and 4.59, a 1008 x 168 x 336 RK4 step
// 113.5, 103.9 and 102.6. Neither the bytes past the L2s nor the requests to
// them tell which is best: a right-hand side on the first grid makes 74.6
// million requests at every band, with 28, 28 and 12 million misses, in 664, 641
// and 683 us.
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

// ---- the stencil loop ----------------------------------------------------------
// whether d_k d_l, kl = sy(k, l), vanishes identically (mixed with phi on two planes)
template <bool AX, int PD>
__device__ __forceinline__ constexpr bool zero_pair(int kl) {
  return AX && (kl == sy(0, PD) || kl == sy(3 - PD, PD));
}

// For each gridfunction list[t], t < N: fn(t, raw sums along the three
// directions, raw second differences dd[sy(k, l)], value at the point); dd is
// formed for t in [F0, F1), first derivatives are used for t in [F0, F2), the
// upwinded sums where ADV. Identically vanishing phi derivatives of two-plane
// grids are literal zeros. Loads run one gridfunction (two-plane grids at 4th
// order: a batch of two) ahead of their use: at 4th order all of the next
// gridfunction's at the start of an iteration (those of other phi planes in
// its middle: 657 instead of 643 us on the 3-D grid), at 8th order, short of
// registers, the phi planes in the middle. Two ahead takes 3% longer: the
// waves' lines push each other out of the L1.
template <int C, bool AX, int H, int F0, int F1, int F2, bool ADV, int N, class FN>
__device__ __forceinline__ void run_stencils(const Source<H, AX>& S, const int (&list)[N], const FN& fn) {
  constexpr int PD = C == BHAH_SINH_CYLINDRICAL ? 1 : 2, E = 3 - PD, R = H - 1;
  using PG = Patch<H, AX>;
  if constexpr (AX) {
    constexpr int PER = StageSize<AX, H>::PER, NB = (N + PER - 1) / PER;
    typename Source<H, AX>::MainRegs m[PER];
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
      if constexpr (b > 0) wave_fence();  // the last batch's reads, before its patches are overwritten
#pragma unroll
      for (int t = 0; t < PER; t++)
        if (b * PER + t < N) {
          S.commit_main(m[t], t);
          o[t] = ph[t];
        }
      if constexpr (b + 1 < NB) issue(b + 1);
      BHAH_PHASE_BARRIER();
      wave_fence();
      // every read of the batch's main patches, then its D_e patches, so that
      // one gridfunction's reads are under way while another's are waited for
      double v0[PER][2 * H + 1], vE[PER][2 * H + 1], vh[PER][2 * R + 1];
      AxisSums s[PER][3];
      static_for<PER>([&](auto tc) BHAH_INLINE {
        constexpr int t = decltype(tc)::value, tt = b * PER + t;
        if constexpr (tt < N) {
          S.cross(t, v0[t], vE[t]);
          if constexpr (tt >= F0 && tt < F1) S.halo_column(t, vh[t]);
        }
      });
      static_for<PER>([&](auto tc) BHAH_INLINE {
        constexpr int t = decltype(tc)::value, tt = b * PER + t;
        if constexpr (tt < N) {
          s[t][E] = axis_sums<R>(vE[t]);
          pin<ADV>(s[t][E], tt >= F0 && tt < F2, tt >= F0 && tt < F1);
          if constexpr (tt >= F0 && tt < F1) S.put_e(t, s[t][E].d1, d1_sum<R>(vh[t]));
        }
      });
      if constexpr (b * PER < F1 && (b + 1) * PER > F0) wave_fence();
      static_for<PER>([&](auto tc) BHAH_INLINE {
        constexpr int t = decltype(tc)::value, tt = b * PER + t;
        if constexpr (tt < N) {
          constexpr bool full = tt >= F0 && tt < F1;
          double dd[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, w[2 * R + 1];
          if constexpr (full) S.e_along_0(t, w);
          s[t][0] = axis_sums<R>(v0[t]);
          pin<ADV>(s[t][0], tt >= F0 && tt < F2, full);
          if constexpr (full) {
            dd[sy(0, E)] = d1_sum<R>(w);
            pin(dd[sy(0, E)]);
          }
          s[t][PD] = axis_sums_two_planes<R>(v0[t][H], o[t]);
#pragma unroll
          for (int k = 0; k < 3; k++) dd[sy(k, k)] = s[t][k].d2;
          fn(tt, s[t], dd, v0[t][H]);
        }
      });
    });
  } else {
    constexpr bool RAW = PG::RAW;
    typename Source<H, AX>::MainRegs m;
    typename Source<H, AX>::HaloRegs h[RAW ? PG::HR : 1];
    double col[2 * H];  // phi offsets -H..-1, 1..H
    // a gridfunction's values at other phi planes are fetched together: they
    // share cache lines
    auto issue_phi = [&](auto tc) BHAH_INLINE {
      constexpr int t = decltype(tc)::value;
      if constexpr (t < N) {
        constexpr bool full = t >= F0 && t < F1;
        if constexpr (RAW && full) {
          S.issue_halo(list[t], 0, h[0]);
          S.issue_halo(list[t], 1, h[PG::HR - 1]);
        }
#pragma unroll
        for (int o = 1; o <= (ADV ? H : R); o++)
          if (o == H || !(RAW && full)) {
            col[H - o] = S.column(list[t], -o);
            col[H + o - 1] = S.column(list[t], o);
          }
        if constexpr (!RAW && full) S.issue_halo(list[t], 0, h[0]);
      }
    };
    S.issue_main(list[0], m);
    issue_phi(std::integral_constant<int, 0>{});
    static_for<N>([&](auto tc) BHAH_INLINE {
      constexpr int t = decltype(tc)::value;
      constexpr bool full = t >= F0 && t < F1;
      double vP[2 * H + 1];
      vP[0] = vP[2 * H] = 0.0;
      if constexpr (t > 0) wave_fence();  // the last gridfunction's reads, before its patches are overwritten
      S.commit_main(m, 0);
#pragma unroll
      for (int o = 1; o <= (ADV ? H : R); o++)
        if (o == H || !(RAW && full)) {
          vP[H - o] = col[H - o];
          vP[H + o] = col[H + o - 1];
        }
      double dP[4];  // D_phi of the lane's pairs (4th order)
      if constexpr (RAW && full) {
        S.commit_raw(h[0]);
#pragma unroll
        for (int r = 0; r < 2; r++) {
          dP[2 * r] = d1_sum<R>(h[r].lo);
          dP[2 * r + 1] = d1_sum<R>(h[r].hi);
          pin(dP[2 * r]);
          pin(dP[2 * r + 1]);
        }
      }
      // two rounds of halo loads (8th order): the first, the rows, now
      if constexpr (!RAW && full && PG::HR == 2) {
        S.commit_halo(h[0], 0);
        S.issue_halo(list[t], 1, h[0]);
      }
      if constexpr (t + 1 < N) S.issue_main(list[t + 1], m);
      if constexpr (RAW) issue_phi(std::integral_constant<int, t + 1>{});
      BHAH_PHASE_BARRIER();
      wave_fence();
      AxisSums s[3];
      double dd[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, v0[2 * H + 1], vE[2 * H + 1];
      constexpr bool first = t >= F0 && t < F2;
      S.cross(0, v0, vE);
      vP[H] = v0[H];
      if constexpr (RAW && full) S.raw_column(vP);
      auto sum = [&](int k, const double(&v)[2 * H + 1]) BHAH_INLINE {
        s[k] = axis_sums<R>(v);
        pin<ADV>(s[k], first, full);
      };
      auto mixed = [&](int kl, const double(&v)[2 * R + 1]) BHAH_INLINE {
        dd[kl] = d1_sum<R>(v);
        pin(dd[kl]);
      };
      sum(PD, vP);
      if constexpr (full) {
        double vh[2 * R + 1], w[3][2 * R + 1];
        S.halo_column(0, vh);
        if constexpr (RAW) {
          wave_fence();  // the derivative patches lie over the raw one
          S.put_halo(0, dP[0], dP[1]);
          S.put_halo(1, dP[2], dP[3]);
        } else {
          S.put_p(s[PD].d1);
          S.commit_halo(h[0], PG::HR - 1);
        }
        sum(E, vE);
        S.put_e(0, s[E].d1, d1_sum<R>(vh));
        if constexpr (!RAW) issue_phi(std::integral_constant<int, t + 1>{});
        // at 4th order the reads of the derivative patches are under way
        // during the sums along i0; at 8th there are no registers for that
        if constexpr (H != 3) sum(0, v0);
        BHAH_PHASE_BARRIER();
        wave_fence();
        S.p_along_0(w[0]);
        if constexpr (H != 3) mixed(sy(0, PD), w[0]);
        S.p_along_e(w[1]);
        if constexpr (H != 3) {
          mixed(sy(E, PD), w[1]);
          BHAH_PHASE_BARRIER();
        }
        S.e_along_0(0, w[2]);
        if constexpr (H == 3) {
          sum(0, v0);
          mixed(sy(0, PD), w[0]);
          mixed(sy(E, PD), w[1]);
        }
        mixed(sy(0, E), w[2]);
      } else {
        if constexpr (!RAW) issue_phi(std::integral_constant<int, t + 1>{});
        sum(E, vE);
        sum(0, v0);
      }
#pragma unroll
      for (int k = 0; k < 3; k++) dd[sy(k, k)] = s[k].d2;
      fn(t, s, dd, v0[H]);
    });
  }
  wave_fence();  // the caller may use the stage's slots
}

// the number of a tile as the pushed ghosts are grouped (PushDev)
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

template <int C, bool AX, int H>
__device__ __forceinline__ Source<H, AX> make_source(const double* y, const GridDev& G, const TilePoint& p, int lane,
                                                     double* lds) {
  if constexpr (C == BHAH_SINH_CYLINDRICAL) return Source<H, AX>(y, G, 1, p.t0, p.t2, p.t1, lane, lds);
  else return Source<H, AX>(y, G, 2, p.t0, p.t1, p.t2, lane, lds);
}

}  // namespace bhah
