// rhs_fused.hip -- kernels of the BSSN + gauge right-hand side with the
// Runge-Kutta stage combination (rhs_point.h): one block of two waves per
// 64-point tile for one grid, and the persistent form for ensembles.
#include "rhs_point.h"

// The library builds this source in parts (one set of instantiations each);
// without a part every kernel is instantiated in one unit.
#ifndef BHAH_PART
#define BHAH_PART -1
#endif

namespace bhah {

#ifndef BHAH_RHS_WAVES
#define BHAH_RHS_WAVES 2
#endif

// One tile per block. PUSH: the form for Runge-Kutta stages, with the stage
// ghosts of its tile where the launch passes some.
template <int C, bool AX, bool KO, int H, bool PUSH>
__global__ void __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(BHAH_RHS_WAVES, BHAH_RHS_WAVES)))
k_rhs_fused(GridDev G, TileMap T, Gauge ga, const double* __restrict__ y, StageArgs st, PushDev P,
            double* __restrict__ aux) {
  const int per = (T.ntiles + BHAH_NXCD - 1) / BHAH_NXCD;
  const int w = xcd_remap((int)blockIdx.x, per);
  if (w >= T.ntiles) return;
  __shared__ __attribute__((aligned(16))) double xs[X_SLOTS * 64];
  rhs_tile<C, AX, KO, H, PUSH>(G, T, w, ga, y, st, P, aux, xs);
}

// Persistent form for ensembles: a fixed grid of blocks (a multiple of the
// XCD count) strides over one kernel variant's (job, tile) work list (the
// jobs of one family, phi extent and order, H ghost layers); every point
// runs the same rhs_tile as above.
template <int C, bool AX, bool KO, int H>
__global__ void __launch_bounds__(128) __attribute__((amdgpu_waves_per_eu(BHAH_RHS_WAVES, BHAH_RHS_WAVES)))
k_rhs_batch(const BatchJob* __restrict__ jobs, const BatchHdr* __restrict__ hdr, const int2* __restrict__ work,
            int stage, const int* __restrict__ counts, int kk, Gauge ga) {
  constexpr int V = 2 * C + AX + (H == 5 ? 6 : 0);
  const int n = hdr->n_tiles[V];
  const int2* wl = work + hdr->tile_off[V];
  const int per = (n + BHAH_NXCD - 1) / BHAH_NXCD;
  __shared__ __attribute__((aligned(16))) double xs[X_SLOTS * 64];
  for (int t = (int)blockIdx.x; t < per * BHAH_NXCD; t += (int)gridDim.x) {
    const int w = xcd_remap(t, per);
    if (w >= n) continue;
    const int2 wk = wl[w];
    if (counts && kk >= counts[wk.x]) continue;  // the job takes no step kk in this launch
    const BatchJob* J = jobs + wk.x;
    const GridDev G = J->G;
    const StageArgs st = J->st[stage];
    rhs_tile<C, AX, KO, H, false>(G, J->T, wk.y, ga, J->in[stage], st, PushDev{}, nullptr, xs);
    __syncthreads();  // the next tile's stencil stage reuses slots that the other wave reads to the end
  }
}

using FusedLaunch = void (*)(dim3, hipStream_t, const GridDev&, const TileMap&, const Gauge&, const double*,
                             const StageArgs&, const PushDev&, double*);
using BatchLaunch = void (*)(dim3, hipStream_t, const BatchJob*, const BatchHdr*, const int2*, int, const int*, int,
                             const Gauge&);
template <int C, bool AX, bool KO, int H, bool PUSH>
void launch_fused_t(dim3 g, hipStream_t s, const GridDev& G, const TileMap& T, const Gauge& ga, const double* y,
                    const StageArgs& st, const PushDev& P, double* aux) {
  hipLaunchKernelGGL((k_rhs_fused<C, AX, KO, H, PUSH>), g, dim3(128), 0, s, G, T, ga, y, st, P, aux);
}
template <int C, bool AX, bool KO, int H>
void launch_batch_t(dim3 g, hipStream_t s, const BatchJob* jobs, const BatchHdr* hdr, const int2* work, int stage,
                    const int* counts, int kk, const Gauge& ga) {
  hipLaunchKernelGGL((k_rhs_batch<C, AX, KO, H>), g, dim3(128), 0, s, jobs, hdr, work, stage, counts, kk, ga);
}

// launch tables of one variant (rhs_variant): [dissipation]
struct RhsKernels {
  FusedLaunch plain[2], push[2];  // push: none where rhs_pushes is false
  BatchLaunch batch[2];
};
template <int C, bool AX, int H>
constexpr RhsKernels rhs_kernels() {
  RhsKernels k{{launch_fused_t<C, AX, false, H, false>, launch_fused_t<C, AX, true, H, false>},
               {nullptr, nullptr},
               {launch_batch_t<C, AX, false, H>, launch_batch_t<C, AX, true, H>}};
  if constexpr (AX || H == 3) {
    k.push[0] = launch_fused_t<C, AX, false, H, true>;
    k.push[1] = launch_fused_t<C, AX, true, H, true>;
  }
  return k;
}
// part p holds variant p: family p / 2 % 3, two phi planes p % 2, order p / 6
template <int V>
const RhsKernels& rhs_part();
#define BHAH_DEFINE_PART(V)                                                            \
  template <>                                                                          \
  const RhsKernels& rhs_part<V>() {                                                    \
    static const RhsKernels k = rhs_kernels<(V) / 2 % 3, (V) % 2 == 1, (V) >= 6 ? 5 : 3>(); \
    return k;                                                                          \
  }
#if BHAH_PART >= 0
BHAH_DEFINE_PART(BHAH_PART)
#else
BHAH_DEFINE_PART(0) BHAH_DEFINE_PART(1) BHAH_DEFINE_PART(2) BHAH_DEFINE_PART(3) BHAH_DEFINE_PART(4)
BHAH_DEFINE_PART(5) BHAH_DEFINE_PART(6) BHAH_DEFINE_PART(7) BHAH_DEFINE_PART(8) BHAH_DEFINE_PART(9)
BHAH_DEFINE_PART(10) BHAH_DEFINE_PART(11)
#endif

#if BHAH_PART <= 0
template <> const RhsKernels& rhs_part<1>();
template <> const RhsKernels& rhs_part<2>();
template <> const RhsKernels& rhs_part<3>();
template <> const RhsKernels& rhs_part<4>();
template <> const RhsKernels& rhs_part<5>();
template <> const RhsKernels& rhs_part<6>();
template <> const RhsKernels& rhs_part<7>();
template <> const RhsKernels& rhs_part<8>();
template <> const RhsKernels& rhs_part<9>();
template <> const RhsKernels& rhs_part<10>();
template <> const RhsKernels& rhs_part<11>();

static const RhsKernels& kernels_of(int variant) {
  using Get = const RhsKernels& (*)();
  static const Get get[NVAR] = {rhs_part<0>, rhs_part<1>, rhs_part<2>, rhs_part<3>, rhs_part<4>,  rhs_part<5>,
                                rhs_part<6>, rhs_part<7>, rhs_part<8>, rhs_part<9>, rhs_part<10>, rhs_part<11>};
  return get[variant]();
}

TileMap make_tilemap(const GridDev& G, int band) {
  TileMap T;
  T.lx = TLX;
  T.ly = G.coord == BHAH_SINH_CYLINDRICAL ? 0 : 6 - TLX;
  const int ex = 1 << T.lx, ey = 1 << T.ly, ez = 64 >> (T.lx + T.ly);
  T.tx = (G.N0 + ex - 1) / ex;
  T.ty = (G.N1 + ey - 1) / ey;
  T.tz = (G.N2 + ez - 1) / ez;
  T.ntiles = T.tx * T.ty * T.tz;
  T.band = band < 1 ? 1 : (band > T.ty ? T.ty : band);
  return T;
}

void launch_rhs_fused(const GridDev& G, const Gauge& ga, const double* y, double* aux, const StageArgs& st,
                      hipStream_t s, int band, const PushDev& push) {
  const TileMap T = make_tilemap(G, band);
  const int per = (T.ntiles + BHAH_NXCD - 1) / BHAH_NXCD;
  const RhsKernels& k = kernels_of(rhs_variant(G.coord, G.N1, G.N2, G.ng));
  // one form for all stages of a step, also the last, which pushes nothing:
  // a change of kernel between stages costs a cold instruction cache (the
  // 32 x 16 x 2 RK4 step 41.0 us so, 41.8 with the plain form at the last stage)
  const FusedLaunch stage = k.push[ga.ko() ? 1 : 0];
  (!st.rhs && stage ? stage : k.plain[ga.ko() ? 1 : 0])(dim3(per * BHAH_NXCD), s, G, T, ga, y, st, push, aux);
}

void launch_rhs_batch(int variant, const BatchJob* jobs, const BatchHdr* hdr, const int2* work, int stage,
                      const int* counts, int kk, const Gauge& ga, int blocks, hipStream_t s) {
  kernels_of(variant).batch[ga.ko() ? 1 : 0](dim3(blocks), s, jobs, hdr, work, stage, counts, kk, ga);
}
#endif

}  // namespace bhah
