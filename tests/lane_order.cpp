// lane_order.cpp -- the tiles of the right-hand side and of the constraints on
// the CPU: every lane of a block is a fibre that runs alone from one
// synchronisation (wave_fence, a wave's vote or shuffle, __syncthreads) to the
// next, in an order of the caller's choice. Whatever a lane takes from another
// one without a synchronisation between then depends on that order.
#include <hip/hip_runtime.h>
#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <functional>
#include <memory>
#include <vector>

namespace fibres {
enum State { READY, AT_WAVE, AT_BLOCK, DONE };
constexpr int N = 128;
ucontext_t home, ctx[N];
State state[N];
int cur;
double val[N];
const std::function<void()>* body;
std::vector<char> stacks((size_t)N << 19);

void yield(State s) {
  state[cur] = s;
  swapcontext(&ctx[cur], &home);
}
void entry() {
  (*body)();
  state[cur] = DONE;
}
// lanes of wave w, each to its next synchronisation, until all of them wait for the block or are done
bool run_wave(int w, int order) {
  for (;;) {
    for (int k = 0; k < 64; k++) {
      cur = 64 * w + (order == 0 ? k : order == 1 ? 63 - k : (29 * k + 7) & 63);
      if (state[cur] != DONE) swapcontext(&home, &ctx[cur]);
    }
    for (int l = 1; l < 64; l++)
      if (state[64 * w + l] != state[64 * w]) return false;  // lanes at different synchronisations
    if (state[64 * w] != AT_WAVE) return true;
  }
}
bool run_block(const std::function<void()>& f, int order) {
  body = &f;
  for (int l = 0; l < N; l++) {
    state[l] = READY;
    getcontext(&ctx[l]);
    ctx[l].uc_stack.ss_sp = &stacks[(size_t)l << 19];
    ctx[l].uc_stack.ss_size = (size_t)1 << 19;
    ctx[l].uc_link = &home;
    makecontext(&ctx[l], entry, 0);
  }
  for (;;) {
    const int first = order & 1;
    if (!run_wave(first, order) || !run_wave(1 - first, order)) return false;
    if (state[0] != state[64]) return false;
    if (state[0] == DONE) return true;
  }
}
struct Dim {
  unsigned x;
};
double wave_value(double v, int lane) {  // v of a lane of this wave
  val[cur] = v;
  yield(AT_WAVE);
  const double r = val[(cur & ~63) + (lane & 63)];
  yield(AT_WAVE);
  return r;
}
}  // namespace fibres

using std::min;
inline int __shfl(int v, int lane) { return (int)fibres::wave_value(v, lane); }
inline int __all(bool p) {
  bool all = true;
  for (int l = 0; l < 64; l++) all = fibres::wave_value(p, l) != 0.0 && all;
  return all;
}
// a buffer descriptor and its range check
struct Rsrc {
  const char* p;
  unsigned n;
};
template <class T>
T buffer_load(const Rsrc& r, unsigned off) {
  T v;
  for (unsigned k = 0; k < sizeof(T) / 4; k++) {
    unsigned w = 0;
    if ((unsigned long long)off + 4 * k + 4 <= r.n) std::copy_n(r.p + off + 4 * k, 4, (char*)&w);
    v[k] = w;
  }
  return v;
}
typedef unsigned u2_ __attribute__((ext_vector_type(2)));
typedef unsigned u4_ __attribute__((ext_vector_type(4)));
#define threadIdx (fibres::Dim{(unsigned)fibres::cur})
#define blockIdx (fibres::Dim{0})
#define gridDim (fibres::Dim{1})
#define __syncthreads() fibres::yield(fibres::AT_BLOCK)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_wave_barrier() fibres::yield(fibres::AT_WAVE)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __amdgpu_buffer_rsrc_t Rsrc
#define __builtin_amdgcn_make_buffer_rsrc(p, s, n, f) (Rsrc{(const char*)(p), (unsigned)(n)})
#define __builtin_amdgcn_raw_buffer_load_b64(r, v, s, c) buffer_load<u2_>(r, (v) + (unsigned)(s))
#define __builtin_amdgcn_raw_buffer_load_b128(r, v, s, c) buffer_load<u4_>(r, (v) + (unsigned)(s))
#define amdgpu_waves_per_eu(...) unused
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...)
#ifndef __launch_bounds__
#define __launch_bounds__(n)
#endif

#include "../paper_2505_00097_amd/csrc/rhs_point.h"
#define BHAH_PART 1  // any part without the dispatch; the tiles are instantiated below
#include "../paper_2505_00097_amd/csrc/hamiltonian.hip"
#include "../paper_2505_00097_amd/csrc/grid.cpp"

namespace bhah {
int fail(int code, const std::string&) { return code; }
}  // namespace bhah
using namespace bhah;

constexpr int C = VARIANT / 2 % 3, H = VARIANT >= 6 ? 5 : 3;
constexpr bool AX = VARIANT % 2 == 1;

// what 0: right-hand side into out, with aux; 1: the stage out = base + c k with
// the pushed ghosts (those left to the ghost kernel are not written); 2: the
// seven constraints into out. Tiles are walked in bands of `band`. Returns 0, or 1 where lanes of a wave or the waves
// come to different synchronisations.
extern "C" int run_tiles(const bhah_grid_params* par, const bhah_gauge_params* gp, int what, int order, int band, const double* y,
                         const double* base, double c, double* out, double* aux) {
  std::unique_ptr<bhah_grid> g(new bhah_grid());
  if (int rc = build_grid_host(par, g.get())) return rc;
  const int* n = g->info.n_total;
  GridDev G{par->coord, par->N[0], par->N[1], par->N[2], n[0], n[1], n[2], n[0], n[0] * n[1], par->nghosts,
            g->info.n_points, {1.0 / g->info.dxx[0], 1.0 / g->info.dxx[1], 1.0 / g->info.dxx[2]},
            g->tab[0].data(), g->tab[1].data(), g->tab[2].data()};
  if (rhs_variant(C, G.N1, G.N2, G.ng) != VARIANT || G.coord != C) return -100;
  TileMap T;
  T.lx = TLX;
  T.ly = C == BHAH_SINH_CYLINDRICAL ? 0 : 6 - TLX;
  T.tx = (G.N0 + TEX - 1) / TEX;
  T.ty = (G.N1 + (1 << T.ly) - 1) >> T.ly;
  T.tz = C == BHAH_SINH_CYLINDRICAL ? (G.N2 + TEE - 1) / TEE : G.N2;
  T.ntiles = T.tx * T.ty * T.tz;
  T.band = std::min(T.ty, band);
  const HostPush& P = g->push;
  const PushDev push = what == 1 && !P.start.empty()
                           ? PushDev{P.start.data(), P.rec.data(), P.terms.data(), P.nx, P.ne}
                           : PushDev{};
  const Gauge ga = gauge_of(*gp);
  StageArgs st{};
  if (what == 0) st.rhs = out;
  else st = StageArgs{nullptr, base, out, c, nullptr, 0.0, 0.0, nullptr, nullptr};
  std::vector<double> lds(5121, NAN);
  double* xs = lds.data() + ((size_t)lds.data() & 8 ? 1 : 0);
  for (int w = 0; w < T.ntiles; w++) {
    const std::function<void()> rhs = [&] { rhs_tile<C, AX, true, H, AX || H == 3>(G, T, w, ga, y, st, push, aux, xs); };
    const std::function<void()> con = [&] {
      constraints_tile<C, AX, H, true>(G, T, w, y, out, out + G.sgf, out + 4 * G.sgf, xs);
    };
    if (!fibres::run_block(what == 2 ? con : rhs, order)) return 1;
  }
  return 0;
}
