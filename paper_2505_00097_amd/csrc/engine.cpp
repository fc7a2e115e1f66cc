// engine.cpp -- ensemble engine: work lists, graph cache and tile autotuner.
#include "engine.h"

#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstring>
#include <set>

namespace bhah {

namespace {

constexpr size_t kAlign = 256;
size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

SizeClass class_of(const bhah_grid* g) {
  return SizeClass{g->params.coord, g->params.N[0], g->params.N[1], g->params.N[2]};
}

struct Layout {
  size_t jobs, counts, tiles, chunks, total;
};

// header | job table | per-job active step counts | tile list | chunk list
Layout layout(int cap_jobs, int cap_tiles, int cap_chunks) {
  Layout L;
  L.jobs = align_up(sizeof(BatchHdr));
  L.counts = L.jobs + align_up(sizeof(BatchJob) * (size_t)cap_jobs);
  L.tiles = L.counts + align_up(sizeof(int) * (size_t)cap_jobs);
  L.chunks = L.tiles + align_up(sizeof(int2) * (size_t)cap_tiles);
  L.total = L.chunks + align_up(sizeof(int2) * (size_t)cap_chunks);
  return L;
}

double now_s() {
  using namespace std::chrono;
  return duration<double>(steady_clock::now().time_since_epoch()).count();
}

}  // namespace

// candidate tile configurations for one size class
std::vector<TileCfg> tile_candidates(const SizeClass& c) {
  const int N1 = std::get<2>(c), ty = std::get<0>(c) == BHAH_SINH_CYLINDRICAL ? N1 : (N1 + PATCH_E - 1) / PATCH_E;
  std::vector<TileCfg> out;
  // bands of 16, 4 and 1 tile rows: which planes tiles that run at the same
  // time share (times of each beside the walk, rhs_stencil.h). A grid's tuner
  // gives near-ties to the first, a batch takes the fastest
  if (ty > 8) out.push_back(TileCfg{6, 0, 16});
  if (ty > 1) out.push_back(TileCfg{6, 0, 4});
  out.push_back(TileCfg{6, 0, 1});
  return out;
}

Engine::Engine(const bhah_gauge_params& gp, const char* cache_path) : gp_(gp) {
  if (cache_path) cache_path_ = cache_path;
}

Engine::~Engine() {
  drop_graphs();
  if (cap_stream_) (void)hipStreamDestroy(cap_stream_);
  if (upload_done_) (void)hipEventDestroy(upload_done_);
  for (hipEvent_t& e : counts_done_)
    if (e) (void)hipEventDestroy(e);
  if (h_counts_) (void)hipHostFree(h_counts_);
  if (d_blob_) (void)hipFree(d_blob_);
  if (h_blob_) (void)hipHostFree(h_blob_);
}

TileCfg Engine::tile_of_class(const SizeClass& c) const {
  auto it = tuned_.find(c);
  return it == tuned_.end() ? TileCfg{6, 0, BHAH_DEFAULT_BAND} : it->second;
}

int Engine::set_jobs(const std::vector<EngineJob>& jobs) {
  for (const EngineJob& j : jobs) {
    if (!j.g || !j.y || !j.ws) return fail(BHAH_EINVAL, "batch: NULL grid, state or workspace");
    if (j.g->params.coord < 0 || j.g->params.coord > 2) return fail(BHAH_EINVAL, "batch: bad coordinate family");
  }
  if (jobs != jobs_) {
    jobs_ = jobs;
    dirty_ = true;
  } else {
    // the step limits change from call to call without touching the blob
    for (size_t j = 0; j < jobs.size(); j++) jobs_[j].limit = jobs[j].limit;
  }
  return BHAH_OK;
}

Engine::ListSizes Engine::list_sizes() const {
  ListSizes n;
  for (int j = 0; j < (int)jobs_.size(); j++) {
    const GridDev& G = jobs_[j].g->dev;
    n.tiles[rhs_variant(G.coord, G.N1, G.N2, G.ng)] += make_tilemap(G, 1).ntiles;
    n.rad += lists_of(j).rad.n;
  }
  return n;
}

// Blocks of the right-hand-side kernel for one variant whose jobs have `list`
// tiles, to run `tiles` of them: blocks_per_cu_ per compute unit (blocks of two
// waves, two waves per SIMD, so 4 fill a CU) striding over the work list, or
// with blocks_per_cu_ == 0 one block per tile; always a multiple of the XCD
// count. A list of more than 8 tiles per block runs one block per tile as
// well: blocks that stride drift apart, and the planes that their tiles share
// leave the L2s. One 1008 x 168 x 336 job: 171 ms a step striding, 105 with
// one block per tile; 256 x 128 x 64 (32 tiles per block) 3.56, 3.25; 16
// head-on jobs (13) 1.154, 1.135; four 96 x 32 x 32 jobs (6) 0.651, 0.686.
// One block per tile is rounded up in steps of 1/64 to 1/32 of the tiles, so
// that job sets of nearly one size share a captured graph.
int Engine::rhs_grid(long long list, long long tiles) const {
  if (tiles <= 0) return 0;
  const long long stride = (long long)blocks_per_cu_ * n_cus_;
  if (stride > 0 && list <= 8 * stride) return (int)((stride + BHAH_NXCD - 1) / BHAH_NXCD * BHAH_NXCD);
  long long step = BHAH_NXCD;
  while (64 * step <= tiles) step *= 2;
  return (int)((tiles + step - 1) / step * step);
}

Engine::LaunchShape Engine::launch_shape() const {
  const ListSizes n = list_sizes();
  LaunchShape l{};
  for (int v = 0; v < NVAR; v++) l[v] = rhs_grid(n.tiles[v], n.tiles[v]);
  l[NVAR] = n.rad > 0 ? 1 : 0;
  return l;
}

int Engine::ensure_device(hipStream_t s) {
  (void)s;
  if (upload_done_) return BHAH_OK;
  int dev = 0, cus = 0;
  int rc = check_hip(hipGetDevice(&dev), "hipGetDevice");
  if (rc) return rc;
  if ((rc = check_hip(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev), "CU count")))
    return rc;
  hipDeviceProp_t prop;
  if ((rc = check_hip(hipGetDeviceProperties(&prop, dev), "hipGetDeviceProperties"))) return rc;
  arch_ = prop.gcnArchName;
  const size_t colon = arch_.find(':');
  if (colon != std::string::npos) arch_ = arch_.substr(0, colon);
  n_cus_ = std::max(cus, 1);
  ghost_blocks_ = 2 * n_cus_;  // times NGF / GF_PER gridfunction groups
  if ((rc = check_hip(hipEventCreateWithFlags(&upload_done_, hipEventDisableTiming), "hipEventCreate"))) return rc;
  for (hipEvent_t& e : counts_done_)
    if ((rc = check_hip(hipEventCreateWithFlags(&e, hipEventDisableTiming), "hipEventCreate"))) return rc;
  if ((rc = check_hip(hipStreamCreateWithFlags(&cap_stream_, hipStreamNonBlocking), "hipStreamCreate"))) return rc;
  load_cache();
  return BHAH_OK;
}

void Engine::drop_graphs() {
  for (auto& kv : graphs_) (void)hipGraphExecDestroy(kv.second);
  graphs_.clear();
}

// Fill the host blob: header, job table (all jobs) and work lists of the
// jobs listed in `only` (all jobs if empty), with tile configuration cfg[j],
// the tile list repeated `repeat` times (timing only: repeated tiles store
// identical values). Grows the buffers if needed (dropping graphs, whose
// arguments point into the old device buffer).
void Engine::build_blob(const std::vector<TileCfg>& cfg, const std::vector<int>& only, int repeat) {
  std::vector<int> sel = only;
  if (sel.empty())
    for (int j = 0; j < (int)jobs_.size(); j++) sel.push_back(j);
  std::vector<TileMap> maps(jobs_.size());
  int nt = 0, nc = 0;
  for (int j = 0; j < (int)jobs_.size(); j++)
    maps[j] = make_tilemap(jobs_[j].g->dev, cfg[j].band);
  for (int j : sel) {
    nt += maps[j].ntiles * repeat;
    const JobLists l = lists_of(j);
    nc += (l.gh[0].n_ghost + 255) / 256 + (l.gh[1].n_ghost + 255) / 256 + (l.rad.n + 255) / 256;
  }
  // the previous upload must have left the pinned buffer before it is reused
  if (upload_done_) (void)hipEventSynchronize(upload_done_);
  if ((int)jobs_.size() > cap_jobs_ || nt > cap_tiles_ || nc > cap_chunks_) {
    (void)hipDeviceSynchronize();
    drop_graphs();
    if (d_blob_) (void)hipFree(d_blob_);
    if (h_blob_) (void)hipHostFree(h_blob_);
    if (h_counts_) (void)hipHostFree(h_counts_);
    d_blob_ = h_blob_ = nullptr;
    h_counts_ = nullptr;
    cap_jobs_ = std::max<int>(cap_jobs_, (int)jobs_.size() * 3 / 2 + 1);
    cap_tiles_ = std::max(cap_tiles_, nt * 3 / 2 + 64);
    cap_chunks_ = std::max(cap_chunks_, nc * 3 / 2 + 64);
    const Layout L = layout(cap_jobs_, cap_tiles_, cap_chunks_);
    cap_bytes_ = L.total;
    if (hipMalloc((void**)&d_blob_, cap_bytes_) != hipSuccess ||
        hipHostMalloc((void**)&h_blob_, cap_bytes_, hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc((void**)&h_counts_, sizeof(int) * kRing * (size_t)cap_jobs_, hipHostMallocDefault) !=
            hipSuccess) {
      set_error("batch: cannot allocate the work description");
      cap_bytes_ = 0;
      cap_jobs_ = cap_tiles_ = cap_chunks_ = 0;
      return;
    }
  }
  const Layout L = layout(cap_jobs_, cap_tiles_, cap_chunks_);
  BatchHdr* hdr = (BatchHdr*)h_blob_;
  BatchJob* J = (BatchJob*)(h_blob_ + L.jobs);
  int2* tiles = (int2*)(h_blob_ + L.tiles);
  int2* chunks = (int2*)(h_blob_ + L.chunks);
  std::memset(hdr, 0, sizeof(BatchHdr));
  for (int j = 0; j < (int)jobs_.size(); j++) {
    const EngineJob& e = jobs_[j];
    BatchJob& b = J[j];
    b.G = e.g->dev;
    const JobLists l = lists_of(j);
    b.gh[0] = l.gh[0];
    b.gh[1] = l.gh[1];
    b.rad = l.rad;
    b.T = maps[j];
    const double* in[4] = {nullptr, nullptr, nullptr, nullptr};
    double* gd[4] = {nullptr, nullptr, nullptr, nullptr};
    if (integrator_ == BHAH_SSPRK3) {
      ssprk3_stages(e.dt, e.y, e.ws, e.g->info.state_doubles, b.st, in, gd);
      b.st[3] = StageArgs{};
    } else {
      rk4_stages(e.dt, e.y, e.ws, e.g->info.state_doubles, b.st, in, gd);
    }
    for (int k = 0; k < 4; k++) {
      b.in[k] = in[k];
      b.gdst[k] = gd[k];
    }
    b.st[4] = StageArgs{e.ws, nullptr, nullptr, 0.0, nullptr, 0.0, 0.0, nullptr, nullptr};
    b.in[4] = e.y;
    b.gdst[4] = nullptr;
  }
  int pos = 0;
  for (int f = 0; f < NVAR; f++) {
    hdr->tile_off[f] = pos;
    for (int r = 0; r < repeat; r++)
      for (int j : sel) {
        const GridDev& G = jobs_[j].g->dev;
        if (rhs_variant(G.coord, G.N1, G.N2, G.ng) != f) continue;
        for (int t = 0; t < maps[j].ntiles; t++) tiles[pos++] = int2{j, t};
      }
    hdr->n_tiles[f] = pos - hdr->tile_off[f];
  }
  int cpos = 0;
  for (int w = 0; w < 3; w++) {
    hdr->chunk_off[w] = cpos;
    for (int j : sel) {
      const JobLists l = lists_of(j);
      const int pts = w < 2 ? l.gh[w].n_ghost : l.rad.n;
      const int n = (pts + 255) / 256;
      for (int c = 0; c < n; c++) chunks[cpos++] = int2{j, c};
    }
    hdr->n_chunks[w] = cpos - hdr->chunk_off[w];
  }
  n_tiles_ = pos;
  n_chunks_ = cpos;
  blob_bytes_ = (size_t)(L.chunks + sizeof(int2) * (size_t)cpos);
}

int Engine::upload(hipStream_t s) {
  if (!d_blob_) return fail(BHAH_ENOMEM, "batch: no work description buffer");
  int rc = check_hip(hipMemcpyAsync(d_blob_, h_blob_, blob_bytes_, hipMemcpyHostToDevice, s), "batch upload");
  if (rc) return rc;
  return check_hip(hipEventRecord(upload_done_, s), "hipEventRecord");
}

int Engine::upload_counts(long long first, int k, hipStream_t s) {
  if (!d_blob_ || !h_counts_) return fail(BHAH_ENOMEM, "batch: no work description buffer");
  const int slot = counts_slot_;
  counts_slot_ = (counts_slot_ + 1) % kRing;
  int rc = check_hip(hipEventSynchronize(counts_done_[slot]), "batch counts slot");
  if (rc) return rc;
  int* h = h_counts_ + (size_t)slot * cap_jobs_;
  for (size_t j = 0; j < jobs_.size(); j++) {
    const long long lim = jobs_[j].limit < 0 ? first + k : jobs_[j].limit;
    h[j] = (int)std::max<long long>(0, std::min<long long>(k, lim - first));
  }
  const Layout L = layout(cap_jobs_, cap_tiles_, cap_chunks_);
  rc = check_hip(hipMemcpyAsync(d_blob_ + L.counts, h, sizeof(int) * jobs_.size(), hipMemcpyHostToDevice, s),
                 "batch counts upload");
  if (rc) return rc;
  return check_hip(hipEventRecord(counts_done_[slot], s), "hipEventRecord");
}

int Engine::time_class(const SizeClass& c, const TileCfg& cfg, hipStream_t s, double* us) {
  std::vector<int> only;
  std::vector<TileCfg> cfgs(jobs_.size(), TileCfg{6, 0, 1});
  long long tiles = 0;
  for (int j = 0; j < (int)jobs_.size(); j++)
    if (class_of(jobs_[j].g) == c) {
      only.push_back(j);
      cfgs[j] = cfg;
      tiles += make_tilemap(jobs_[j].g->dev, cfg.band).ntiles;
    }
  // time the class at full occupancy: repeat its tiles until every
  // persistent block slot sees several
  const long long target = 16LL * n_cus_;
  const int repeat = (int)std::max<long long>(1, (target + tiles - 1) / std::max<long long>(tiles, 1));
  build_blob(cfgs, only, repeat);
  int rc = upload(s);
  if (rc) return rc;
  const Layout L = layout(cap_jobs_, cap_tiles_, cap_chunks_);
  const BatchJob* dj = (const BatchJob*)(d_blob_ + L.jobs);
  const BatchHdr* dh = (const BatchHdr*)d_blob_;
  const int2* dt = (const int2*)(d_blob_ + L.tiles);
  // the kernel variants of the class's jobs (4th- and 8th-order grids of one
  // shape share the class), launched in the form that the whole job set gets
  const ListSizes all = list_sizes();
  long long own[NVAR] = {};
  for (int j : only) {
    const GridDev& G = jobs_[j].g->dev;
    own[rhs_variant(G.coord, G.N1, G.N2, G.ng)] += (long long)repeat * make_tilemap(G, cfg.band).ntiles;
  }
  int blocks[NVAR];
  for (int v = 0; v < NVAR; v++) blocks[v] = rhs_grid(all.tiles[v], own[v]);
  hipEvent_t e0, e1;
  if ((rc = check_hip(hipEventCreate(&e0), "hipEventCreate"))) return rc;
  if ((rc = check_hip(hipEventCreate(&e1), "hipEventCreate"))) { (void)hipEventDestroy(e0); return rc; }
  const int reps = 3;
  for (int v = 0; v < NVAR; v++)
    if (blocks[v]) launch_rhs_batch(v, dj, dh, dt, 4, nullptr, 0, gauge_of(gp_), blocks[v], s);
  (void)hipEventRecord(e0, s);
  for (int r = 0; r < reps; r++)
    for (int v = 0; v < NVAR; v++)
      if (blocks[v]) launch_rhs_batch(v, dj, dh, dt, 4, nullptr, 0, gauge_of(gp_), blocks[v], s);
  (void)hipEventRecord(e1, s);
  rc = check_hip(hipEventSynchronize(e1), "tile timing");
  float ms = 0.f;
  if (!rc) rc = check_hip(hipEventElapsedTime(&ms, e0, e1), "hipEventElapsedTime");
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  *us = 1e3 * ms / reps / repeat;
  return rc;
}

int Engine::tune_missing(hipStream_t s) {
  std::set<SizeClass> todo;
  for (const EngineJob& j : jobs_)
    if (!tuned_.count(class_of(j.g))) todo.insert(class_of(j.g));
  if (todo.empty()) return BHAH_OK;
  const double t0 = now_s();
  for (const SizeClass& c : todo) {
    double best = 1e300;
    TileCfg bc{6, 0, 1};
    for (const TileCfg& cfg : tile_candidates(c)) {
      double us = 0.0;
      const int rc = time_class(c, cfg, s, &us);
      if (rc) return rc;
      if (us < best) {
        best = us;
        bc = cfg;
      }
    }
    tuned_[c] = bc;
    tuned_us_[c] = best;
  }
  tune_seconds_ += now_s() - t0;
  dirty_ = true;
  save_cache();
  return BHAH_OK;
}

int Engine::capture(int nsteps, const LaunchShape& shape, hipGraphExec_t* out) {
  const Layout L = layout(cap_jobs_, cap_tiles_, cap_chunks_);
  const BatchJob* dj = (const BatchJob*)(d_blob_ + L.jobs);
  const BatchHdr* dh = (const BatchHdr*)d_blob_;
  const int2* dt = (const int2*)(d_blob_ + L.tiles);
  const int2* dc = (const int2*)(d_blob_ + L.chunks);
  const int* dn = (const int*)(d_blob_ + L.counts);
  int rc = check_hip(hipStreamBeginCapture(cap_stream_, hipStreamCaptureModeThreadLocal), "graph capture");
  if (rc) return rc;
  // Step k of the graph runs the jobs with more than k active steps in this
  // launch (counts, uploaded before each launch). The stencils never read
  // phi ghost planes (they wrap phi onto the interior), so within a job's
  // steps only the ghosts with an interior phi index are filled; the last
  // stage of its last active step fills all of them.
  const int nst = integrator_ == BHAH_SSPRK3 ? 3 : 4;
  for (int k = 0; k < nsteps; k++)
    for (int stage = 0; stage < nst; stage++) {
      for (int f = 0; f < NVAR; f++)
        if (shape[f]) launch_rhs_batch(f, dj, dh, dt, stage, dn, k, gauge_of(gp_), shape[f], cap_stream_);
      // outer points of radiation-boundary jobs, before their inner ghosts are copied
      if (shape[NVAR]) launch_radiation_batch(dj, dh, dc, stage, dn, k, ghost_blocks_, cap_stream_);
      launch_ghosts_batch(dj, dh, dc, stage, dn, k, stage == nst - 1, ghost_blocks_, cap_stream_);
    }
  hipGraph_t graph = nullptr;
  const hipError_t le = hipGetLastError();
  rc = check_hip(hipStreamEndCapture(cap_stream_, &graph), "graph capture end");
  if (!rc && le != hipSuccess) rc = check_hip(le, "graph capture launch");
  if (rc) {
    if (graph) (void)hipGraphDestroy(graph);
    return rc;
  }
  rc = check_hip(hipGraphInstantiate(out, graph, nullptr, nullptr, 0), "hipGraphInstantiate");
  (void)hipGraphDestroy(graph);
  return rc;
}

// the graph of nsteps steps of the current job set, captured if no kept one
// launches the same kernels
int Engine::graph_for(int nsteps, hipStream_t s, hipGraphExec_t* out) {
  const LaunchShape shape = launch_shape();
  rhs_blocks_ = most_blocks(shape);
  const GraphKey key{nsteps, integrator_, shape};
  const auto it = graphs_.find(key);
  if (it != graphs_.end()) {
    *out = it->second;
    return BHAH_OK;
  }
  if (graphs_.size() >= kMaxGraphs) {
    if (int rc = check_hip(hipStreamSynchronize(s), "batch graphs")) return rc;  // none of them still runs
    drop_graphs();
  }
  if (int rc = capture(nsteps, shape, out)) return rc;
  graphs_.emplace(key, *out);
  return BHAH_OK;
}

int Engine::step(int nsteps, hipStream_t s) {
  if (nsteps < 0) return fail(BHAH_EINVAL, "batch: nsteps < 0");
  if (jobs_.empty() || nsteps == 0) return BHAH_OK;
  int rc = ensure_device(s);
  if (rc) return rc;
  if ((rc = tune_missing(s))) return rc;
  if (dirty_) {
    std::vector<TileCfg> cfg;
    for (const EngineJob& j : jobs_) cfg.push_back(tile_of_class(class_of(j.g)));
    build_blob(cfg, {});
    if ((rc = upload(s))) return rc;
    dirty_ = false;
  }
  if (tune_launch_ && (rc = tune_launch(s))) return rc;
  // jobs that take fewer steps than the call idle through the rest: launch
  // graphs only while some job still has steps to take
  long long most = 0;
  for (const EngineJob& j : jobs_) most = std::max<long long>(most, j.limit < 0 ? nsteps : std::min<long long>(nsteps, j.limit));
  long long first = 0;
  while (first < most) {
    const int k = (int)std::min<long long>(most - first, graph_steps_);
    hipGraphExec_t ex = nullptr;
    if ((rc = graph_for(k, s, &ex))) return rc;
    if ((rc = upload_counts(first, k, s))) return rc;
    if ((rc = check_hip(hipGraphLaunch(ex, s), "hipGraphLaunch"))) return rc;
    first += k;
  }
  return BHAH_OK;
}

std::string Engine::launch_signature() const {
  std::map<std::string, int> count;
  for (const EngineJob& j : jobs_) {
    const bhah_grid_params& p = j.g->params;
    char b[96];
    std::snprintf(b, sizeof b, "%d:%dx%dx%d:%d:%d", p.coord, p.N[0], p.N[1], p.N[2], p.nghosts, p.bc_kind);
    count[b]++;
  }
  std::string full;
  for (auto& kv : count) full += std::to_string(kv.second) + "*" + kv.first + " ";
  unsigned long long h = 1469598103934665603ULL;  // FNV-1a, stable across runs and builds
  for (unsigned char c : full) h = (h ^ c) * 1099511628211ULL;
  char b[96];
  std::snprintf(b, sizeof b, "%s %zu jobs %016llx", integrator_ == BHAH_SSPRK3 ? "ssprk3" : "rk4", jobs_.size(), h);
  return b;
}

int Engine::tune_launch(hipStream_t s) {
  const std::string sig = launch_signature();
  const auto hit = launch_cache_.find(sig);
  if (hit != launch_cache_.end()) {
    // a choice stands for the launch that was timed: where its blocks per CU
    // come to another one here, the job set is timed again
    const LaunchChoice& c = hit->second;
    const int bpc = blocks_per_cu_;
    blocks_per_cu_ = c.blocks_per_cu;
    const bool same = c.blocks == 0 || c.blocks == most_blocks(launch_shape());
    blocks_per_cu_ = bpc;
    if (same) {
      if (c.graph_steps != graph_steps_ || c.blocks_per_cu != blocks_per_cu_) {
        set_graph_steps(c.graph_steps);
        set_blocks_per_cu(c.blocks_per_cu);
      }
      last_tune_.graph_steps = graph_steps_;
      last_tune_.blocks_per_cu = blocks_per_cu_;
      last_tune_.from_cache = true;
      last_tune_.us_per_step = c.us;
      return BHAH_OK;
    }
  }
  const double t0 = now_s();
  // copies of the states: the candidates run real steps
  size_t total = 0;
  for (const EngineJob& j : jobs_) total += (size_t)j.g->info.state_doubles;
  double* copies = nullptr;
  if (hipMalloc((void**)&copies, total * sizeof(double)) != hipSuccess) {
    (void)hipGetLastError();
    return fail(BHAH_ENOMEM, "batch: no device memory for the launch tuning's state copies");
  }
  const std::vector<EngineJob> saved = jobs_;
  size_t off = 0;
  int rc = BHAH_OK;
  for (EngineJob& j : jobs_) {
    const size_t n = (size_t)j.g->info.state_doubles;
    if (!rc) rc = check_hip(hipMemcpyAsync(copies + off, j.y, n * sizeof(double), hipMemcpyDeviceToDevice, s),
                            "launch tuning copy");
    j.y = copies + off;
    j.limit = -1;
    off += n;
  }
  std::vector<TileCfg> cfg;
  for (const EngineJob& j : jobs_) cfg.push_back(tile_of_class(class_of(j.g)));
  if (!rc) {
    build_blob(cfg, {});
    rc = upload(s);
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (!rc) rc = check_hip(hipEventCreate(&e0), "hipEventCreate");
  if (!rc) rc = check_hip(hipEventCreate(&e1), "hipEventCreate");
  // lists of more than 8 tiles per block come to one launch whatever the
  // blocks per CU: each launch is timed once, under the first of its names
  const int steps_c[3] = {4, 10, 25}, bpc_c[4] = {4, 2, 8, 0};
  int best_s = 10, best_b = 4;
  double best = 1e300, def = 0.0;
  std::set<std::pair<int, LaunchShape>> timed;
  for (int a = 0; a < 3 && !rc; a++)
    for (int b = 0; b < 4 && !rc; b++) {
      set_graph_steps(steps_c[a]);
      set_blocks_per_cu(bpc_c[b]);
      if (!timed.insert({graph_steps_, launch_shape()}).second) continue;
      hipGraphExec_t ex = nullptr;
      if ((rc = graph_for(graph_steps_, s, &ex))) break;
      if ((rc = upload_counts(0, graph_steps_, s))) break;
      (void)hipGraphLaunch(ex, s);  // warm-up
      (void)hipEventRecord(e0, s);
      for (int r = 0; r < 2; r++) (void)hipGraphLaunch(ex, s);
      (void)hipEventRecord(e1, s);
      if ((rc = check_hip(hipEventSynchronize(e1), "launch tuning"))) break;
      float ms = 0.f;
      (void)hipEventElapsedTime(&ms, e0, e1);
      const double us = 1e3 * ms / (2.0 * graph_steps_);
      if (steps_c[a] == 10 && bpc_c[b] == 4) def = us;
      if (us < best) {
        best = us;
        best_s = steps_c[a];
        best_b = bpc_c[b];
      }
    }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipStreamSynchronize(s);
  (void)hipFree(copies);
  jobs_ = saved;
  dirty_ = true;
  drop_graphs();
  if (rc) return rc;
  if (def > 0.0 && best >= def / 1.02) {  // within 2% of the default: keep it
    best_s = 10;
    best_b = 4;
    best = def;
  }
  set_graph_steps(best_s);
  set_blocks_per_cu(best_b);
  // the tuning blob held the copies: rebuild with the jobs' own states
  build_blob(cfg, {});
  if ((rc = upload(s))) return rc;
  dirty_ = false;
  launch_cache_[sig] = LaunchChoice{best_s, best_b, most_blocks(launch_shape()), best};
  last_tune_ = LaunchTune{best_s, best_b, best, def, now_s() - t0, (int)timed.size(), false};
  save_cache();
  return BHAH_OK;
}

// ---- tile cache: one JSON object per line inside an "entries" array -----
void Engine::load_cache() {
  if (cache_path_.empty()) return;
  FILE* f = std::fopen(cache_path_.c_str(), "r");
  if (!f) return;
  char line[512];
  while (std::fgets(line, sizeof line, f)) {
    char arch[64];
    int coord, n0, n1, n2, lx, ly, band;
    double us;
    const char* p = std::strchr(line, '{');
    if (!p) continue;
    {  // a launch-configuration entry
      char sig[96];
      int S, bpc, blocks = 0;
      if (std::sscanf(p,
                      "{\"arch\": \"%63[^\"]\", \"launch\": \"%95[^\"]\", \"S\": %d, \"bpc\": %d, \"us\": %lf, "
                      "\"blocks\": %d}",
                      arch, sig, &S, &bpc, &us, &blocks) >= 5) {
        if (arch_ == arch && S >= 1 && bpc >= 0) launch_cache_[sig] = LaunchChoice{S, bpc, std::max(blocks, 0), us};
        continue;
      }
    }
    if (std::sscanf(p, "{\"arch\": \"%63[^\"]\", \"coord\": %d, \"N\": [%d, %d, %d], \"lx\": %d, \"ly\": %d, "
                       "\"band\": %d, \"us\": %lf}",
                    arch, &coord, &n0, &n1, &n2, &lx, &ly, &band, &us) != 9)
      continue;
    if (arch_ != arch) continue;
    if (lx < 0 || ly < 0 || lx + ly > 6 || band < 1) continue;
    if (coord < 0 || coord > 2 || !tile_fits_periodic(coord, TileCfg{lx, ly, band})) continue;
    tuned_[SizeClass{coord, n0, n1, n2}] = TileCfg{lx, ly, band};
    tuned_us_[SizeClass{coord, n0, n1, n2}] = us;
  }
  std::fclose(f);
}

void Engine::save_cache() {
  if (cache_path_.empty()) return;
  // keep entries of other architectures that are in the file
  std::vector<std::string> keep;
  if (FILE* f = std::fopen(cache_path_.c_str(), "r")) {
    char line[512];
    while (std::fgets(line, sizeof line, f)) {
      const char* p = std::strstr(line, "{\"arch\": \"");
      if (!p) continue;
      const std::string a = std::string("{\"arch\": \"") + arch_ + "\"";
      if (std::strncmp(p, a.c_str(), a.size()) == 0) continue;
      std::string l(p);
      while (!l.empty() && (l.back() == '\n' || l.back() == ',' || l.back() == ' ')) l.pop_back();
      keep.push_back(l);
    }
    std::fclose(f);
  }
  const std::string tmp = cache_path_ + ".tmp";
  FILE* f = std::fopen(tmp.c_str(), "w");
  if (!f) return;
  std::fprintf(f, "{\"bhah_tile_cache\": 1, \"entries\": [\n");
  bool first = true;
  for (const std::string& l : keep) {
    std::fprintf(f, "%s%s", first ? "" : ",\n", l.c_str());
    first = false;
  }
  for (const auto& kv : tuned_) {
    const SizeClass& c = kv.first;
    const auto u = tuned_us_.find(c);
    std::fprintf(f,
                 "%s{\"arch\": \"%s\", \"coord\": %d, \"N\": [%d, %d, %d], \"lx\": %d, \"ly\": %d, \"band\": %d, "
                 "\"us\": %.3f}",
                 first ? "" : ",\n", arch_.c_str(), std::get<0>(c), std::get<1>(c), std::get<2>(c),
                 std::get<3>(c), kv.second.lx, kv.second.ly, kv.second.band,
                 u == tuned_us_.end() ? 0.0 : u->second);
    first = false;
  }
  for (const auto& kv : launch_cache_) {
    const LaunchChoice& c = kv.second;
    std::fprintf(f,
                 "%s{\"arch\": \"%s\", \"launch\": \"%s\", \"S\": %d, \"bpc\": %d, \"us\": %.3f, "
                 "\"blocks\": %d}",
                 first ? "" : ",\n", arch_.c_str(), kv.first.c_str(), c.graph_steps, c.blocks_per_cu, c.us, c.blocks);
    first = false;
  }
  std::fprintf(f, "\n]}\n");
  std::fclose(f);
  std::rename(tmp.c_str(), cache_path_.c_str());
}

}  // namespace bhah
