// Serving entry points: batched stepping of many resident contexts through
// the persistent batch kernel (with hipGraph replay of step sequences), its
// allocation-free variant, and the workgroup-size autotuner with its on-disk
// cache.
#include <hip/hip_runtime.h>
#include <sys/stat.h>

#include <algorithm>
#include <climits>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <map>
#include <mutex>
#include <sstream>
#include <string>
#include <vector>

#include "runtime.hpp"

namespace hrlbm {

// Steps captured per graph: each step is one batch launch plus a one-thread
// launch that advances the device step counter.
static constexpr int kBatchGraphSteps = 16;

struct BatchRunner {
  int device = -1;
  hipStream_t stream = nullptr;
  BatchJob* d_jobs = nullptr;
  size_t cap = 0;
  BatchHeader* d_hdr = nullptr;
  BatchJob* h_jobs = nullptr;  // pinned staging
  BatchHeader* h_hdr = nullptr;
  hipEvent_t staged = nullptr;  // the last upload finished reading staging
  hipStream_t capture = nullptr;
  // (kernel variant, block, or -fused steps)
  std::map<std::pair<int, int>, GraphEntry> graphs;
  std::map<std::pair<int, int>, int> grids;
  // Lanes: the second and later groups of a batch run on runners of their
  // own with their own streams, concurrently with the first group (on the
  // caller's stream): ordered after the caller's stream by `fork`, joined
  // back into it by each lane's `done`.
  std::vector<BatchRunner*> lanes;
  hipEvent_t fork = nullptr;
  hipEvent_t done = nullptr;
};

static std::mutex g_batch_mu;

static hipError_t setup_runner(BatchRunner* r) {
  hipError_t e = hipMalloc(&r->d_hdr, sizeof(BatchHeader));
  if (e == hipSuccess) e = hipHostMalloc((void**)&r->h_hdr, sizeof(BatchHeader), 0);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&r->staged, hipEventDisableTiming);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&r->fork, hipEventDisableTiming);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&r->done, hipEventDisableTiming);
  if (e == hipSuccess) e = hipStreamCreateWithFlags(&r->capture, hipStreamNonBlocking);
  return e;
}
static std::map<std::pair<int, hipStream_t>, BatchRunner*> g_runners;

static int runner_for(int device, hipStream_t st, BatchRunner** out) {
  auto key = std::make_pair(device, st);
  auto it = g_runners.find(key);
  if (it != g_runners.end()) {
    *out = it->second;
    return LBM_OK;
  }
  BatchRunner* r = new BatchRunner();
  r->device = device;
  r->stream = st;
  hipError_t e = setup_runner(r);
  if (e != hipSuccess) {
    delete r;
    return hip_error(e, "batch runner setup");
  }
  g_runners[key] = r;
  *out = r;
  return LBM_OK;
}

// Lane k of a runner (created on first use; streams at the default
// priority).
static int lane_for(BatchRunner* r, size_t k, BatchRunner** out) {
  while (r->lanes.size() <= k) {
    BatchRunner* l = new BatchRunner();
    l->device = r->device;
    hipError_t e = hipStreamCreateWithFlags(&l->stream, hipStreamNonBlocking);
    if (e == hipSuccess) e = setup_runner(l);
    if (e != hipSuccess) {
      if (l->stream) (void)hipStreamDestroy(l->stream);
      delete l;
      return hip_error(e, "batch lane setup");
    }
    r->lanes.push_back(l);
  }
  *out = r->lanes[k];
  return LBM_OK;
}

static int ensure_capacity(BatchRunner* r, size_t n) {
  if (n <= r->cap) return LBM_OK;
  hipError_t e = hipEventSynchronize(r->staged);
  if (e != hipSuccess) return hip_error(e, "batch staging wait");
  e = hipStreamSynchronize(r->stream);
  if (e != hipSuccess) return hip_error(e, "batch stream wait");
  size_t cap = std::max<size_t>(64, r->cap);
  while (cap < n) cap *= 2;
  if (r->d_jobs) (void)hipFree(r->d_jobs);
  if (r->h_jobs) (void)hipHostFree(r->h_jobs);
  r->d_jobs = nullptr;
  r->h_jobs = nullptr;
  e = hipMalloc(&r->d_jobs, cap * sizeof(BatchJob));
  if (e == hipSuccess) e = hipHostMalloc((void**)&r->h_jobs, cap * sizeof(BatchJob), 0);
  if (e != hipSuccess) {
    r->cap = 0;
    return hip_error(e, "batch table allocation");
  }
  r->cap = cap;
  // graphs captured the old table pointer
  for (auto& kv : r->graphs) {
    (void)hipGraphExecDestroy(kv.second.exec);
    (void)hipGraphDestroy(kv.second.graph);
  }
  r->graphs.clear();
  return LBM_OK;
}

static int graph_for(BatchRunner* r, int variant, int fused, int block, int grid,
                     GraphEntry** out) {
  const int launches = kBatchGraphSteps / fused;
  auto key = std::make_pair(variant, fused > 1 ? -fused : block);
  auto it = r->graphs.find(key);
  if (it == r->graphs.end()) {
    GraphEntry g{};
    hipError_t e = hipStreamBeginCapture(r->capture, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return hip_error(e, "batch capture begin");
    // launches base + 0 ... base + launches - 1, then base += launches
    for (int k = 0; k < launches && e == hipSuccess; ++k)
      e = launch_batch(variant, fused, r->d_jobs, r->d_hdr, (int32_t)k, block, grid, r->capture);
    if (e == hipSuccess) e = launch_batch_bump(r->d_hdr, (int32_t)launches, r->capture);
    hipGraph_t graph = nullptr;
    hipError_t e2 = hipStreamEndCapture(r->capture, &graph);
    if (e != hipSuccess) return hip_error(e, "batch launch during capture");
    if (e2 != hipSuccess) return hip_error(e2, "batch capture end");
    e = hipGraphInstantiate(&g.exec, graph, nullptr, nullptr, 0);
    if (e != hipSuccess) {
      (void)hipGraphDestroy(graph);
      return hip_error(e, "batch graph instantiate");
    }
    g.graph = graph;
    it = r->graphs.emplace(key, g).first;
  }
  *out = &it->second;
  return LBM_OK;
}

// Batch kernel variant of a context: lattice code, storage, sweep path.
static int batch_variant(const lbm_ctx* c) {
  const SweepHost h = sweep_args(c, 0, 0, 0);
  return sweep_lattice(c->cfg) * 16 + c->cfg.storage * 2 + (h.general ? 1 : 0);
}

// A group is stepped in passes where they are expected to take under this share
// of the time of single steps.  Beside other groups single steps compete for
// memory, which passes spare, so there passes are kept unless they are clearly
// slower.  ms of 64 steps, single / passes: alone, eight FP32 channels of
// 300 x 280 1.05 / 0.93, one of 300 x 300 0.48 / 0.55, two FP16S ones of 2000 x 1000
// 2.9 / 4.6; four groups together, 12 jobs of 256 to 2048 cells a side 7.0 / 6.4, of 128
// to 512 1.17 / 1.04.
constexpr double kPaysAlone = 0.95, kPaysBeside = 1.5;
// A job whose pass takes more than this many times its single steps at full
// load has a grid too narrow for the tiles; it takes single steps in any group
// (64 steps of eight FP32 channels of 8 x 20000: 1.8 ms, 10.7 in passes).
constexpr double kNarrow = 2.0;

static bool takes_passes(const lbm_ctx* c, int fused) {
  if (fused == 1) return false;
  const bool general = sweep_args(c, 0, 0, 0).general;
  const uint32_t nx = (uint32_t)c->cfg.nx, ny = (uint32_t)c->cfg.ny;
  return nx >= 4 && ny >= 4 &&
         batch2d_time(c->cfg.storage, general, nx, ny).cells <
             kNarrow * fused * step2d_time(c->cfg.storage, general, true, nx, ny).cells;
}

// Steps the `count` contexts ctx(0), ctx(1), ... of a group take at a time (1:
// single steps): the time of passes is that of the jobs that take them and, in
// launches of their own, of the single steps of the others.
template <class F>
static int group_fused(size_t count, bool alone, F&& ctx) {
  const lbm_ctx* c0 = ctx(0);
  const bool general = sweep_args(c0, 0, 0, 0).general;
  if (c0->cfg.lattice != LBM_D2Q9 || (c0->cfg.flags & (LBM_BGK | LBM_MRT))) return 1;
  const int steps = batch2d_steps(c0->cfg.storage, general);
  Time2d step{}, pass{};
  double all = 0, passes = 0, beside = 0;  // cells of single steps, of passes, of the steps beside
  for (size_t k = 0; k < count; ++k) {
    const lbm_ctx* c = ctx(k);
    const uint32_t nx = (uint32_t)c->cfg.nx, ny = (uint32_t)c->cfg.ny;
    step = step2d_time(c->cfg.storage, general, true, nx, ny);
    pass = batch2d_time(c->cfg.storage, general, nx, ny);
    const bool takes = takes_passes(c, steps);
    all += step.cells;
    (takes ? passes : beside) += takes ? pass.cells : step.cells;
  }
  if (passes == 0) return 1;
  const double mixed = (pass.launch + passes) / steps + (beside > 0 ? step.launch + beside : 0.0);
  return mixed < (alone ? kPaysAlone : kPaysBeside) * (step.launch + all) ? steps : 1;
}

// The batch table entry of a context.
static void fill_job(BatchJob& J, lbm_ctx* c, int64_t steps, int fused, int block,
                     uint32_t tile_begin, uint32_t ftile_begin) {
  const Level& L = c->lv[0];
  std::memset(&J, 0, sizeof J);
  J.h = sweep_args(c, 0, L.cur, 0);
  J.buf[0] = L.buf[0];
  J.buf[1] = L.buf[1];
  J.storage = c->cfg.storage;
  J.cur0 = L.cur;
  J.t0 = (uint64_t)L.t;
  J.steps = steps;
  if (takes_passes(c, fused)) {
    J.flips0 = steps / fused;
    J.done0 = J.flips0 * fused;
  }
  J.tile_begin = tile_begin;
  J.ftile_begin = ftile_begin;
  J.ntiles = (uint32_t)((L.N + block - 1) / block);
  fill_fastdiv((uint32_t)L.nx, J.div_nx);
  fill_fastdiv((uint32_t)L.ny, J.div_ny);
}

// What the launches of a group cover.
struct GroupPlan {
  int64_t fused_launches = 0, single_launches = 0;
  uint32_t tiles = 0, ftiles = 0;
  void add(const lbm_ctx* c, const BatchJob& J) {
    fused_launches = std::max(fused_launches, J.flips0);
    single_launches = std::max(single_launches, J.steps - J.done0);
    tiles += J.ntiles;
    ftiles += multi2d_tiles((uint32_t)c->cfg.nx, (uint32_t)c->cfg.ny);
  }
};

// A context after its steps of a batch.
static void advance_job(lbm_ctx* c, const BatchJob& J) {
  c->lv[0].t += J.steps;
  c->lv[0].cur ^= (int)((J.flips0 + J.steps - J.done0) & 1);
  c->t += J.steps;
}

// One batch of contexts sharing a kernel variant and workgroup size (alone: the
// only group of the call).
static int run_group(BatchRunner* r, const std::vector<std::pair<lbm_ctx*, int64_t>>& grp,
                     bool alone) {
  lbm_ctx* c0 = grp[0].first;
  const int variant = batch_variant(c0);
  const int block = c0->block;
  int rc = ensure_capacity(r, grp.size());
  if (rc != LBM_OK) return rc;
  hipError_t e = hipEventSynchronize(r->staged);
  if (e != hipSuccess) return hip_error(e, "batch staging wait");
  const int fused = group_fused(grp.size(), alone, [&](size_t k) { return grp[k].first; });
  GroupPlan plan;
  for (size_t k = 0; k < grp.size(); ++k) {
    fill_job(r->h_jobs[k], grp[k].first, grp[k].second, fused, block, plan.tiles, plan.ftiles);
    plan.add(grp[k].first, r->h_jobs[k]);
  }
  if (plan.fused_launches + plan.single_launches == 0) return LBM_OK;
  r->h_hdr->njobs = (uint32_t)grp.size();
  r->h_hdr->total_tiles = plan.tiles;
  r->h_hdr->total_ftiles = plan.ftiles;
  r->h_hdr->step = 0;
  e = hipMemcpyAsync(r->d_jobs, r->h_jobs, grp.size() * sizeof(BatchJob),
                     hipMemcpyHostToDevice, r->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(r->d_hdr, r->h_hdr, sizeof(BatchHeader), hipMemcpyHostToDevice,
                       r->stream);
  if (e == hipSuccess) e = hipEventRecord(r->staged, r->stream);
  if (e != hipSuccess) return hip_error(e, "batch table upload");
  const bool use_graph = !(c0->cfg.flags & LBM_NO_GRAPH);
  int64_t base = 0;  // the device-side step index, advanced by the graphs
  // `count` launches, index 0 ... count - 1, of the fused or the one-step
  // kernel
  auto launches = [&](int per_launch, int64_t count) -> int {
    if (count == 0) return LBM_OK;
    auto gk = std::make_pair(variant, per_launch > 1 ? -per_launch : block);
    if (!r->grids.count(gk)) r->grids[gk] = batch_grid(variant, per_launch, block);
    const int grid = r->grids[gk];
    if (grid <= 0) return set_error(LBM_EDEVICE, "batch occupancy query failed");
    int64_t done = 0;
    const int64_t per = kBatchGraphSteps / per_launch;
    // (a graph counts from the index the device holds)
    if (use_graph && base == 0 && count >= per) {
      GraphEntry* g = nullptr;
      const int rc2 = graph_for(r, variant, per_launch, block, grid, &g);
      if (rc2 != LBM_OK) return rc2;
      for (; done + per <= count; done += per) {
        e = hipGraphLaunch(g->exec, r->stream);
        if (e != hipSuccess) return hip_error(e, "batch graph launch");
      }
      base = done;
    }
    for (; done < count; ++done) {
      e = launch_batch(variant, per_launch, r->d_jobs, r->d_hdr, (int32_t)(done - base), block,
                       grid, r->stream);
      if (e != hipSuccess) return hip_error(e, "batch launch");
    }
    return LBM_OK;
  };
  rc = launches(fused, plan.fused_launches);
  if (rc == LBM_OK) rc = launches(1, plan.single_launches);
  if (rc != LBM_OK) return rc;
  for (size_t k = 0; k < grp.size(); ++k) advance_job(grp[k].first, r->h_jobs[k]);
  return LBM_OK;
}

// ------------------------------------------------------- allocation-free --
// lbm_step_batch_noalloc keeps its job tables in `scratch`, an array of
// static storage that every device the library runs on holds until the
// process ends: kNoAllocMaxJobs batch headers (one per group), then
// kNoAllocMaxJobs jobs.  Host code never uses the array's name as an
// address: the device address comes from hipGetSymbolAddress, once per
// device, and is what the kernels receive.
static constexpr int kNoAllocMaxJobs = LBM_NOALLOC_MAX_JOBS;
static constexpr size_t kNoAllocHdrBytes = kNoAllocMaxJobs * sizeof(BatchHeader);
static constexpr size_t kNoAllocBytes = kNoAllocHdrBytes + kNoAllocMaxJobs * sizeof(BatchJob);
static_assert(kNoAllocHdrBytes % 256 == 0, "job table alignment");
static __device__ __align__(256) unsigned char scratch[kNoAllocBytes];

static constexpr int kScratchDevices = 64;
static std::mutex g_scratch_mu;
static unsigned char* g_scratch[kScratchDevices] = {};

// Device address of `scratch` on `device`, which must be current.
static int scratch_for(int device, unsigned char** out) {
  if (device < 0 || device >= kScratchDevices)
    return set_error(LBM_EINVAL, "device %d beyond the %d the allocation-free tables cover",
                     device, kScratchDevices);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch[device]) {
    void* p = nullptr;
    hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_error(e, "address of the allocation-free job tables");
    if (!p) return set_error(LBM_EDEVICE, "allocation-free job tables have no address");
    g_scratch[device] = (unsigned char*)p;
  }
  *out = g_scratch[device];
  return LBM_OK;
}

// Jobs written per table launch: the chunk travels as the kernel argument.
static constexpr int kTableChunk = 2;
struct TableChunk {
  BatchHeader hdr;     // the group's header, written with the first chunk
  uint32_t count;      // jobs in this chunk
  uint32_t write_hdr;
  BatchJob jobs[kTableChunk];
};

// One thread copies the chunk from its kernel argument into the tables
// (plain global stores); the batch launches that follow on the same stream
// read them.
__global__ void k_write_table(TableChunk c, BatchHeader* hdr, BatchJob* jobs) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
#pragma unroll
  for (int k = 0; k < kTableChunk; ++k)
    if ((uint32_t)k < c.count) jobs[k] = c.jobs[k];
  if (c.write_hdr) *hdr = c.hdr;
}

// One group (contexts order[0..count) sharing kernel variant and workgroup
// size) through the tables at hdr / jobs: upload by kernel arguments, then
// one batch launch per step with the step as the launch's offset (the
// header's base stays 0).  No graphs, no host staging, no allocation.
static int run_group_noalloc(lbm_ctx* const* ctxs, const int64_t* steps, const int* order,
                             int count, BatchHeader* hdr, BatchJob* jobs) {
  lbm_ctx* c0 = ctxs[order[0]];
  const int variant = batch_variant(c0);
  const int block = c0->block;
  hipStream_t st = c0->stream;
  const int fused = group_fused((size_t)count, true, [&](size_t k) { return ctxs[order[k]]; });
  GroupPlan plan;
  for (int k = 0; k < count; ++k) {
    BatchJob J;
    fill_job(J, ctxs[order[k]], steps[order[k]], fused, block, 0, 0);
    plan.add(ctxs[order[k]], J);
  }
  if (plan.fused_launches + plan.single_launches == 0) return LBM_OK;
  TableChunk chunk;
  uint32_t tile_begin = 0, ftile_begin = 0;
  for (int k0 = 0; k0 < count; k0 += kTableChunk) {
    std::memset(&chunk, 0, sizeof chunk);
    chunk.count = (uint32_t)std::min(kTableChunk, count - k0);
    for (uint32_t k = 0; k < chunk.count; ++k) {
      const int j = order[k0 + (int)k];
      fill_job(chunk.jobs[k], ctxs[j], steps[j], fused, block, tile_begin, ftile_begin);
      tile_begin += chunk.jobs[k].ntiles;
      ftile_begin += multi2d_tiles((uint32_t)ctxs[j]->cfg.nx, (uint32_t)ctxs[j]->cfg.ny);
    }
    if (k0 == 0) {
      chunk.write_hdr = 1;
      chunk.hdr.njobs = (uint32_t)count;
      chunk.hdr.total_tiles = plan.tiles;
      chunk.hdr.total_ftiles = plan.ftiles;
      chunk.hdr.step = 0;
    }
    hipLaunchKernelGGL(k_write_table, dim3(1), dim3(64), 0, st, chunk, hdr, jobs + k0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_error(e, "allocation-free table upload");
  }
  auto launches = [&](int per_launch, int64_t n) -> int {
    if (n == 0) return LBM_OK;
    const int grid = batch_grid(variant, per_launch, block);
    if (grid <= 0) return set_error(LBM_EDEVICE, "batch occupancy query failed");
    for (int64_t s = 0; s < n; ++s) {
      hipError_t e = launch_batch(variant, per_launch, jobs, hdr, (int32_t)s, block, grid, st);
      if (e != hipSuccess) return hip_error(e, "batch launch");
    }
    return LBM_OK;
  };
  int rc = launches(fused, plan.fused_launches);
  if (rc == LBM_OK) rc = launches(1, plan.single_launches);
  if (rc != LBM_OK) return rc;
  for (int k = 0; k < count; ++k) {
    BatchJob J;
    fill_job(J, ctxs[order[k]], steps[order[k]], fused, block, 0, 0);
    advance_job(ctxs[order[k]], J);
  }
  return LBM_OK;
}

// Checks shared by the batched entry points: every context initialised,
// unrefined, population-stored, without halo faces, on one device and stream,
// listed once, with a non-negative step count.
static int check_batch(lbm_ctx* const* ctxs, const int64_t* steps, int n) {
  for (int k = 0; k < n; ++k) {
    int rc = check_ready(ctxs[k]);
    if (rc != LBM_OK) return rc;
    if (steps[k] < 0) return set_error(LBM_EINVAL, "negative step count for job %d", k);
    if (ctxs[k]->nlevels > 1)
      return set_error(LBM_EUNSUPPORTED, "refined contexts cannot be batched");
    if (moment_storage(ctxs[k]->cfg.storage))
      return set_error(LBM_EUNSUPPORTED, "moment-stored contexts cannot be batched");
    if (has_halo(ctxs[k]->cfg))
      return set_error(LBM_EUNSUPPORTED, "contexts with halo faces cannot be batched");
    if (ctxs[k]->device != ctxs[0]->device || ctxs[k]->stream != ctxs[0]->stream)
      return set_error(LBM_EINVAL, "batched contexts must share device and stream");
    for (int m = 0; m < k; ++m)
      if (ctxs[m] == ctxs[k]) return set_error(LBM_EINVAL, "context %d appears twice", k);
  }
  return LBM_OK;
}

// ---------------------------------------------------------------- tuning --
static std::mutex g_tune_mu;

static std::string tune_path() {
  const char* p = std::getenv("HRLBM_TUNE_CACHE");
  if (p && *p) return p;
  const char* home = std::getenv("HOME");
  return std::string(home ? home : "/tmp") + "/.cache/hrlbm_tune.json";
}

// flat JSON object {"key": int, ...}
static std::map<std::string, int> read_cache() {
  std::map<std::string, int> m;
  std::ifstream f(tune_path());
  if (!f) return m;
  std::stringstream ss;
  ss << f.rdbuf();
  const std::string s = ss.str();
  size_t i = 0;
  while ((i = s.find('"', i)) != std::string::npos) {
    const size_t j = s.find('"', i + 1);
    if (j == std::string::npos) break;
    const std::string key = s.substr(i + 1, j - i - 1);
    const size_t colon = s.find(':', j);
    if (colon == std::string::npos) break;
    m[key] = std::atoi(s.c_str() + colon + 1);
    i = s.find_first_of(",}", colon);
    if (i == std::string::npos) break;
  }
  return m;
}

static void write_cache(const std::map<std::string, int>& m) {
  const std::string path = tune_path();
  const size_t slash = path.rfind('/');
  if (slash != std::string::npos) {
    const std::string dir = path.substr(0, slash);
    for (size_t k = 1; k <= dir.size(); ++k)
      if (k == dir.size() || dir[k] == '/') {
        const std::string part = dir.substr(0, k);
        (void)::mkdir(part.c_str(), 0755);
      }
  }
  const std::string tmp = path + ".tmp";
  std::ofstream f(tmp);
  if (!f) return;
  f << "{";
  bool first = true;
  for (auto& kv : m) {
    f << (first ? "" : ",") << "\n  \"" << kv.first << "\": " << kv.second;
    first = false;
  }
  f << "\n}\n";
  f.close();
  (void)std::rename(tmp.c_str(), path.c_str());
}

// (arch, lattice, storage, path, size class) key of the tuning cache
std::string tune_key(const lbm_ctx* ctx) {
  hipDeviceProp_t prop{};
  std::string arch = "gpu";
  if (hipGetDeviceProperties(&prop, ctx->device) == hipSuccess) arch = prop.gcnArchName;
  const size_t colon = arch.find(':');
  if (colon != std::string::npos) arch = arch.substr(0, colon);
  const Level& L = ctx->lv[0];
  int cls = 0;
  for (int64_t n = L.N; n > 1; n >>= 2) ++cls;  // log4 of the cell count
  const SweepHost h = sweep_args(ctx, 0, 0, 0);
  char buf[128];
  std::snprintf(buf, sizeof buf, "%s/q%d/s%d/%s/n4^%d", arch.c_str(), sweep_lattice(ctx->cfg),
                ctx->cfg.storage, h.general ? "general" : "periodic", cls);
  return buf;
}

int tuned_block(const lbm_ctx* ctx) {
  std::lock_guard<std::mutex> lk(g_tune_mu);
  const auto m = read_cache();
  auto it = m.find(tune_key(ctx));
  if (it == m.end()) return 0;
  const int b = it->second;
  return (b >= 64 && b <= 1024 && b % 64 == 0) ? b : 0;
}

}  // namespace hrlbm

using namespace hrlbm;

extern "C" {

int lbm_step_batch(lbm_ctx* const* ctxs, const int64_t* steps, int n) {
  if (n < 0 || (n > 0 && (!ctxs || !steps))) return set_error(LBM_EINVAL, "batch arguments");
  if (n == 0) return LBM_OK;
  int rc = check_batch(ctxs, steps, n);
  if (rc != LBM_OK) return rc;
  rc = ensure_device(ctxs[0]);
  if (rc != LBM_OK) return rc;
  std::lock_guard<std::mutex> lk(g_batch_mu);
  BatchRunner* r = nullptr;
  rc = runner_for(ctxs[0]->device, ctxs[0]->stream, &r);
  if (rc != LBM_OK) return rc;
  // one persistent launch sequence per (kernel variant, workgroup size)
  std::map<std::pair<int, int>, std::vector<std::pair<lbm_ctx*, int64_t>>> groups;
  for (int k = 0; k < n; ++k)
    groups[std::make_pair(batch_variant(ctxs[k]), ctxs[k]->block)].push_back(
        {ctxs[k], steps[k]});
  if (groups.size() == 1) return run_group(r, groups.begin()->second, true);
  // groups after the first run concurrently on lanes (one stream each):
  // a small group's launches fill the device poorly on their own
  hipError_t e = hipEventRecord(r->fork, r->stream);
  if (e != hipSuccess) return hip_error(e, "batch fork");
  size_t g = 0;
  for (auto& kv : groups) {
    BatchRunner* x = r;
    if (g > 0) {
      rc = lane_for(r, g - 1, &x);
      if (rc != LBM_OK) break;
      e = hipStreamWaitEvent(x->stream, r->fork, 0);
      if (e != hipSuccess) {
        rc = hip_error(e, "batch lane wait");
        break;
      }
    }
    rc = run_group(x, kv.second, false);
    if (g > 0) {
      e = hipEventRecord(x->done, x->stream);
      if (e == hipSuccess) e = hipStreamWaitEvent(r->stream, x->done, 0);
      if (e != hipSuccess && rc == LBM_OK) rc = hip_error(e, "batch lane join");
    }
    if (rc != LBM_OK) break;
    ++g;
  }
  return rc;
}

int lbm_step_batch_noalloc(lbm_ctx* const* ctxs, const int64_t* steps, int n) {
  if (n < 0 || (n > 0 && (!ctxs || !steps))) return set_error(LBM_EINVAL, "batch arguments");
  if (n > kNoAllocMaxJobs)
    return set_error(LBM_EINVAL, "%d contexts; the allocation-free batch takes at most %d", n,
                     kNoAllocMaxJobs);
  if (n == 0) return LBM_OK;
  int rc = check_batch(ctxs, steps, n);
  if (rc != LBM_OK) return rc;
  for (int k = 0; k < n; ++k)
    if (steps[k] > INT32_MAX)
      return set_error(LBM_EINVAL, "step count of job %d beyond 2^31 - 1", k);
  rc = ensure_device(ctxs[0]);
  if (rc != LBM_OK) return rc;
  unsigned char* base = nullptr;
  rc = scratch_for(ctxs[0]->device, &base);
  if (rc != LBM_OK) return rc;
  BatchHeader* hdrs = (BatchHeader*)base;
  BatchJob* jobs = (BatchJob*)(base + kNoAllocHdrBytes);
  // group by (kernel variant, workgroup size), stable in the callers' order
  int var[kNoAllocMaxJobs], order[kNoAllocMaxJobs];
  for (int k = 0; k < n; ++k) {
    var[k] = batch_variant(ctxs[k]);
    order[k] = k;
  }
  auto before = [&](int a, int b) {
    if (var[a] != var[b]) return var[a] < var[b];
    if (ctxs[a]->block != ctxs[b]->block) return ctxs[a]->block < ctxs[b]->block;
    return a < b;
  };
  for (int i = 1; i < n; ++i)
    for (int j = i; j > 0 && before(order[j], order[j - 1]); --j) std::swap(order[j], order[j - 1]);
  int groups = 0;
  for (int g0 = 0; g0 < n;) {
    int g1 = g0 + 1;
    while (g1 < n && var[order[g1]] == var[order[g0]] &&
           ctxs[order[g1]]->block == ctxs[order[g0]]->block)
      ++g1;
    // group `groups` uses header `groups` and the jobs from position g0 on
    rc = run_group_noalloc(ctxs, steps, order + g0, g1 - g0, hdrs + groups, jobs + g0);
    if (rc != LBM_OK) return rc;
    ++groups;
    g0 = g1;
  }
  return LBM_OK;
}

int lbm_autotune(lbm_ctx* ctx, int trials) {
  int rc = check_ready(ctx);
  if (rc != LBM_OK) return rc;
  if (trials < 1) trials = 1;
  rc = ensure_device(ctx);
  if (rc != LBM_OK) return rc;
  // Each trial sweeps the current state into the other buffer without
  // swapping: the current state is untouched, the other buffer is scratch
  // (cells the sweep never writes keep their values).
  const Level& L = ctx->lv[0];
  const int cands[] = {64, 128, 256, 512, 1024};
  hipEvent_t a, b;
  hipError_t e = hipEventCreate(&a);
  if (e == hipSuccess) e = hipEventCreate(&b);
  if (e != hipSuccess) return hip_error(e, "autotune events");
  SweepHost h = sweep_args(ctx, 0, L.cur, (uint64_t)(L.t + 1));
  // the timing sweeps leave the halo send buffers as they are
  h.hsend[0] = h.hsend[1] = nullptr;
  const int reps = std::max(3, (int)std::min<int64_t>(50, (int64_t)(2e8 / (double)L.N)));
  float best_ms = 1e30f;
  int best = ctx->block;
  for (int blk : cands) {
    e = launch_step_kernel(ctx, h, blk, ctx->stream);
    if (e != hipSuccess) break;
    float tot = 0.f;
    for (int t = 0; t < trials && e == hipSuccess; ++t) {
      e = hipEventRecord(a, ctx->stream);
      for (int k = 0; k < reps && e == hipSuccess; ++k)
        e = launch_step_kernel(ctx, h, blk, ctx->stream);
      if (e == hipSuccess) e = hipEventRecord(b, ctx->stream);
      if (e == hipSuccess) e = hipEventSynchronize(b);
      float ms = 0.f;
      if (e == hipSuccess) e = hipEventElapsedTime(&ms, a, b);
      tot += ms;
    }
    if (e != hipSuccess) break;
    if (tot < best_ms) {
      best_ms = tot;
      best = blk;
    }
  }
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  if (e != hipSuccess) return hip_error(e, "autotune");
  ctx->block = best;
  {
    std::lock_guard<std::mutex> lk(g_tune_mu);
    auto m = read_cache();
    m[tune_key(ctx)] = best;
    write_cache(m);
  }
  // graphs captured the old workgroup size
  for (auto& kv : ctx->graphs) {
    (void)hipGraphExecDestroy(kv.second.exec);
    (void)hipGraphDestroy(kv.second.graph);
  }
  ctx->graphs.clear();
  return best;
}

}  // extern "C"
