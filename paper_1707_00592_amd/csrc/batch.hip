// Many independent 1D problems of uneven length (isweno_batch_*).
//
// Layout: U[c * total + cell], problem p owns cells offsets[p] ..
// offsets[p+1]-1.  A step is two launches: one workgroup per problem forms its
// time step and copies the cells next to tile ends, then one workgroup per
// tile carries its tile through the three stages in place
// (batch_step_kernel).  Plans with a periodic end run one PERSISTENT launch
// per stage instead: a grid of (compute units x blocks per CU) workgroups
// walks a static list of tiles in round-robin order, so the assignment is
// deterministic and the launch count does not grow with the number of
// problems.  Ghost cells come from each problem's own boundary conditions, so
// tiles never straddle problems.  A step is captured once into a HIP graph and
// replayed.  The lanes per tile (and the grid size of the stage launches) are
// chosen by timing every candidate on the caller's data
// (isweno_batch_autotune).
#include "batch_kernels.hpp"

#include <algorithm>
#include <iterator>
#include <map>
#include <new>
#include <tuple>
#include <vector>

namespace isw {

// Start of a step, one workgroup per problem: a problem is advanced in this
// step when its status is still OK (active[p]); then, when cfl > 0,
// dt[p] = cfl / max_cells (|u| + c)/dx_p (clipped to dt_max), and with halo the
// cells next to tile ends are copied on the way.  Frozen problems keep their
// last dt.
__global__ __launch_bounds__(256) void batch_dt_kernel(const double* U, int64_t total,
                                                       const int64_t* offsets,
                                                       const double* dx, double cfl,
                                                       double dt_max, double* dt,
                                                       const int32_t* pstatus,
                                                       int32_t* active, int tc,
                                                       const int64_t* first, double* halo) {
  const int p = blockIdx.x;
  const int act = pstatus[p] == ST_OK;
  if (threadIdx.x == 0) active[p] = act;
  if (!act || !(cfl > 0.0)) return;
  const int64_t lo = offsets[p], n = offsets[p + 1] - lo;
  double m = 0.0;
  for (int64_t l = threadIdx.x; l < n; l += blockDim.x) {
    double u[5], q[5];
#pragma unroll
    for (int k = 0; k < 5; k++) u[k] = U[k * total + lo + l];
    if (halo) {
      // copies of the cells next to the ends of tiles of tc cells, for the
      // tiles on the other side: [tile][kHalo before it, kHalo after it][5]
      const int64_t t = n >> 31 ? l / tc : (int64_t)((unsigned)l / (unsigned)tc);
      const int pos = (int)(l - t * tc);
      if (pos < kHalo && t > 0) {
        double* d = halo + ((first[p] + t - 1) * 2 * kHalo + kHalo + pos) * 5;
#pragma unroll
        for (int k = 0; k < 5; k++) d[k] = u[k];
      }
      if (pos >= tc - kHalo && (t + 1) * tc < n) {
        double* d = halo + ((first[p] + t + 1) * 2 * kHalo + pos - (tc - kHalo)) * 5;
#pragma unroll
        for (int k = 0; k < 5; k++) d[k] = u[k];
      }
    }
    cons_prim<1>(u, q);
    const double cs = sqrt(sound2<double>(q[0], q[2], q[3], q[4]));
    const double s = (fabs(q[1]) + cs) / dx[p];
    m = (s > m || s != s) ? s : m;
  }
  __shared__ double red[256];
  red[threadIdx.x] = m;
  __syncthreads();
  for (unsigned o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      const double x = red[threadIdx.x + o];
      if (x > red[threadIdx.x] || x != x) red[threadIdx.x] = x;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double h = cfl / red[0];
    if (dt_max > 0.0 && h > dt_max) h = dt_max;
    dt[p] = h;
  }
}

// The copies of the cells next to tile ends alone, a group of 32 lanes per
// tile; the groups of problems' first tiles write active.  With fixed time
// steps there is nothing else to do at the start of a step (the kernel above
// walks every cell, one workgroup a problem: 8 tubes of 200 000 cells, float,
// 534 us a step, 58 so).
constexpr int kEdgeLanes = 32;
__global__ __launch_bounds__(256) void batch_edges_kernel(const double* U, int64_t total,
                                                          const int64_t* offsets,
                                                          const int64_t* tstart,
                                                          const int32_t* tprob, int64_t ntiles,
                                                          const int32_t* pstatus, int32_t* active,
                                                          int tc, double* halo) {
  const int64_t t = (int64_t)blockIdx.x * (256 / kEdgeLanes) + threadIdx.x / kEdgeLanes;
  const int k = threadIdx.x % kEdgeLanes;
  if (t >= ntiles) return;
  const int p = tprob[t];
  const int64_t lo = offsets[p], hi = offsets[p + 1], c0 = tstart[t];
  if (k == 0 && c0 == lo) active[p] = pstatus[p] == ST_OK;
  if (k >= 2 * kHalo) return;
  const int64_t c1 = c0 + tc < hi ? c0 + tc : hi;
  const int64_t cell = k < kHalo ? c0 - kHalo + k : c1 + (k - kHalo);
  if (cell < lo || cell >= hi) return;
  double u[5];
#pragma unroll
  for (int c = 0; c < 5; c++) u[c] = U[c * total + cell];
#pragma unroll
  for (int c = 0; c < 5; c++) halo[(t * 2 * kHalo + k) * 5 + c] = u[c];
}

static hipError_t launch_batch_stage(int precision, int tl, const BatchArgs& a, int mode,
                                     int blocks, hipStream_t s) {
  return precision == ISWENO_FP32 ? launch_batch_stage_f32(tl, a, mode, blocks, s)
                                  : launch_stage_t<double>(tl, a, mode, blocks, s);
}

static hipError_t launch_batch_step(int precision, int nthr, const BatchArgs& a, hipStream_t s) {
  return precision == ISWENO_FP32 ? launch_batch_step_f32(nthr, a, s)
                                  : launch_step_t<double>(nthr, a, s);
}

}  // namespace isw

// ---------------------------------------------------------------------------
// Plan
// ---------------------------------------------------------------------------
static const int kTiles[] = {63, 127, 255};
static const int kBlocksPerCU[] = {2, 4, 8, 16};
// Cells of a plan's longest problem from which batch_edges_kernel runs beside
// the start kernel instead of in it.  A problem is one workgroup's walk there
// and the copies lengthen it by about 0.46 us per 1000 cells, against about 1.5
// us for one more launch: 2 tubes of 500 000 cells 1250 us a step in one kernel
// and 1017 apart, 50 of 3000 to 9000 80 and 77, 100 of 2000 to 6000 92 and 90
// (float 56.0 and 56.3), 300 of 50 to 1500 82 and 83.
static const int64_t kLongWalk = 8192;

struct TileTable {
  int64_t* start = nullptr;
  int32_t* prob = nullptr;
  int64_t ntiles = 0;
  int64_t* first = nullptr;  // whole steps: first tile of each problem
  double* halo = nullptr;    // whole steps: the cells next to every tile's ends
};

struct isweno_batch_plan {
  int device = 0;
  int ncu = 256;
  int32_t nprob = 0;
  int64_t longest = 0;         // cells of the longest problem
  int64_t total = 0;
  int32_t bc_lo = 0, bc_hi = 0;
  int64_t* offsets = nullptr;  // device
  double* dx = nullptr;        // device
  double* ws = nullptr;        // U1, U2 (device, 2 x 5 x total; stage launches only)
  int32_t* active = nullptr;   // per problem, written at the start of each step
  int32_t* tune_status = nullptr;  // per problem, for the autotuner's scratch runs
  std::map<int, TileTable> tables;  // by lanes per workgroup - 1
  int tl = 255;
  int blocks_per_cu = 4;
  hipStream_t cap = nullptr;   // capture stream
  // graph cache keyed by everything a captured step depends on
  using Key = std::tuple<const void*, const void*, const void*, const void*, int, int, int,
                         double, double, double, int, int>;
  std::map<Key, hipGraphExec_t> graphs;
  std::vector<int64_t> host_offsets;
};

static void free_graphs(isweno_batch_plan* p) {
  for (auto& kv : p->graphs) (void)hipGraphExecDestroy(kv.second);
  p->graphs.clear();
}

// Whole steps in one launch: every plan but those with a periodic end.  In
// FP64 at the default lanes 20 tubes of 50 to 150 cells take 45 us a step where
// one launch per stage took 46, 60 of 100 to 600 49 and 51, 1000 of 20 to 80 61
// and 62, 300 of 50 to 1500 85 and 100, 4096 of 128 to 4096 1024 and 1790
// (float 31 and 33, 33 and 36, 38 and 40, 48 and 59, 559 and 1090).
static bool whole_steps(const isweno_batch_plan* p) {
  return p->bc_lo != ISWENO_BC_PERIODIC && p->bc_hi != ISWENO_BC_PERIODIC;
}

static void free_table(TileTable& t) {
  (void)hipFree(t.start);
  (void)hipFree(t.prob);
  (void)hipFree(t.first);
  (void)hipFree(t.halo);
  t = TileTable{};
}

// The tile list for a workgroup of tl + 1 lanes: tiles of tl cells per stage
// launch, or of step_tile(tl + 1) cells for whole steps.
static int build_table(isweno_batch_plan* p, int key) {
  if (p->tables.count(key)) return ISWENO_OK;
  const bool whole = whole_steps(p);
  const int tl = whole ? isw::step_tile(key + 1) : key;
  std::vector<int64_t> st, first;
  std::vector<int32_t> pr;
  for (int32_t q = 0; q < p->nprob; q++) {
    first.push_back((int64_t)st.size());
    for (int64_t c = p->host_offsets[q]; c < p->host_offsets[q + 1]; c += tl) {
      st.push_back(c);
      pr.push_back(q);
    }
  }
  TileTable t;
  t.ntiles = (int64_t)st.size();
  auto put = [](auto** d, const auto& v) {
    const size_t bytes = v.size() * sizeof(v[0]);
    return hipMalloc(d, bytes) == hipSuccess &&
           hipMemcpy(*d, v.data(), bytes, hipMemcpyHostToDevice) == hipSuccess;
  };
  bool ok = put(&t.start, st) && put(&t.prob, pr);
  if (ok && whole)
    ok = put(&t.first, first) &&
         hipMalloc(&t.halo, sizeof(double) * 5 * 2 * isw::kHalo * st.size()) == hipSuccess;
  if (!ok) {
    free_table(t);
    return ISWENO_ERR_DEVICE;
  }
  p->tables[key] = t;
  return ISWENO_OK;
}

static int check_batch_opts(const isweno_opts* o) {
  if (!o || o->reserved != 0 || o->reserved2 != 0) return ISWENO_ERR_ARG;
  if (o->precision != ISWENO_FP64 && o->precision != ISWENO_FP32) return ISWENO_ERR_ARG;
  if (o->weights < 0 || o->weights > 3 || o->mood < 0 || o->mood > 2) return ISWENO_ERR_ARG;
  if (!(o->eps >= 0.0)) return ISWENO_ERR_ARG;
  if (o->weights == ISWENO_W_MLP) return ISWENO_ERR_UNSUPPORTED;
  return ISWENO_OK;
}

// Enqueue one RK3 step on s: the start-of-step kernel, then the step kernel, or
// three persistent stages with a periodic end.
static hipError_t enqueue_step(isweno_batch_plan* p, const isweno_opts* o, double* U, double* dt,
                               isweno_stats* stats, int32_t* pstatus, int tl, int bpc,
                               hipStream_t s) {
  const TileTable& t = p->tables[tl];
  const int tc = isw::step_tile(tl + 1);
  // Whole steps: the copies next to tile ends in a kernel of their own where
  // there is no time step to form or a problem is long (kLongWalk)
  const bool edges = whole_steps(p) && (!(o->cfl > 0.0) || p->longest > kLongWalk);
  hipError_t e;
  if (!edges || o->cfl > 0.0) {
    hipLaunchKernelGGL(isw::batch_dt_kernel, dim3(p->nprob), dim3(256), 0, s, U, p->total,
                       p->offsets, p->dx, o->cfl, o->dt_max, dt, pstatus, p->active, tc, t.first,
                       edges ? nullptr : t.halo);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  if (edges) {
    const int64_t groups = 256 / isw::kEdgeLanes;
    hipLaunchKernelGGL(isw::batch_edges_kernel, dim3((unsigned)((t.ntiles + groups - 1) / groups)),
                       dim3(256), 0, s, U, p->total, p->offsets, t.start, t.prob, t.ntiles, pstatus,
                       p->active, tc, t.halo);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  isw::BatchArgs a{};
  a.active = p->active;
  a.pstatus = pstatus;
  a.dt = dt;
  a.dx = p->dx;
  a.offsets = p->offsets;
  a.tstart = t.start;
  a.tprob = t.prob;
  a.ntiles = t.ntiles;
  a.total = p->total;
  a.stats = reinterpret_cast<isw::StatsDev*>(stats);
  a.bc_lo = p->bc_lo;
  a.bc_hi = p->bc_hi;
  a.weights = o->weights;
  a.mood = o->mood;
  a.eps = o->eps;
  if (whole_steps(p)) {
    a.U = U;
    a.halo = t.halo;
    return isw::launch_batch_step(o->precision, tl + 1, a, s);
  }
  a.U0 = U;
  int64_t blocks64 = (int64_t)p->ncu * bpc;
  if (blocks64 > t.ntiles) blocks64 = t.ntiles;
  if (blocks64 < 1) blocks64 = 1;
  const int blocks = (int)blocks64;
  double* U1 = p->ws;
  double* U2 = p->ws + 5 * p->total;
  a.Uin = U;
  a.Uout = U1;
  if ((e = isw::launch_batch_stage(o->precision, tl, a, isw::OUT_RK1, blocks, s)) != hipSuccess)
    return e;
  a.Uin = U1;
  a.Uout = U2;
  if ((e = isw::launch_batch_stage(o->precision, tl, a, isw::OUT_RK2, blocks, s)) != hipSuccess)
    return e;
  a.Uin = U2;
  a.Uout = U;
  return isw::launch_batch_stage(o->precision, tl, a, isw::OUT_RK3, blocks, s);
}

extern "C" {

int isweno_batch_plan_create(isweno_ctx* ctx, int32_t nprob, const int64_t* offsets,
                             const double* dx, int32_t bc_lo, int32_t bc_hi,
                             isweno_batch_plan** out) {
  if (!out) return ISWENO_ERR_ARG;
  *out = nullptr;
  if (!ctx || nprob < 1 || !offsets || !dx) return ISWENO_ERR_ARG;
  if (bc_lo < 0 || bc_lo > 2 || bc_hi < 0 || bc_hi > 2) return ISWENO_ERR_ARG;
  if (offsets[0] != 0) return ISWENO_ERR_ARG;
  const int minlen = (bc_lo == ISWENO_BC_REFLECTIVE || bc_hi == ISWENO_BC_REFLECTIVE) ? 3 : 1;
  for (int32_t q = 0; q < nprob; q++) {
    if (offsets[q + 1] - offsets[q] < minlen || !(dx[q] > 0.0)) return ISWENO_ERR_ARG;
  }
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return ISWENO_ERR_DEVICE;
  isweno_batch_plan* p = new (std::nothrow) isweno_batch_plan();
  if (!p) return ISWENO_ERR_DEVICE;
  p->device = dev;
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
    p->ncu = prop.multiProcessorCount;
  p->nprob = nprob;
  p->total = offsets[nprob];
  p->bc_lo = bc_lo;
  p->bc_hi = bc_hi;
  p->host_offsets.assign(offsets, offsets + nprob + 1);
  for (int32_t q = 0; q < nprob; q++)
    p->longest = std::max(p->longest, offsets[q + 1] - offsets[q]);
  // The fewest lanes that hold every problem in one tile, else the most (1000
  // tubes of 20 to 80 cells: 128 lanes 61.3 us a step, 256 lanes 63.3,
  // float with periodic ends 41.5 and 42.8).  The autotuner tries all.
  for (int tl : kTiles)
    if (p->longest <= (whole_steps(p) ? isw::step_tile(tl + 1) : tl)) {
      p->tl = tl;
      break;
    }
  bool ok = hipMalloc(&p->offsets, sizeof(int64_t) * (nprob + 1)) == hipSuccess &&
            hipMalloc(&p->dx, sizeof(double) * nprob) == hipSuccess &&
            (whole_steps(p) ||
             hipMalloc(&p->ws, sizeof(double) * 10 * p->total) == hipSuccess) &&
            hipMalloc(&p->active, sizeof(int32_t) * nprob) == hipSuccess &&
            hipMalloc(&p->tune_status, sizeof(int32_t) * nprob) == hipSuccess &&
            hipMemcpy(p->offsets, offsets, sizeof(int64_t) * (nprob + 1),
                      hipMemcpyHostToDevice) == hipSuccess &&
            hipMemcpy(p->dx, dx, sizeof(double) * nprob, hipMemcpyHostToDevice) == hipSuccess &&
            hipStreamCreateWithFlags(&p->cap, hipStreamNonBlocking) == hipSuccess;
  if (ok) ok = build_table(p, p->tl) == ISWENO_OK;
  if (!ok) {
    isweno_batch_plan_destroy(p);
    return ISWENO_ERR_DEVICE;
  }
  *out = p;
  return ISWENO_OK;
}

void isweno_batch_plan_destroy(isweno_batch_plan* p) {
  if (!p) return;
  (void)hipSetDevice(p->device);
  (void)hipDeviceSynchronize();
  free_graphs(p);
  for (auto& kv : p->tables) free_table(kv.second);
  if (p->offsets) (void)hipFree(p->offsets);
  if (p->dx) (void)hipFree(p->dx);
  if (p->ws) (void)hipFree(p->ws);
  if (p->active) (void)hipFree(p->active);
  if (p->tune_status) (void)hipFree(p->tune_status);
  if (p->cap) (void)hipStreamDestroy(p->cap);
  delete p;
}

int isweno_batch_autotune(isweno_ctx* ctx, isweno_batch_plan* p, const isweno_opts* o,
                          const double* U, int32_t* chosen_tile, void* stream) {
  int r;
  if (!ctx || !p || !U) return ISWENO_ERR_ARG;
  if ((r = check_batch_opts(o)) != ISWENO_OK) return r;
  if (hipSetDevice(p->device) != hipSuccess) return ISWENO_ERR_DEVICE;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const size_t bytes = sizeof(double) * 5 * p->total;
  double* S = nullptr;
  double* dt = nullptr;
  if (hipMalloc(&S, bytes) != hipSuccess) return ISWENO_ERR_DEVICE;
  if (hipMalloc(&dt, sizeof(double) * p->nprob) != hipSuccess) {
    (void)hipFree(S);
    return ISWENO_ERR_DEVICE;
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  (void)hipEventCreate(&e0);
  (void)hipEventCreate(&e1);
  isweno_opts to = *o;
  if (!(to.cfl > 0.0)) to.cfl = 0.5;  // keep the scratch run physical
  float best = 1e30f;
  int best_tl = p->tl, best_bpc = p->blocks_per_cu;
  r = ISWENO_OK;
  for (int tl : kTiles) {
    if ((r = build_table(p, tl)) != ISWENO_OK) break;
    for (int bpc : kBlocksPerCU) {
      if (whole_steps(p) && bpc != kBlocksPerCU[0]) continue;  // one workgroup per tile
      float ms_min = 1e30f;
      for (int rep = 0; rep < 3 && r == ISWENO_OK; rep++) {
        if (hipMemcpyAsync(S, U, bytes, hipMemcpyDeviceToDevice, s) != hipSuccess ||
            hipMemsetAsync(p->tune_status, 0, sizeof(int32_t) * p->nprob, s) != hipSuccess ||
            hipEventRecord(e0, s) != hipSuccess ||
            enqueue_step(p, &to, S, dt, nullptr, p->tune_status, tl, bpc, s) != hipSuccess ||
            hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess) {
          r = ISWENO_ERR_DEVICE;
          break;
        }
        float ms = 0.f;
        (void)hipEventElapsedTime(&ms, e0, e1);
        ms_min = std::min(ms_min, ms);
      }
      if (r != ISWENO_OK) break;
      if (ms_min < best) {
        best = ms_min;
        best_tl = tl;
        best_bpc = bpc;
      }
    }
    if (r != ISWENO_OK) break;
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  (void)hipFree(S);
  (void)hipFree(dt);
  if (r != ISWENO_OK) return r;
  if (best_tl != p->tl || best_bpc != p->blocks_per_cu) free_graphs(p);
  p->tl = best_tl;
  p->blocks_per_cu = best_bpc;
  if (chosen_tile) *chosen_tile = best_tl;
  return ISWENO_OK;
}

// Not part of the ABI (isweno.h does not declare it): the tests compare every
// lane count with the oracle, which the autotuner's timing would leave to chance.
ISWENO_API int isweno_test_batch_lanes(isweno_batch_plan* p, int32_t lanes) {
  if (!p || std::find(std::begin(kTiles), std::end(kTiles), lanes - 1) == std::end(kTiles))
    return ISWENO_ERR_ARG;
  if (hipSetDevice(p->device) != hipSuccess || hipDeviceSynchronize() != hipSuccess)
    return ISWENO_ERR_DEVICE;
  free_graphs(p);
  const int r = build_table(p, lanes - 1);
  if (r == ISWENO_OK) p->tl = lanes - 1;
  return r;
}

int isweno_batch_step(isweno_ctx* ctx, isweno_batch_plan* p, const isweno_opts* o, double* U,
                      double* dt, int32_t nsteps, isweno_stats* stats, int32_t* status,
                      void* stream) {
  int r;
  if (!ctx || !p || !U || !dt || !status || nsteps < 0) return ISWENO_ERR_ARG;
  if ((r = check_batch_opts(o)) != ISWENO_OK) return r;
  if (nsteps == 0) return ISWENO_OK;
  if (hipSetDevice(p->device) != hipSuccess) return ISWENO_ERR_DEVICE;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  isweno_batch_plan::Key key{U, dt, stats, status, o->precision, o->weights, o->mood, o->eps,
                             o->cfl, o->dt_max, p->tl, p->blocks_per_cu};
  auto it = p->graphs.find(key);
  hipGraphExec_t exec = nullptr;
  if (it == p->graphs.end()) {
    // capture one step on the plan's own stream (the caller's may be the
    // legacy default stream, which cannot be captured)
    hipGraph_t graph = nullptr;
    if (hipStreamBeginCapture(p->cap, hipStreamCaptureModeThreadLocal) != hipSuccess)
      return ISWENO_ERR_DEVICE;
    const hipError_t e =
        enqueue_step(p, o, U, dt, stats, status, p->tl, p->blocks_per_cu, p->cap);
    const hipError_t e2 = hipStreamEndCapture(p->cap, &graph);
    if (e != hipSuccess || e2 != hipSuccess || !graph) {
      if (graph) (void)hipGraphDestroy(graph);
      return ISWENO_ERR_DEVICE;
    }
    const hipError_t e3 = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e3 != hipSuccess) return ISWENO_ERR_DEVICE;
    p->graphs[key] = exec;
  } else {
    exec = it->second;
  }
  for (int32_t k = 0; k < nsteps; k++) {
    if (hipGraphLaunch(exec, s) != hipSuccess) return ISWENO_ERR_DEVICE;
  }
  return ISWENO_OK;
}

}  // extern "C"
