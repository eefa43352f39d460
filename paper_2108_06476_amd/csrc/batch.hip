// batch.hip -- ensembles of independent solvers (dgx_batch_*): runs of different grid
// sizes and polynomial degrees advanced together.  An RK stage of the runs in element tiles is
// one launch over (run, element tile) work items: one block per item, or a persistent grid whose
// blocks loop over the items; runs with a line of nodes per thread are a launch per polynomial
// degree.  Steps (per-run time step + 5 stages) are replayed from a captured hipGraph, in which
// each of these groups is a branch.  The tile shape (block size) and the grid are chosen by timing the
// candidates on the batch (dgx_batch_tune) or set by hand (dgx_batch_set_shape).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <string>
#include <vector>

#include "../../include/dgx.h"
#include "batch_kernels.h"
#include "tables.h"

using namespace dgx;

namespace {

const double CK_A[5] = {0.0, -567301805773.0 / 1357537059087.0, -2404267990393.0 / 2016746695238.0,
                        -3550918686646.0 / 2091501179385.0, -1275806237668.0 / 842570457699.0};
const double CK_B[5] = {1432997174477.0 / 9575080441755.0, 5161836677717.0 / 13612068292357.0,
                        1720146321549.0 / 2090206949498.0, 3134564353537.0 / 4481467310338.0,
                        2277821191437.0 / 14882151754819.0};

}  // namespace

struct dgx_batch_s {
  int nruns = 0;
  int prec = 0;
  hipStream_t stream = nullptr;
  std::vector<dgx_config> cfgs;
  std::vector<int64_t> nodes;     // per run, per variable
  std::vector<void*> allocs;
  std::vector<RunDesc> desc;      // host copy
  RunDesc* desc_d = nullptr;
  int* flag_d = nullptr;
  // Groups of runs that a kernel takes in one launch (device lists order_d and prefix_d): every
  // run (the wave speeds), the runs in tiles of the current shape, and, of each polydeg, the
  // runs with a line of nodes per thread.
  enum { ALL = 0, TILED = 1, PENCIL = 2, GROUPS = PENCIL + BATCH_NMAX - BATCH_NMIN + 1 };
  int* order_d[GROUPS] = {};
  int* prefix_d[GROUPS] = {};
  std::vector<int> order[GROUPS];
  BatchLaunch bl[GROUPS] = {};
  int budget = 256;
  int grid = 0;       // blocks of the TILED launch
  int cus = 0;
  std::vector<int> groups;   // the groups that hold runs, in the order of their branches
  // recording of the steps' graphs: the main branch and one for each group after the first
  hipStream_t cap = nullptr;
  hipStream_t side[GROUPS] = {};
  hipEvent_t fork = nullptr, joined[GROUPS] = {};
  // [0]: the last step of an odd count, [1]: two steps; each for the cfl it was recorded with
  struct Steps {
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    double cfl = -1.0;
  } steps[2];
  double odd_cfl = -1.0;   // the last odd count's
  std::string err;
};

namespace {

dgx_status bfail(dgx_batch b, dgx_status st, const std::string& m) {
  if (b) b->err = m;
  return st;
}

#define BHIP(b, expr)                                                                 \
  do {                                                                                \
    hipError_t e_ = (expr);                                                           \
    if (e_ != hipSuccess)                                                             \
      return bfail(b, DGX_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_));   \
  } while (0)

bool dev_alloc(dgx_batch b, void** p, size_t bytes) {
  if (hipMalloc(p, bytes) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  b->allocs.push_back(*p);
  return true;
}

// array argument: inside one device allocation of at least `bytes`
bool dev_ok(const void* p, size_t bytes) {
  if (!p) return false;
  hipPointerAttribute_t at;
  if (hipPointerGetAttributes(&at, p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  if (at.type != hipMemoryTypeDevice && at.type != hipMemoryTypeManaged) return false;
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  if (hipMemGetAddressRange(&base, &size, (hipDeviceptr_t)p) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return (const char*)p + bytes <= (const char*)base + size;
}

void drop_graph(dgx_batch b) {
  for (dgx_batch_s::Steps& g : b->steps) {
    if (g.exec) (void)hipGraphExecDestroy(g.exec);
    if (g.graph) (void)hipGraphDestroy(g.graph);
    g = dgx_batch_s::Steps();
  }
}

// The device lists of a group: its runs' tile counts for `elems(N)` elements per tile.
template <typename Elems>
dgx_status upload_group(dgx_batch b, int gi, Elems elems) {
  const std::vector<int>& order = b->order[gi];
  const int nr = (int)order.size();
  std::vector<int> prefix(nr + 1, 0);
  for (int i = 0; i < nr; ++i) {
    const int r = order[i], ne = elems(b->desc[r].N);
    prefix[i + 1] = prefix[i] + (b->desc[r].E + ne - 1) / ne;
  }
  if (nr > 0)
    BHIP(b, hipMemcpy(b->order_d[gi], order.data(), sizeof(int) * nr, hipMemcpyHostToDevice));
  BHIP(b, hipMemcpy(b->prefix_d[gi], prefix.data(), sizeof(int) * (nr + 1), hipMemcpyHostToDevice));
  b->bl[gi].runs = b->desc_d;
  b->bl[gi].order = b->order_d[gi];
  b->bl[gi].prefix = b->prefix_d[gi];
  b->bl[gi].nruns = nr;
  b->bl[gi].total = prefix[nr];
  return DGX_OK;
}

int round8(int n) { return ((n + 7) / 8) * 8; }   // blocks: a multiple of the 8 XCDs

// work items of the current block size: runs heaviest (highest polydeg) first
dgx_status set_shape(dgx_batch b, int budget, int grid) {
  BHIP(b, hipStreamSynchronize(b->stream));
  for (int gi : {(int)dgx_batch_s::ALL, (int)dgx_batch_s::TILED}) {
    dgx_status st = upload_group(b, gi, [&](int N) { return batch_tile_elems(N, budget); });
    if (st != DGX_OK) return st;
  }
  b->budget = budget;
  // grid 0 or >= the items: one block per item
  const int total = b->bl[dgx_batch_s::TILED].total;
  b->grid = (grid <= 0 || grid >= total) ? round8(total) : grid;
  drop_graph(b);
  return DGX_OK;
}

// One RK stage (or right-hand side) of a group's runs.
dgx_status enqueue_group(dgx_batch b, hipStream_t st, int gi, int epi, int cur, double A, double B,
                         int emit, int kw) {
  const BatchLaunch& l = b->bl[gi];
  if (l.total == 0) return DGX_OK;
  if (gi == dgx_batch_s::TILED)
    BHIP(b, batch_stage(st, l, b->budget, b->grid, b->prec, epi, cur, A, B, emit, kw));
  else
    BHIP(b, batch_pencil_stage(st, l, gi - dgx_batch_s::PENCIL + BATCH_NMIN, epi, cur, A, B, emit, kw));
  return DGX_OK;
}

dgx_status upload_desc(dgx_batch b) {
  // work already enqueued may still read the descriptors
  BHIP(b, hipStreamSynchronize(b->stream));
  BHIP(b, hipMemcpy(b->desc_d, b->desc.data(), sizeof(RunDesc) * b->nruns, hipMemcpyHostToDevice));
  return DGX_OK;
}

// Point the descriptors at the caller's arrays; re-upload only when something changed.
dgx_status bind(dgx_batch b, double* const* u, double* const* du, double* t) {
  bool changed = false;
  for (int r = 0; r < b->nruns; ++r) {
    const size_t bytes = sizeof(double) * 5 * (size_t)b->nodes[r];
    if (u && !dev_ok(u[r], bytes))
      return bfail(b, DGX_EINVAL, "u[" + std::to_string(r) + "]: not a device array of the run's size");
    if (du && !dev_ok(du[r], bytes))
      return bfail(b, DGX_EINVAL, "du[" + std::to_string(r) + "]: not a device array of the run's size");
    RunDesc& d = b->desc[r];
    double* nu = u ? u[r] : d.u;
    double* ndu = du ? du[r] : d.du;
    double* nt = t ? t + r : nullptr;
    changed |= (nu != d.u) || (ndu != d.du) || (nt != d.t);
    d.u = nu;
    d.du = ndu;
    d.t = nt;
  }
  if (t && !dev_ok(t, sizeof(double) * b->nruns)) return bfail(b, DGX_EINVAL, "t: not a device array of nruns");
  if (changed) return upload_desc(b);
  return DGX_OK;
}

// Streams and events of the graphs' branches.
dgx_status ensure_branches(dgx_batch b) {
  if (!b->fork) BHIP(b, hipEventCreateWithFlags(&b->fork, hipEventDisableTiming));
  for (size_t i = 1; i < b->groups.size(); ++i) {
    const int gi = b->groups[i];
    if (!b->side[gi]) BHIP(b, hipStreamCreateWithFlags(&b->side[gi], hipStreamNonBlocking));
    if (!b->joined[gi]) BHIP(b, hipEventCreateWithFlags(&b->joined[gi], hipEventDisableTiming));
  }
  return DGX_OK;
}

// work(group, stream) for every group in turn on st, or (branch: st records a graph) the first on st
// and each other one on a branch that leaves st here and comes back to it (the groups share no run).
// Branches fill each other's last rounds of blocks, where launches in turn leave compute units idle
// at the end of each.
template <typename Work>
dgx_status branch_groups(dgx_batch b, hipStream_t st, bool branch, Work work) {
  const size_t ng = b->groups.size();
  branch = branch && ng > 1;
  if (branch) BHIP(b, hipEventRecord(b->fork, st));
  dgx_status r = DGX_OK;
  for (size_t i = 0; i < ng; ++i) {
    const int gi = b->groups[i];
    hipStream_t sg = branch && i > 0 ? b->side[gi] : st;
    if (sg != st) BHIP(b, hipStreamWaitEvent(sg, b->fork, 0));
    if (r == DGX_OK) r = work(gi, sg);
    if (sg != st) BHIP(b, hipEventRecord(b->joined[gi], sg));   // (also after a failed launch)
  }
  for (size_t i = 1; branch && i < ng; ++i)
    BHIP(b, hipStreamWaitEvent(st, b->joined[b->groups[i]], 0));
  return r;
}

// The time steps and the five stages of a step, a branch per group (in a graph) or the groups in turn.
dgx_status enqueue_step(dgx_batch b, hipStream_t st, double cfl, int cur, bool emit, bool branch) {
  BHIP(b, batch_dt(st, b->desc_d, b->nruns, cfl));
  return branch_groups(b, st, branch, [&](int gi, hipStream_t sg) {
    for (int s = 0, c = cur; s < 5; ++s, c = 1 - c) {
      dgx_status r = enqueue_group(b, sg, gi, EPI_RK, c, CK_A[s], CK_B[s], (emit && s == 4) ? 1 : 0, s < 4);
      if (r != DGX_OK) return r;
    }
    return DGX_OK;
  });
}

// The graph of one step, or of two: the state returns to the caller's buffer (10 stages), and the
// second step's last stage emits the wave speeds of the next, so that it can be replayed.
dgx_status ensure_graph(dgx_batch b, int nsteps, double cfl) {
  dgx_batch_s::Steps& g = b->steps[nsteps - 1];
  if (g.exec && g.cfl == cfl) return DGX_OK;
  if (g.exec) (void)hipGraphExecDestroy(g.exec);
  if (g.graph) (void)hipGraphDestroy(g.graph);
  g = dgx_batch_s::Steps();
  if (!b->cap) BHIP(b, hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking));
  dgx_status st = ensure_branches(b);
  if (st != DGX_OK) return st;
  BHIP(b, hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal));
  st = enqueue_step(b, b->cap, cfl, 0, nsteps == 2, true);
  if (st == DGX_OK && nsteps == 2) st = enqueue_step(b, b->cap, cfl, 1, true, true);
  hipGraph_t graph = nullptr;
  hipError_t e = hipStreamEndCapture(b->cap, &graph);
  if (st != DGX_OK || e != hipSuccess) {
    if (graph) (void)hipGraphDestroy(graph);
    return st != DGX_OK ? st : bfail(b, DGX_EHIP, std::string("hipStreamEndCapture: ") + hipGetErrorString(e));
  }
  g.graph = graph;
  BHIP(b, hipGraphInstantiate(&g.exec, graph, nullptr, nullptr, 0));
  g.cfl = cfl;
  return DGX_OK;
}

// The last step of an odd count.  Replayed from a graph, whose branches overlap the groups (five runs
// of 8^3 to 24^3, two in lines: a call of one step 1 322 us, 1 421 with the groups in turn, 1 526 with
// every run in k_batch_stage).  In turn where that is not worth a recording or not possible: one
// group, the first such call with a cfl, a stream that the caller is recording.  (Branches beside the
// caller's stream without a graph are no faster than in turn when their streams share a hardware
// queue with it.)
dgx_status odd_step(dgx_batch b, double cfl) {
  const bool again = b->odd_cfl == cfl;
  b->odd_cfl = cfl;
  hipStreamCaptureStatus rec = hipStreamCaptureStatusNone;
  if (b->groups.size() > 1 && again) BHIP(b, hipStreamIsCapturing(b->stream, &rec));
  if (b->groups.size() < 2 || !again || rec != hipStreamCaptureStatusNone)
    return enqueue_step(b, b->stream, cfl, 0, false, false);
  dgx_status st = ensure_graph(b, 1, cfl);
  if (st == DGX_OK) BHIP(b, hipGraphLaunch(b->steps[0].exec, b->stream));
  return st;
}

}  // namespace

extern "C" {

dgx_status dgx_batch_create(const dgx_config* cfgs, int32_t nruns, void* hip_stream,
                            dgx_batch* out) {
  if (!cfgs || !out || nruns < 1) return DGX_EINVAL;
  *out = nullptr;
  for (int r = 0; r < nruns; ++r) {
    const dgx_config& c = cfgs[r];
    if (c.dim != 3 || c.volume != DGX_VOL_EC ||
        (c.surface != DGX_SURF_LLF && c.surface != DGX_SURF_HLL) || !(c.gamma > 1.0) ||
        (c.precision != DGX_FP64 && c.precision != DGX_MIXED) || c.precision != cfgs[0].precision)
      return DGX_EINVAL;
    for (int d = 0; d < 3; ++d)
      if (c.cells[d] < 1 || !(c.xmax[d] > c.xmin[d])) return DGX_EINVAL;
    if (c.polydeg < BATCH_NMIN || c.polydeg > BATCH_NMAX) return DGX_EUNSUPPORTED;
    const int n = c.polydeg + 1;
    if ((int64_t)5 * c.cells[0] * c.cells[1] * c.cells[2] * n * n * n >= ((int64_t)1 << 31))
      return DGX_EUNSUPPORTED;
  }
  dgx_batch b = new dgx_batch_s();
  b->nruns = nruns;
  b->prec = cfgs[0].precision;
  b->stream = (hipStream_t)hip_stream;
  b->cfgs.assign(cfgs, cfgs + nruns);
  b->desc.resize(nruns);
  int dev = 0;
  (void)hipGetDevice(&dev);
  if (hipDeviceGetAttribute(&b->cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      b->cus < 1)
    b->cus = 256;
  bool ok = dev_alloc(b, (void**)&b->desc_d, sizeof(RunDesc) * nruns) &&
            dev_alloc(b, (void**)&b->flag_d, sizeof(int) * 2);
  for (int gi = 0; ok && gi < dgx_batch_s::GROUPS; ++gi)
    ok = dev_alloc(b, (void**)&b->order_d[gi], sizeof(int) * nruns) &&
         dev_alloc(b, (void**)&b->prefix_d[gi], sizeof(int) * (nruns + 1));
  for (int r = 0; ok && r < nruns; ++r) {
    const dgx_config& c = cfgs[r];
    const int n = c.polydeg + 1;
    RunDesc& d = b->desc[r];
    d.E = c.cells[0] * c.cells[1] * c.cells[2];
    d.K[0] = c.cells[0];
    d.K[1] = c.cells[1];
    d.K[2] = c.cells[2];
    d.N = c.polydeg;
    d.surf = c.surface;
    d.gamma = c.gamma;
    d.inv_gm1 = 1.0 / (c.gamma - 1.0);
    d.flag = b->flag_d;
    d.u = d.du = d.t = nullptr;
    b->nodes.push_back((int64_t)d.E * n * n * n);
    const size_t sb = sizeof(double) * 5 * (size_t)b->nodes[r];
    double h[3];
    for (int k = 0; k < 3; ++k) h[k] = (c.xmax[k] - c.xmin[k]) / c.cells[k];
    std::vector<double> T(TAB_SIZE, 0.0);
    ok = stage_tables(c.polydeg, h, T.data()) && dev_alloc(b, (void**)&d.u2, sb) &&
         dev_alloc(b, (void**)&d.k, sb) && dev_alloc(b, (void**)&d.speed, sizeof(double) * d.E) &&
         dev_alloc(b, (void**)&d.dt, sizeof(double)) &&
         dev_alloc(b, (void**)&d.tab, sizeof(double) * TAB_SIZE) &&
         hipMemcpy((void*)d.tab, T.data(), sizeof(double) * TAB_SIZE, hipMemcpyHostToDevice) == hipSuccess &&
         hipMemset(d.k, 0, sb) == hipSuccess;
  }
  if (!ok || hipMemset(b->flag_d, 0, sizeof(int) * 2) != hipSuccess) {
    dgx_batch_destroy(b);
    return DGX_ENOMEM;
  }
  size_t state = 0;
  for (int64_t m : b->nodes) state += sizeof(double) * 5 * (size_t)m;
  for (RunDesc& d : b->desc) d.nt_out = stream_output(state, 0);
  std::vector<int>& all = b->order[dgx_batch_s::ALL];
  all.resize(nruns);
  for (int r = 0; r < nruns; ++r) all[r] = r;
  std::stable_sort(all.begin(), all.end(),
                   [&](int x, int y) { return b->desc[x].N > b->desc[y].N; });
  for (int r : all) {   // the kernel of a run is that of dgx_step on it (the same results)
    const RunDesc& d = b->desc[r];
    const bool pencil = b->prec == DGX_FP64 && batch_pencil_run(d.N, d.E, d.surf);
    b->order[pencil ? dgx_batch_s::PENCIL + d.N - BATCH_NMIN : (int)dgx_batch_s::TILED].push_back(r);
  }
  bool up = upload_desc(b) == DGX_OK && set_shape(b, 256, 0) == DGX_OK;
  for (int gi = dgx_batch_s::PENCIL; up && gi < dgx_batch_s::GROUPS; ++gi)
    up = upload_group(b, gi, [](int N) { return batch_pencil_elems(N); }) == DGX_OK;
  // The groups in the order of their branches.  A graph's branches are submitted one after the other,
  // so where one group holds nearly all the work (pair fluxes) it comes first: two steps of N = 3 28^3
  // with 8^3 558 us, 580 in the other order; N = 4 24^3 with 3 8^3 787 / 818.  Else the tiles do (seven
  // runs 2 313 us, 2 355 with the most work first; five runs 2 385 / 2 425).
  double work[dgx_batch_s::GROUPS] = {}, total = 0.0;
  for (int gi = dgx_batch_s::TILED; gi < dgx_batch_s::GROUPS; ++gi) {
    for (int r : b->order[gi]) work[gi] += (double)b->nodes[r] * b->desc[r].N;
    if (!b->order[gi].empty()) b->groups.push_back(gi);
    total += work[gi];
  }
  const auto most = std::max_element(b->groups.begin(), b->groups.end(),
                                     [&](int x, int y) { return work[x] < work[y]; });
  if (total < 1.1 * work[*most]) std::rotate(b->groups.begin(), most, most + 1);
  if (!up) {
    dgx_batch_destroy(b);
    return DGX_EHIP;
  }
  *out = b;
  return DGX_OK;
}

dgx_status dgx_batch_destroy(dgx_batch b) {
  if (!b) return DGX_EINVAL;
  (void)hipDeviceSynchronize();
  drop_graph(b);
  if (b->cap) (void)hipStreamDestroy(b->cap);
  if (b->fork) (void)hipEventDestroy(b->fork);
  for (int gi = 0; gi < dgx_batch_s::GROUPS; ++gi) {
    if (b->side[gi]) (void)hipStreamDestroy(b->side[gi]);
    if (b->joined[gi]) (void)hipEventDestroy(b->joined[gi]);
  }
  for (void* p : b->allocs) (void)hipFree(p);
  delete b;
  return DGX_OK;
}

int64_t dgx_batch_num_nodes(dgx_batch b, int32_t r) {
  if (!b || r < 0 || r >= b->nruns) return -1;
  return b->nodes[r];
}

dgx_status dgx_batch_step(dgx_batch b, double* const* u, int32_t nsteps, double cfl, double* t) {
  if (!b || !u) return DGX_EINVAL;
  if (!(cfl > 0.0)) return bfail(b, DGX_EINVAL, "cfl must be > 0");
  if (nsteps < 0) return bfail(b, DGX_EINVAL, "nsteps < 0");
  dgx_status st = bind(b, u, nullptr, t);
  if (st != DGX_OK) return st;
  if (nsteps == 0) return DGX_OK;
  const BatchLaunch& all = b->bl[dgx_batch_s::ALL];
  BHIP(b, batch_maxspeed(b->stream, all, b->budget, round8(all.total)));
  int pairs = nsteps / 2;
  if (pairs > 0) {
    st = ensure_graph(b, 2, cfl);
    if (st != DGX_OK) return st;
    for (int p = 0; p < pairs; ++p) BHIP(b, hipGraphLaunch(b->steps[1].exec, b->stream));
  }
  if (nsteps % 2) {
    st = odd_step(b, cfl);
    if (st != DGX_OK) return st;
    int64_t mx = 0;
    for (int64_t v : b->nodes) mx = std::max(mx, 5 * v);
    BHIP(b, batch_copy(b->stream, b->desc_d, b->nruns, mx));
  }
  return DGX_OK;
}

dgx_status dgx_batch_rhs(dgx_batch b, const double* const* u, double* const* du) {
  if (!b || !u || !du) return DGX_EINVAL;
  for (int r = 0; r < b->nruns; ++r) {
    const size_t bytes = sizeof(double) * 5 * (size_t)b->nodes[r];
    const char *pu = (const char*)u[r], *pd = (const char*)du[r];
    if (pu < pd + bytes && pd < pu + bytes)
      return bfail(b, DGX_EINVAL, "u[" + std::to_string(r) + "] and du[" + std::to_string(r) + "] overlap");
  }
  dgx_status st = bind(b, const_cast<double* const*>(u), du, nullptr);
  if (st != DGX_OK) return st;
  // in turn: a right-hand side is too short for the waits of a fork and join (28^3 and 8^3, N = 3:
  // 46 us, 54 on branches)
  return branch_groups(b, b->stream, false, [&](int gi, hipStream_t sg) {
    return enqueue_group(b, sg, gi, EPI_RHS, 0, 0.0, 0.0, 0, 0);
  });
}

dgx_status dgx_batch_tune(dgx_batch b, double* const* u, int32_t budget_ms) {
  if (!b || !u) return DGX_EINVAL;
  // times one right-hand side of the runs in element tiles (written into the RK registers, which
  // hold no state between steps) for each candidate tile shape and persistent grid; the runs with
  // a line of nodes per thread do not depend on them
  std::vector<double*> kbuf(b->nruns);
  for (int r = 0; r < b->nruns; ++r) kbuf[r] = b->desc[r].k;
  dgx_status st = bind(b, u, kbuf.data(), nullptr);
  if (st != DGX_OK) return st;
  auto unbind = [&]() {
    for (int r = 0; r < b->nruns; ++r) b->desc[r].du = nullptr;
    return upload_desc(b);
  };
  if (b->order[dgx_batch_s::TILED].empty()) return unbind();
  hipEvent_t e0, e1;
  BHIP(b, hipEventCreate(&e0));
  BHIP(b, hipEventCreate(&e1));
  const int budgets[2] = {256, 512};
  const int mult[4] = {0, 2, 4, 8};   // 0: one block per work item; else persistent blocks per CU
  double best = 1e300, used = 0.0;
  int bb = b->budget, bg = b->grid;
  for (int budget : budgets) {
    for (int m : mult) {   // (persistent candidates beyond the item count are skipped)
      if (used > budget_ms) break;
      st = set_shape(b, budget, m ? ((b->cus * m + 7) / 8) * 8 : 0);
      if (st != DGX_OK) break;
      float ms = 0.f, total = 0.f;
      bool fail = false;
      for (int rep = 0; rep < 4 && !fail; ++rep) {
        fail |= hipEventRecord(e0, b->stream) != hipSuccess;
        fail |= enqueue_group(b, b->stream, dgx_batch_s::TILED, EPI_RHS, 0, 0.0, 0.0, 0, 0) != DGX_OK;
        fail |= hipEventRecord(e1, b->stream) != hipSuccess;
        fail |= hipEventSynchronize(e1) != hipSuccess;
        fail |= hipEventElapsedTime(&ms, e0, e1) != hipSuccess;
        if (rep > 0) total += ms;   // the first launch warms up
        used += ms;
      }
      if (fail) {
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
        return bfail(b, DGX_EHIP, "tuning launch failed");
      }
      if (total / 3 < best) {
        best = total / 3;
        bb = budget;
        bg = b->grid;
      }
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  st = unbind();
  if (st != DGX_OK) return st;
  return set_shape(b, bb, bg);
}

dgx_status dgx_batch_check(dgx_batch b, int32_t* flag) {
  if (!b || !flag) return DGX_EINVAL;
  BHIP(b, hipStreamSynchronize(b->stream));
  int f = 0;
  BHIP(b, hipMemcpy(&f, b->flag_d, sizeof(int), hipMemcpyDeviceToHost));
  BHIP(b, hipMemset(b->flag_d, 0, sizeof(int)));
  *flag = f;
  return f ? DGX_ENONPHYS : DGX_OK;
}

dgx_status dgx_batch_set_shape(dgx_batch b, int32_t block, int32_t grid) {
  if (!b) return DGX_EINVAL;
  if (block != 256 && block != 512) return bfail(b, DGX_EINVAL, "block must be 256 or 512");
  if (grid < 0 || grid % 8 != 0) return bfail(b, DGX_EINVAL, "grid must be 0 or a positive multiple of 8");
  return set_shape(b, block, grid);
}

dgx_status dgx_batch_shape(dgx_batch b, int32_t* block, int32_t* grid) {
  if (!b) return DGX_EINVAL;
  if (block) *block = b->budget;
  if (grid) *grid = b->grid;
  return DGX_OK;
}

const char* dgx_batch_last_error(dgx_batch b) { return b ? b->err.c_str() : "invalid batch"; }

}  // extern "C"
