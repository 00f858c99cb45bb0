// C ABI of the A-term IDG library: plan creation (host partition + device
// upload), batched gridding/degridding launches and error reporting.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "aidg_internal.h"

using namespace aidg;

namespace {

thread_local std::string g_last_error;

aidg_status fail(aidg_status st, const std::string& msg) {
  g_last_error = msg;
  return st;
}

aidg_status hip_fail(hipError_t e, const char* what) {
  return fail(AIDG_E_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

// One library stream per device on which plan memory is returned to the device's
// stream-ordered pool (null if it cannot be created: memory is then freed
// synchronously).  Default priority, non-blocking.
hipStream_t release_stream(int device) {
  static std::mutex mu;
  static std::map<int, hipStream_t> streams;
  std::lock_guard<std::mutex> lock(mu);
  auto it = streams.find(device);
  if (it != streams.end()) return it->second;
  int cur = 0;
  hipStream_t s = nullptr;
  if (hipGetDevice(&cur) == hipSuccess && (cur == device || hipSetDevice(device) == hipSuccess)) {
    if (hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) {
      (void)hipGetLastError();
      s = nullptr;
    }
    if (cur != device) (void)hipSetDevice(cur);
  }
  streams[device] = s;
  return s;
}

}  // namespace

// Byte offsets of a plan's tables in their one allocation: taper times (-1)^(x+y) [L][L] and
// twiddles [L] in the plan's precision, and in FP32 plans the matrix kernels' n1 and b along
// the axis [L] and taper and cross term [L][L].
struct TableLayout {
  size_t taper_cross, axis_n1, twiddle, taper, axis_b, bytes;
  TableLayout(int L, size_t elem) {
    const size_t n = (size_t)L * L, matrix = elem == 8 ? 1 : 0;
    taper_cross = 0;
    axis_n1 = taper_cross + matrix * 8 * n;
    twiddle = axis_n1 + matrix * 8 * L;
    taper = twiddle + elem * L;
    axis_b = taper + elem / 2 * n;
    bytes = axis_b + matrix * 8 * L;
  }
};

struct aidg_plan {
  Geometry g{};
  int n_st = 0, nbl = 0, nt = 0, nc = 0, n_int = 0, W = 1, max_nv = 1, device = 0;
  int64_t n_pervis = 0, n_direct = 0;  // subgrids the degridder takes in these forms
  std::vector<aidg_subgrid> table;
  std::vector<double> w0;
  int64_t n_excluded = 0;
  // Subgrids sharing w-layer and centre are consecutive and form a group;
  // group k holds subgrids [grp_begin[k], grp_begin[k+1]).  sg_group maps a
  // subgrid to its group.  Batches are runs of whole groups: [batch_begin[b],
  // batch_begin[b+1]) in subgrids, at most `batch` groups each.
  std::vector<int64_t> grp_begin, batch_begin;
  std::vector<int32_t> sg_group;
  // Gridding may take a group in parts [part_begin[p], part_begin[p + 1]) (sg_part: a
  // subgrid's; the groups themselves where no part is worth it), see split_groups.
  // cost_prefix: prefix sums of the gridder's cost over the table; max_group_cost.
  std::vector<int64_t> part_begin, cost_prefix;
  std::vector<int32_t> sg_part;
  int64_t max_group_cost = 0;
  double b_peak = 0;  // matrix kernels: largest factor of the cross term
  bool split = false;  // the plan's own calls grid by parts (all of them fit the workspace)
  int64_t batch = 1;
  size_t elem = 8, aterm_bytes = 0, device_bytes = 0, scratch_bytes = 0;
  SubgridDev* d_sg = nullptr;
  double* d_uvw = nullptr;
  double* d_fc = nullptr;
  void* d_aterms = nullptr;
  char* d_tables = nullptr;  // taper, twiddles and the matrix kernels' tables, see table_layout
  void* d_scratch = nullptr;
  int64_t* d_excl = nullptr;
  int64_t* d_grp = nullptr;
  KernelArgs* d_args = nullptr;  // device copy of args()
  // matrix kernels: all of the plan's subgrids qualify (degridding: and they are not so
  // sparse that the other forms take less time, and the geometry asks for none)
  MatrixForm matrix_grid = kMatrixNone, matrix_degrid = kMatrixNone;
  int32_t w_terms = 0;  // of the series, most in a subgrid
  int64_t n_split = 0;  // subgrids with kWSplit
  // image level (invert / predict): Stockham radices of N, twiddles exp(-2 pi i k / N)
  // and the reciprocal of the taper's axis at image resolution (FP64); absent when N
  // is not supported
  ImageRadices img_fr{};
  bool img_ok = false;
  void* d_img_tw = nullptr;
  double* d_img_itaper = nullptr;
  // inverse A-term mode: (A^-1)^H planes for the gridder, the distinct (A_p plane,
  // A_q plane) pairs of the table [n][2] with their visibility counts, the partial sums
  // [chunks][L^2] and the weighted-average normalisation map [L^2]
  void* d_ainvh = nullptr;
  int32_t* d_npairs = nullptr;
  double* d_ncount = nullptr;
  double* d_npartial = nullptr;
  double* d_nmap = nullptr;
  int64_t n_pairs = 0, pair_chunk = 1;
  int n_chunks = 1;
  double n_total = 0.0;
  hipEvent_t last = nullptr;
  std::atomic<bool> busy{false};
  // profiling: events around each kernel launch
  struct Timed {
    int kind;
    int64_t vp, nsg;
    hipEvent_t a, b;
  };
  bool profiling = false;
  std::vector<hipEvent_t> pool;
  size_t pool_next = 0;
  std::vector<Timed> timed;
  std::vector<int64_t> vp_prefix;  // prefix sums of n_vis * L^2 over the table

  KernelArgs args() const {
    KernelArgs a;
    a.sg = d_sg;
    a.uvw = d_uvw;
    a.fc = d_fc;
    a.aterms = d_aterms;
    a.ainvh = d_ainvh;
    const TableLayout tl(g.L, elem);
    a.taper = d_tables + tl.taper;
    a.twiddle = d_tables + tl.twiddle;
    a.axis_n1 = reinterpret_cast<const double*>(d_tables + tl.axis_n1);
    a.axis_b = reinterpret_cast<const uint32_t*>(d_tables + tl.axis_b);
    a.taper_cross = reinterpret_cast<const float2*>(d_tables + tl.taper_cross);
    a.w_series = 2.0 * M_PI * b_peak * b_peak;
    a.grp_begin = d_grp;
    a.part_begin = d_grp + (part_begin.size() == grp_begin.size() ? 0 : grp_begin.size());
    a.nt_total = nt;
    a.nc_total = nc;
    a.N = g.N;
    a.npol = g.npol;
    a.du = g.du;
    a.lstep = g.fov / g.L;
    return a;
  }

  // Device memory comes from the device's stream-ordered pool (hipMallocAsync on
  // the creation stream) where the device supports it.  It goes back on a library
  // stream after the plan's last recorded work, so destroying a plan never
  // synchronises the device: a serving loop retires plans while other jobs run.
  bool async_mem = false;

  void release() {
    void* ptrs[] = {d_sg,     d_uvw,       d_fc,    d_aterms,  d_tables,   d_scratch,
                    d_excl,   d_grp,       d_args,  d_img_tw,  d_img_itaper, d_ainvh, d_npairs,
                    d_ncount, d_npartial,  d_nmap};
    hipStream_t fs = async_mem ? release_stream(device) : nullptr;
    int cur = device;
    if (fs) {
      (void)hipGetDevice(&cur);
      if (cur != device) (void)hipSetDevice(device);
      if (last) (void)hipStreamWaitEvent(fs, last, 0);
    }
    for (void* p : ptrs) {
      if (!p) continue;
      if (!fs)
        (void)hipFree(p);
      else if (hipFreeAsync(p, fs) != hipSuccess)
        (void)hipGetLastError();
    }
    if (fs && cur != device) (void)hipSetDevice(cur);
    if (last) (void)hipEventDestroy(last);
    for (hipEvent_t e : pool) (void)hipEventDestroy(e);
    pool.clear();
    timed.clear();
    d_sg = nullptr;
    d_uvw = d_fc = nullptr;
    d_aterms = d_scratch = nullptr;
    d_tables = nullptr;
    d_excl = nullptr;
    d_grp = nullptr;
    d_args = nullptr;
    d_img_tw = nullptr;
    d_img_itaper = nullptr;
    d_ainvh = nullptr;
    d_npairs = nullptr;
    d_ncount = d_npartial = d_nmap = nullptr;
    last = nullptr;
  }
};

struct aidg_executor {
  void* d_scratch = nullptr;
  int64_t bytes = 0;
  int device = 0;
  hipEvent_t last = nullptr;
  std::atomic<bool> busy{false};
};

namespace {

struct BusyGuard {
  aidg_plan* p;
  bool ok;
  explicit BusyGuard(aidg_plan* q) : p(q) {
    bool expected = false;
    ok = p->busy.compare_exchange_strong(expected, true);
  }
  ~BusyGuard() {
    if (ok) p->busy.store(false);
  }
};

bool gpu_subgrid_size(int L) { return L == 32 || L == 64 || L == 96; }

// Record a timing event pair around a launch when the plan is profiling.
struct TimedLaunch {
  aidg_plan* p;
  hipStream_t st;
  hipEvent_t ea = nullptr, eb = nullptr;
  TimedLaunch(aidg_plan* plan, hipStream_t stream) : p(plan), st(stream) {
    if (p && p->profiling && p->pool_next + 2 <= p->pool.size()) {
      ea = p->pool[p->pool_next++];
      eb = p->pool[p->pool_next++];
      (void)hipEventRecord(ea, st);
    }
  }
  void done(KernelClass k, int64_t vp, int64_t nsg) {
    if (!ea) return;
    (void)hipEventRecord(eb, st);
    p->timed.push_back({(int)k, vp, nsg, ea, eb});
  }
};

// Gridder cost of a subgrid, in visibilities: the matrix gridder takes 32 at a time, and the
// Jones epilogue about as long as 20.
int64_t grid_cost(const aidg_subgrid& s) { return std::max(s.nt * s.nc, 32) + 20; }

// Gridder workgroups in flight over the chip, in units of a group's (L / 32 per group; 256
// compute units hold three at L = 32, two beyond).
int64_t groups_in_flight(int L) { return L <= 32 ? 768 : 512 / (L / 32); }

// Whether the heaviest group outlasts the launch's work spread evenly by enough: 2.5 times.
// By less gains nothing, as the last workgroups of a launch run faster, with a compute unit
// to themselves, and the sum of the parts takes a launch (at 1.2 and 1.3 times 2179 and 1095
// us split, 2151 and 1067 whole; at 2 times 53 and 58 without the sum's 5 to 17).  400
// visibilities are about 30 us of a workgroup at L = 32, 20 to 30 of them to be gained (30 us
// of 370 groups: 33 split, 30 whole; 37 of 484: 27).  Measured at more: 52 groups of 2664
// subgrids, L = 32, 788 us whole, 45 split; 13 of 703, L = 96, 1058 and 100; FP64, 19 groups,
// L = 96, 4089 and 1221; 156 heavy ones, L = 64, 7705 and 2073.
bool worth_split(int L, int64_t max_cost, int64_t total) {
  return 2 * max_cost * groups_in_flight(L) > 5 * total && max_cost * L > 400 * 32;
}

// Split the groups into parts for the gridder: one workgroup per group leaves the chip to
// the heaviest ones where groups are few or uneven.  Parts of half the work that evenly
// falls to a workgroup in flight, but not of less than three subgrids' least.
void split_groups(aidg_plan* p) {
  const auto& t = p->table;
  const size_t n = t.size(), groups = p->grp_begin.size() - 1;
  p->cost_prefix.assign(n + 1, 0);
  for (size_t i = 0; i < n; ++i) p->cost_prefix[i + 1] = p->cost_prefix[i] + grid_cost(t[i]);
  const int64_t total = p->cost_prefix[n];
  for (size_t k = 0; k < groups; ++k)
    p->max_group_cost = std::max(p->max_group_cost, p->cost_prefix[p->grp_begin[k + 1]] - p->cost_prefix[p->grp_begin[k]]);
  p->part_begin = p->grp_begin;
  p->sg_part = p->sg_group;
  const int64_t cap = std::max<int64_t>(kMinPartCost, total / (2 * groups_in_flight(p->g.L)));
  if (!worth_split(p->g.L, p->max_group_cost, total) || p->max_group_cost <= cap) return;
  p->part_begin.assign(1, 0);
  for (size_t k = 0; k < groups; ++k)
    for (int64_t b = p->grp_begin[k], e = b; b < p->grp_begin[k + 1]; b = e) {
      for (; e < p->grp_begin[k + 1] && (e == b || p->cost_prefix[e + 1] - p->cost_prefix[b] <= cap); ++e)
        p->sg_part[e] = (int32_t)p->part_begin.size() - 1;
      p->part_begin.push_back(e);
    }
}

// Parts beyond one per group that split_groups would make of an estimated partition: its
// rules, each centre's subgrids taken as equal, and a quarter more where they decide.
int64_t estimate_parts(const Geometry& g, const ShapeEstimate& se) {
  double vis = 0, total = 0, heaviest = 0, parts = 0;
  auto cost = [](const CentreEstimate& c) { return std::max(c.n_vis, 32 * c.n_subgrids) + 20 * c.n_subgrids; };
  for (const CentreEstimate& c : se.centres) {
    vis += c.n_vis;
    total += cost(c);
  }
  const double cap_vis = std::max<double>(g.max_sg_vis, kGroupVisFactor * vis / std::max<size_t>(se.centres.size(), 1));
  const double cap = std::max<double>(kMinPartCost, total / (2 * groups_in_flight(g.L)));
  for (const CentreEstimate& c : se.centres) {
    heaviest = std::max(heaviest, cost(c) * std::min(1.0, cap_vis / std::max(c.n_vis, 1.0)));
    parts += std::ceil(c.n_subgrids / std::max(1.0, std::floor(cap * c.n_subgrids / cost(c)))) - 1;
  }
  if (!worth_split(g.L, (int64_t)(1.25 * heaviest) + 1, (int64_t)total) || 1.25 * heaviest <= cap) return 0;
  return std::max<int64_t>(0, std::min<int64_t>((int64_t)parts, se.n_subgrids - se.n_groups));
}

// Launch one kernel class over subgrids [b0, b0 + n) of one plan.
aidg_status run(aidg_plan* p, KernelClass k, int64_t b0, int64_t n, const void* in, void* out,
                void* stream, int adjoint = 0) {
  hipStream_t st = reinterpret_cast<hipStream_t>(stream);
  TimedLaunch tl(p, st);
  int rc;
  if (k == kZeroVis) {
    rc = launch_zero_vis(p->g.precision, p->d_excl, p->n_excluded, out, stream);
  } else {
    Group g;
    std::memset(&g, 0, sizeof(g));
    g.n = 1;
    g.matrix = k == kGridDft ? p->matrix_grid : p->matrix_degrid;
    g.total_sg = n;
    g.total_grp = p->sg_group[b0 + n - 1] - p->sg_group[b0] + 1;
    g.total_part = p->sg_part[b0 + n - 1] - p->sg_part[b0] + 1;
    g.split = p->split && (k == kGridDft || k == kFftAdd);
    g.scratch = p->d_scratch;
    g.job[0] = {p->d_args, in, out, b0, b0 + n, p->sg_group[b0], 0, 0, adjoint, 0, p->sg_part[b0], 0};
    rc = launch_group(k, p->g.L, p->g.precision, g, stream, p->max_nv);
  }
  if (rc != 0) return hip_fail((hipError_t)rc, "kernel launch");
  tl.done(k, k == kZeroVis ? 0 : p->vp_prefix[b0 + n] - p->vp_prefix[b0], k == kZeroVis ? 0 : n);
  return AIDG_OK;
}

template <typename T>
aidg_status dalloc(T** p, size_t bytes, aidg_plan* plan, const char* what, hipStream_t stream) {
  void* q = nullptr;
  const size_t n = std::max<size_t>(bytes, 256);
  const hipError_t e = plan->async_mem ? hipMallocAsync(&q, n, stream) : hipMalloc(&q, n);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    return fail(AIDG_E_NOMEM, std::string("device allocation of ") + what + " failed: " +
                                  hipGetErrorString(e));
  }
  *p = reinterpret_cast<T*>(q);
  plan->device_bytes += n;
  return AIDG_OK;
}

// Inverse A-term mode: recompute the (A^-1)^H planes and the normalisation map from
// the plan's A-terms, on stream.
aidg_status refresh_inverse_aterms(aidg_plan* p, hipStream_t stream) {
  if (!p->g.amode) return AIDG_OK;
  const int64_t n = (int64_t)p->n_int * p->n_st * p->g.L * p->g.L;
  int rc = launch_aterm_inverse_h(p->g.precision, p->d_aterms, p->d_ainvh, n, stream);
  if (rc == 0)
    rc = launch_aterm_norm(p->g.precision, p->d_ainvh, p->d_npairs, p->d_ncount, p->n_pairs, p->n_chunks,
                           p->pair_chunk, p->g.L * p->g.L, p->n_total > 0 ? 1.0 / p->n_total : 0.0,
                           p->d_npartial, p->d_nmap, stream);
  return rc == 0 ? AIDG_OK : hip_fail((hipError_t)rc, "inverse A-term kernels");
}

}  // namespace

namespace {

// Shared checks of aidg_invert / aidg_predict.
aidg_status image_args(aidg_plan* plan, const void* a, const void* b, const void* ws, int64_t ws_bytes) {
  if (!plan || !a || !b || !ws) return fail(AIDG_E_INVALID, "NULL plan, grid, image or workspace");
  if (!plan->img_ok)
    return fail(AIDG_E_UNSUPPORTED, "image-level transforms need N = 2^a 3^b 5^c <= 8192 with a row of N "
                                    "complex values within 64 KB");
  const int64_t N = plan->g.N;
  if (ws_bytes < 2 * N * N * (int64_t)plan->elem)
    return fail(AIDG_E_INVALID, "workspace smaller than aidg_image_workspace_bytes");
  return AIDG_OK;
}

// Run one image-level launcher, timed as class k when the plan is profiling.
template <typename F>
aidg_status image_step(aidg_plan* p, hipStream_t st, KernelClass k, F&& launch) {
  TimedLaunch tl(p, st);
  const int rc = launch();
  if (rc != 0) return hip_fail((hipError_t)rc, "image kernel launch");
  tl.done(k, 0, 0);
  return AIDG_OK;
}

// Gridding and degridding of a whole plan, batch by batch; adjoint = 1 selects the
// exact adjoint of the other direction (differs on Stokes-I plans only).
aidg_status grid_calls(aidg_plan* plan, const void* vis, void* grid, void* hip_stream, int adjoint) {
  if (!plan || !vis || !grid) return fail(AIDG_E_INVALID, "NULL plan, vis or grid");
  BusyGuard guard(plan);
  if (!guard.ok) return fail(AIDG_E_BUSY, "plan in use by another thread");
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  hipError_t e = hipStreamWaitEvent(st, plan->last, 0);
  if (e != hipSuccess) return hip_fail(e, "hipStreamWaitEvent");
  for (size_t b = 0; b + 1 < plan->batch_begin.size(); ++b) {
    const int64_t b0 = plan->batch_begin[b], nb = plan->batch_begin[b + 1] - b0;
    aidg_status r = run(plan, kGridDft, b0, nb, vis, nullptr, hip_stream, adjoint);
    if (r == AIDG_OK) r = run(plan, kFftAdd, b0, nb, nullptr, grid, hip_stream, adjoint);
    if (r != AIDG_OK) return r;
  }
  e = hipEventRecord(plan->last, st);
  return e == hipSuccess ? AIDG_OK : hip_fail(e, "hipEventRecord");
}

aidg_status degrid_calls(aidg_plan* plan, const void* grid, void* vis_out, void* hip_stream, int adjoint) {
  if (!plan || !vis_out || !grid) return fail(AIDG_E_INVALID, "NULL plan, grid or vis");
  BusyGuard guard(plan);
  if (!guard.ok) return fail(AIDG_E_BUSY, "plan in use by another thread");
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  hipError_t e = hipStreamWaitEvent(st, plan->last, 0);
  if (e != hipSuccess) return hip_fail(e, "hipStreamWaitEvent");
  aidg_status r = AIDG_OK;
  if (plan->n_excluded > 0) r = run(plan, kZeroVis, 0, 0, nullptr, vis_out, hip_stream);
  if (r != AIDG_OK) return r;
  for (size_t b = 0; b + 1 < plan->batch_begin.size(); ++b) {
    const int64_t b0 = plan->batch_begin[b], nb = plan->batch_begin[b + 1] - b0;
    r = run(plan, kSplitIfft, b0, nb, grid, nullptr, hip_stream, adjoint);
    if (r == AIDG_OK) r = run(plan, kDegridDft, b0, nb, nullptr, vis_out, hip_stream, adjoint);
    if (r != AIDG_OK) return r;
  }
  e = hipEventRecord(plan->last, st);
  return e == hipSuccess ? AIDG_OK : hip_fail(e, "hipEventRecord");
}

// Shared body of aidg_execute and aidg_execute_static: pack the items' ranges into
// grouped launches whose group images fit in `scratch` (scratch_bytes), after the
// named plans' earlier work and, when `last` is given, after the event's; record the
// plans' events and `last` behind the launches.
aidg_status execute_items(void* scratch, int64_t scratch_bytes, hipEvent_t last, const aidg_work* items,
                          int32_t n_items, void* hip_stream) {
  if ((n_items > 0 && !items) || n_items < 0) return fail(AIDG_E_INVALID, "bad items");
  for (int32_t i = 0; i < n_items; ++i) {
    const aidg_work& w = items[i];
    if (!w.plan || !w.in || !w.out || (w.direction != AIDG_DIR_GRID && w.direction != AIDG_DIR_DEGRID) ||
        w.sg_begin < 0 || w.sg_end < w.sg_begin || w.sg_end > (int64_t)w.plan->table.size())
      return fail(AIDG_E_INVALID, "work item " + std::to_string(i) + ": bad plan, buffers, direction or range");
  }
  std::vector<aidg_plan*> plans;
  for (int32_t i = 0; i < n_items; ++i)
    if (std::find(plans.begin(), plans.end(), items[i].plan) == plans.end()) plans.push_back(items[i].plan);
  size_t held = 0;
  for (; held < plans.size(); ++held) {
    bool ex2 = false;
    if (!plans[held]->busy.compare_exchange_strong(ex2, true)) break;
  }
  auto release = [&]() {
    for (size_t k = 0; k < held; ++k) plans[k]->busy.store(false);
  };
  if (held < plans.size()) {
    release();
    return fail(AIDG_E_BUSY, "a plan is in use by another thread");
  }
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  aidg_status r = AIDG_OK;
  hipError_t e = last ? hipStreamWaitEvent(st, last, 0) : hipSuccess;
  for (aidg_plan* p : plans)
    if (e == hipSuccess) e = hipStreamWaitEvent(st, p->last, 0);
  if (e != hipSuccess) r = hip_fail(e, "hipStreamWaitEvent");
  // degridding ranges that start the table also clear the excluded visibilities
  for (int32_t i = 0; i < n_items && r == AIDG_OK; ++i) {
    const aidg_work& w = items[i];
    if (w.direction == AIDG_DIR_DEGRID && w.sg_begin == 0 && w.plan->n_excluded > 0) {
      const int rc = launch_zero_vis(w.plan->g.precision, w.plan->d_excl, w.plan->n_excluded, w.out,
                                     hip_stream);
      if (rc != 0) r = hip_fail((hipError_t)rc, "zeroing excluded visibilities");
    }
  }
  // group by (direction, L, precision, kernels); pack ranges into launches
  std::vector<bool> done(n_items, false);
  for (int32_t i0 = 0; i0 < n_items && r == AIDG_OK; ++i0) {
    if (done[i0]) continue;
    const int dir = items[i0].direction, L = items[i0].plan->g.L, prec = items[i0].plan->g.precision;
    auto matrix = [&](const aidg_plan* p) { return dir == AIDG_DIR_GRID ? p->matrix_grid : p->matrix_degrid; };
    const MatrixForm mx = matrix(items[i0].plan);
    const int64_t per_sg = (int64_t)4 * L * L * (prec == AIDG_FP32 ? 8 : 16);
    const int64_t cap = std::min<int64_t>(scratch_bytes / per_sg, 65535);
    // grid by parts where they fit one launch's images and the heaviest group of the items
    // would outlast the others
    int64_t parts = 0, items_cost = 0, max_cost = 0;
    for (int32_t i = i0; i < n_items && dir == AIDG_DIR_GRID; ++i) {
      const aidg_work& w = items[i];
      const aidg_plan* p = w.plan;
      if (done[i] || w.direction != dir || p->g.L != L || p->g.precision != prec || matrix(p) != mx ||
          w.sg_begin == w.sg_end)
        continue;
      parts += p->sg_part[w.sg_end - 1] - p->sg_part[w.sg_begin] + 1;
      items_cost += p->cost_prefix[w.sg_end] - p->cost_prefix[w.sg_begin];
      max_cost = std::max(max_cost, p->max_group_cost);
    }
    const bool split = parts > 0 && parts <= cap && worth_split(L, max_cost, items_cost);
    if (cap < 1) {
      r = fail(AIDG_E_INVALID, "workspace smaller than one subgrid image");
      break;
    }
    Group g;
    std::memset(&g, 0, sizeof(g));
    g.scratch = scratch;
    g.matrix = mx;
    g.split = split;
    int max_nv = 1;
    auto flush = [&]() -> aidg_status {
      if (g.total_sg == 0) return AIDG_OK;
      const KernelClass k0 = dir == AIDG_DIR_GRID ? kGridDft : kSplitIfft;
      const KernelClass k1 = dir == AIDG_DIR_GRID ? kFftAdd : kDegridDft;
      int rc = launch_group(k0, L, prec, g, hip_stream, max_nv);
      if (rc == 0) rc = launch_group(k1, L, prec, g, hip_stream, max_nv);
      std::memset(&g, 0, sizeof(g));
      g.scratch = scratch;
      g.matrix = mx;
      g.split = split;
      max_nv = 1;
      return rc == 0 ? AIDG_OK : hip_fail((hipError_t)rc, "grouped kernel launch");
    };
    for (int32_t i = i0; i < n_items && r == AIDG_OK; ++i) {
      const aidg_work& w = items[i];
      if (done[i] || w.direction != dir || w.plan->g.L != L || w.plan->g.precision != prec ||
          matrix(w.plan) != mx)
        continue;
      done[i] = true;
      // a launch takes whole or partial groups until `cap` group images
      const aidg_plan* p = w.plan;
      for (int64_t b = w.sg_begin; b < w.sg_end && r == AIDG_OK;) {
        if (g.n == kMaxGroup || g.total_grp == cap) r = flush();
        if (r != AIDG_OK) break;
        const int64_t g0 = p->sg_group[b], room = cap - g.total_grp;
        const int64_t gn = (int64_t)p->grp_begin.size() - 1;
        const int64_t e = g0 + room < gn ? std::min(w.sg_end, p->grp_begin[g0 + room]) : w.sg_end;
        g.job[g.n] = {p->d_args, w.in, w.out, b, e, g0, g.total_sg, g.total_grp, 0, 0, p->sg_part[b], g.total_part};
        g.n += 1;
        g.total_sg += e - b;
        g.total_grp += p->sg_group[e - 1] - g0 + 1;
        g.total_part += p->sg_part[e - 1] - p->sg_part[b] + 1;
        max_nv = std::max(max_nv, p->max_nv);
        b = e;
      }
    }
    if (r == AIDG_OK) r = flush();
  }
  if (r == AIDG_OK) {
    e = last ? hipEventRecord(last, st) : hipSuccess;
    for (aidg_plan* p : plans)
      if (e == hipSuccess) e = hipEventRecord(p->last, st);
    if (e != hipSuccess) r = hip_fail(e, "hipEventRecord");
  }
  release();
  return r;
}

}  // namespace

extern "C" {

int32_t aidg_abi_version(void) { return AIDG_ABI_VERSION; }

const char* aidg_last_error(void) { return g_last_error.c_str(); }

aidg_status aidg_partition(const aidg_geometry* geo, int32_t n_stations, int32_t n_baselines,
                           int32_t n_times, int32_t n_chans, const int32_t* baselines,
                           const double* uvw_m, const double* freqs_hz, aidg_subgrid* out,
                           int64_t cap, int64_t* n_out, double* w_step_out) {
  try {
    Geometry g;
    std::string err;
    aidg_status st = validate_geometry(geo, &g, &err);
    if (st != AIDG_OK) return fail(st, err);
    PartitionResult pr;
    st = partition(g, n_stations, n_baselines, n_times, n_chans, baselines, uvw_m, freqs_hz, &pr, &err);
    if (st != AIDG_OK) return fail(st, err);
    if (n_out) *n_out = (int64_t)pr.table.size();
    if (w_step_out) *w_step_out = pr.w_step;
    if ((int64_t)pr.table.size() > cap || (pr.table.size() && !out))
      return fail(AIDG_E_INVALID, "output capacity too small for the partition");
    std::copy(pr.table.begin(), pr.table.end(), out);
    return AIDG_OK;
  } catch (const std::bad_alloc&) {
    return fail(AIDG_E_NOMEM, "host allocation failed");
  } catch (...) {
    return fail(AIDG_E_INVALID, "unexpected host exception");
  }
}

aidg_status aidg_plan_create(const aidg_geometry* geo, int32_t n_stations, int32_t n_baselines,
                             int32_t n_times, int32_t n_chans, const int32_t* baselines,
                             const double* uvw_m, const double* freqs_hz, const void* aterms,
                             const aidg_subgrid* table, int64_t n_table, void* hip_stream,
                             aidg_plan** out) {
  if (!out) return fail(AIDG_E_INVALID, "out is NULL");
  *out = nullptr;
  aidg_plan* plan = nullptr;
  try {
    plan = new aidg_plan();
    Geometry& g = plan->g;
    std::string err;
    aidg_status st = validate_geometry(geo, &g, &err);
    if (st != AIDG_OK) {
      delete plan;
      return fail(st, err);
    }
    if (!gpu_subgrid_size(g.L)) {
      delete plan;
      return fail(AIDG_E_UNSUPPORTED, "the GPU kernels support subgrid sizes 32, 64 and 96");
    }
    if (!aterms || n_baselines < 1 || n_times < 1 || n_chans < 1 || n_stations < 1) {
      delete plan;
      return fail(AIDG_E_INVALID, "empty observation or NULL A-terms");
    }
    plan->n_st = n_stations;
    plan->nbl = n_baselines;
    plan->nt = n_times;
    plan->nc = n_chans;
    plan->n_int = (n_times + g.aterm_interval - 1) / g.aterm_interval;
    plan->elem = g.precision == AIDG_FP32 ? 8 : 16;

    PartitionResult pr;
    if (!baselines || !uvw_m || !freqs_hz) {
      st = AIDG_E_INVALID;
      err = "NULL host arrays";
    } else if (!table) {
      st = partition(g, n_stations, n_baselines, n_times, n_chans, baselines, uvw_m, freqs_hz, &pr,
                     &err);
    } else if (n_table < 0) {
      st = AIDG_E_INVALID;
      err = "negative table size";
    } else {
      st = adopt_table(g, n_stations, n_baselines, n_times, n_chans, baselines, table, n_table, &pr,
                       &err);
    }
    if (st != AIDG_OK) {
      delete plan;
      return fail(st, err);
    }
    plan->table = split_large(pr.table, g.max_sg_vis, n_times, n_chans);
    plan->n_excluded = (int64_t)pr.excluded.size();
    if (table) {
      int32_t wmax = 0;
      for (const auto& s : plan->table) wmax = std::max(wmax, s.wlayer);
      plan->W = wmax + 1;
      plan->w0.assign(plan->W, 0.0);
      for (const auto& s : plan->table) plan->w0[s.wlayer] = s.w0;
    } else {
      plan->W = (int)(pr.jmax - pr.jmin + 1);
      plan->w0.resize(plan->W);
      for (int j = 0; j < plan->W; ++j)
        plan->w0[j] = pr.w_step > 0 ? (pr.jmin + j + (g.fold ? 0.5 : 0.0)) * pr.w_step : 0.0;
    }
    // Order: subgrids with the same w-layer and centre are consecutive, so that a
    // group shares one image sum, one FFT and one grid update (gridding) or one
    // split and inverse FFT (degridding).  A group is capped at kGroupVisFactor
    // times the mean group's visibilities (larger ones become several groups with
    // the same centre) so that no gridder workgroup runs far longer than the rest.
    // Groups go longest-first (longest-processing-time-first), and inside a group
    // the largest sub-tables go first for the degridder.
    {
      auto& t = plan->table;
      auto same_centre = [](const aidg_subgrid& x, const aidg_subgrid& y) {
        return x.wlayer == y.wlayer && x.U0 == y.U0 && x.V0 == y.V0;
      };
      std::stable_sort(t.begin(), t.end(), [](const aidg_subgrid& x, const aidg_subgrid& y) {
        if (x.wlayer != y.wlayer) return x.wlayer < y.wlayer;
        if (x.V0 != y.V0) return x.V0 < y.V0;
        if (x.U0 != y.U0) return x.U0 < y.U0;
        if (x.nt * x.nc != y.nt * y.nc) return x.nt * x.nc > y.nt * y.nc;
        return x.aint != y.aint ? x.aint < y.aint : x.bl < y.bl;
      });
      struct Span {
        size_t b, e;
        int64_t nv;
      };
      std::vector<Span> spans;
      int64_t total_nv = 0, n_centres = 0;
      for (size_t i = 0; i < t.size(); ++i) {
        total_nv += (int64_t)t[i].nt * t[i].nc;
        if (i == 0 || !same_centre(t[i], t[i - 1])) ++n_centres;
      }
      const int64_t cap_nv = n_centres ? std::max<int64_t>(
          (int64_t)g.max_sg_vis, kGroupVisFactor * ((total_nv + n_centres - 1) / n_centres)) : 1;
      for (size_t i = 0; i < t.size();) {
        size_t j = i;
        int64_t nv = 0;
        while (j < t.size() && same_centre(t[j], t[i]) &&
               (j == i || nv + (int64_t)t[j].nt * t[j].nc <= cap_nv)) {
          nv += (int64_t)t[j].nt * t[j].nc;
          ++j;
        }
        spans.push_back({i, j, nv});
        i = j;
      }
      std::stable_sort(spans.begin(), spans.end(), [](const Span& x, const Span& y) { return x.nv > y.nv; });
      std::vector<aidg_subgrid> ordered;
      ordered.reserve(t.size());
      plan->grp_begin.assign(1, 0);
      plan->sg_group.clear();
      plan->sg_group.reserve(t.size());
      for (const Span& sp : spans) {
        for (size_t k = sp.b; k < sp.e; ++k) {
          ordered.push_back(t[k]);
          plan->sg_group.push_back((int32_t)(plan->grp_begin.size() - 1));
        }
        plan->grp_begin.push_back((int64_t)ordered.size());
      }
      t.swap(ordered);
    }
    split_groups(plan);
    plan->max_nv = 1;
    plan->vp_prefix.assign(plan->table.size() + 1, 0);
    for (size_t i = 0; i < plan->table.size(); ++i) {
      const aidg_subgrid& s = plan->table[i];
      plan->max_nv = std::max(plan->max_nv, s.nt * s.nc);
      plan->vp_prefix[i + 1] = plan->vp_prefix[i] + (int64_t)s.nt * s.nc * g.L * g.L;
    }

    // device records; folded sub-tables read their rows from a negated copy of uvw
    // and swap the stations' A-terms
    const double inv_c = 1.0 / kSpeedOfLight;
    bool any_folded = false;
    for (const auto& s : plan->table) any_folded = any_folded || s.folded;
    const size_t uvw_rows = (size_t)n_baselines * n_times;
    std::vector<double> uvw_dev(uvw_m, uvw_m + 3 * uvw_rows);
    if (any_folded) {
      uvw_dev.resize(6 * uvw_rows);
      for (size_t i = 0; i < 3 * uvw_rows; ++i) uvw_dev[3 * uvw_rows + i] = -uvw_m[i];
    }
    const int L = g.L;
    const bool f32 = g.precision == AIDG_FP32;
    std::vector<double> T;
    kaiser_bessel_taper(L, g.beta, &T);
    WSeries series;
    if (f32) w_series(L, g.fov, T, &series);
    plan->b_peak = series.b_peak;
    bool matrix = f32 && g.R >= kReseedDefault;  // a shorter run asks for the seeds' precision
    double cost = 0.0;  // of the degridder's other forms
    bool rising = true;  // a caller's table takes frequencies in any order
    for (int c = 1; c < n_chans && table; ++c) rising = rising && freqs_hz[c] > freqs_hz[c - 1];
    auto first_row = [&](const aidg_subgrid& s) {
      return (int64_t)s.bl * n_times + s.t0 + (s.folded ? (int64_t)uvw_rows : 0);
    };
    std::vector<SubgridDev> dev(plan->table.size());
    for (size_t i = 0; i < plan->table.size(); ++i) {
      const aidg_subgrid& s = plan->table[i];
      // the table is in the groups' order, not the rows': without, every subgrid waits for its
      // rows of w (186 thousand subgrids: 74 ms for the plan, 70 with)
      if (matrix && i + 8 < plan->table.size()) {
        const double* ahead = &uvw_dev[3 * first_row(plan->table[i + 8])];
        for (int k = 0; k < 3 * plan->table[i + 8].nt; k += 8) __builtin_prefetch(ahead + k);
      }
      SubgridDev& d = dev[i];
      std::memset(&d, 0, sizeof(d));
      d.t0 = s.t0;
      d.nt = s.nt;
      d.c0 = s.c0;
      d.nc = s.nc;
      d.U0 = s.U0;
      d.V0 = s.V0;
      d.wlayer = s.wlayer;
      d.ap = s.aint * n_stations + (s.folded ? s.st2 : s.st1);
      d.aq = s.aint * n_stations + (s.folded ? s.st1 : s.st2);
      d.part = plan->sg_part[i];
      d.vis0 = s.vis_offset;
      d.uvw0 = first_row(s);
      d.fold = s.folded;
      d.w0 = s.w0;
      d.group = plan->sg_group[i];
      const double df = s.nc > 1 ? freqs_hz[s.c0 + 1] - freqs_hz[s.c0] : 0.0;
      bool uniform = true;
      for (int c = s.c0 + 1; c < s.c0 + s.nc; ++c)
        if (std::fabs((freqs_hz[c] - freqs_hz[c - 1]) - df) > 1e-9 * std::fabs(df)) uniform = false;
      d.dfc = df * inv_c;
      d.R = uniform ? g.R : 1;
      d.kind = degrid_form(g, s.nt, s.nc, uniform);
      if (matrix) {
        // w range of the sub-table; a caller's table may also hold rows that are not finite or
        // far off the window, whose phases the fixed-point reduction would not take
        double f_lo = freqs_hz[s.c0], f_hi = freqs_hz[s.c0 + s.nc - 1];
        if (!rising) {
          f_lo = *std::min_element(freqs_hz + s.c0, freqs_hz + s.c0 + s.nc);
          f_hi = *std::max_element(freqs_hz + s.c0, freqs_hz + s.c0 + s.nc);
        }
        f_lo *= inv_c;
        f_hi *= inv_c;
        const double* x = &uvw_dev[3 * d.uvw0];
        double w_lo = x[2], w_hi = x[2];
        for (int t = 0; t < s.nt; ++t, x += 3) {
          w_lo = std::min(w_lo, x[2]);
          w_hi = std::max(w_hi, x[2]);
          if (!table) continue;
          for (double f : {f_lo, f_hi})
            if (!(std::fabs(x[0] * f * g.fov - (s.U0 - g.N / 2)) <= 0x1p18 &&
                  std::fabs(x[1] * f * g.fov - (s.V0 - g.N / 2)) <= 0x1p18 && std::isfinite(x[2] * f)))
              matrix = false;
        }
        const double lo = std::min(w_lo * f_lo, w_lo * f_hi) - s.w0, hi = std::max(w_hi * f_lo, w_hi * f_hi) - s.w0;
        d.wmid = (float)(0.5 * (lo + hi));
        const double dw = std::max(hi - d.wmid, d.wmid - lo);
        d.order = w_series_order(series, d.wmid, dw);
        matrix = matrix && d.order >= 0;
        if (matrix) {
          plan->w_terms = std::max(plan->w_terms, d.order & kWTerms);
          plan->n_split += (d.order & kWSplit) != 0;
        }
      }
      cost += degrid_cost(d.kind, s.nt, s.nc);
      plan->n_pervis += d.kind == kDegridPerVis;
      plan->n_direct += d.kind == kDegridDirect;
    }
    if (!matrix) plan->w_terms = plan->n_split = 0;
    plan->matrix_grid = !matrix ? kMatrixNone : plan->n_split ? kMatrixWide : kMatrixPlain;
    // The matrix degridder works in blocks of 32 visibilities and takes the same time for 1
    // as for 32: 16, 50 and 105 ns per subgrid at L = 32, 64, 96 with the chip full, and 16.6,
    // 55 to 56 and 118 to 125 where many split the series' first term.  The other forms, with
    // one row per subgrid and a modelled cost of 9 (L = 32) take 10 ns; of 5, 8, 10 and 13
    // (L = 64) 45, 47, 51 and 54; of 6, 10, 13 and 17 (L = 96) 86, 97, 106 and 121; with rows
    // of one channel and costs of 15.6 and 20 17 and 19 (L = 32).  The lines are where the two
    // meet.
    const double n_sg = (double)plan->table.size(), n_split = (double)plan->n_split;
    const double meet = L == 32 ? 14.5 * n_sg + 1.5 * n_split : (L == 64 ? 9.0 : 12.5) * n_sg + 4.0 * n_split;
    if (matrix && g.degrid_form == AIDG_DEGRID_AUTO && cost >= meet)
      plan->matrix_degrid = kMatrixPlain;  // its kernel chooses by subgrid
    // inverse A-term mode: distinct (A_p plane, A_q plane) pairs with their visibility
    // counts, for the normalisation map
    std::vector<int32_t> pairs;
    std::vector<double> pair_count;
    if (g.amode) {
      std::map<std::pair<int32_t, int32_t>, double> cnt;
      for (const SubgridDev& d : dev) cnt[{d.ap, d.aq}] += (double)d.nt * d.nc;
      for (const auto& kv : cnt) {
        pairs.push_back(kv.first.first);
        pairs.push_back(kv.first.second);
        pair_count.push_back(kv.second);
        plan->n_total += kv.second;
      }
      plan->n_pairs = (int64_t)pair_count.size();
      // about 64 pairs per chunk and at most 64 chunks
      plan->n_chunks = (int)std::max<int64_t>(1, std::min<int64_t>(64, (plan->n_pairs + 63) / 64));
      plan->pair_chunk = std::max<int64_t>(1, (plan->n_pairs + plan->n_chunks - 1) / plan->n_chunks);
    }
    std::vector<double> fc(n_chans);
    for (int c = 0; c < n_chans; ++c) fc[c] = freqs_hz[c] * inv_c;
    for (int y = 0; y < L; ++y)
      for (int x = 0; x < L; ++x)
        if ((x + y) & 1) T[(size_t)y * L + x] = -T[(size_t)y * L + x];
    std::vector<double> tw(2 * L);
    for (int k = 0; k < L; ++k) {
      const double ang = -2.0 * M_PI * k / L;
      tw[2 * k] = std::cos(ang);
      tw[2 * k + 1] = std::sin(ang);
    }
    const TableLayout tl(L, plan->elem);
    std::vector<char> tables(tl.bytes);
    for (int i = 0; i < L * L; ++i) {
      if (f32) reinterpret_cast<float*>(tables.data() + tl.taper)[i] = (float)T[i];
      else reinterpret_cast<double*>(tables.data() + tl.taper)[i] = T[i];
    }
    for (int k = 0; k < 2 * L; ++k) {
      if (f32) reinterpret_cast<float*>(tables.data() + tl.twiddle)[k] = (float)tw[k];
      else reinterpret_cast<double*>(tables.data() + tl.twiddle)[k] = tw[k];
    }
    if (f32) {
      double* n1 = reinterpret_cast<double*>(tables.data() + tl.axis_n1);
      uint32_t* b = reinterpret_cast<uint32_t*>(tables.data() + tl.axis_b);
      float* tc = reinterpret_cast<float*>(tables.data() + tl.taper_cross);
      for (int x = 0; x < L; ++x) {
        n1[x] = series.axis_n1[x];
        const double v = series.b_peak > 0 ? series.b[x] / series.b_peak : 0.0;
        const _Float16 part[2] = {(_Float16)v, (_Float16)(v - (double)(_Float16)v)};
        for (int i = 0; i < 2; ++i) {
          uint16_t u;
          std::memcpy(&u, &part[i], 2);
          b[i * L + x] = (uint32_t)u << 16 | u;
        }
      }
      for (int i = 0; i < L * L; ++i) {
        // A value passes through three phasors of the transcendental unit (the two axes and the
        // cross term), whose cosine and sine leave |z| short of 1 by 3.25e-8 on average.
        tc[2 * i] = (float)(T[i] * (1.0 + 3 * 3.25e-8));
        tc[2 * i + 1] = (float)series.cross[i];
      }
    }
    // image level: twiddles exp(-2 pi i k / N) and the reciprocal 1 / t[X] of the taper
    // axis at image resolution
    std::vector<double> img_t, img_tw;
    plan->img_ok = image_radices(g.N, (int)plan->elem, &plan->img_fr);
    if (plan->img_ok) {
      kaiser_bessel_axis(g.N, g.beta, &img_t);
      for (double& v : img_t) v = 1.0 / v;
      img_tw.resize(2 * (size_t)g.N);
      for (int k = 0; k < g.N; ++k) {
        const double ang = -2.0 * M_PI * k / g.N;
        img_tw[2 * (size_t)k] = std::cos(ang);
        img_tw[2 * (size_t)k + 1] = std::sin(ang);
      }
    }
    std::vector<float> img_twf(img_tw.begin(), img_tw.end());

    plan->aterm_bytes = (size_t)plan->n_int * n_stations * L * L * 4 * plan->elem;
    const size_t per_sg = (size_t)4 * L * L * plan->elem;
    const int64_t nsg = (int64_t)plan->table.size();
    const int64_t n_groups = (int64_t)plan->grp_begin.size() - 1, n_parts = (int64_t)plan->part_begin.size() - 1;
    std::vector<int64_t> index(plan->grp_begin);
    if (n_parts > n_groups) index.insert(index.end(), plan->part_begin.begin(), plan->part_begin.end());
    plan->batch = std::max<int64_t>(1, std::min<int64_t>(g.workspace / (int64_t)per_sg, 65535));
    plan->split = n_parts > n_groups && n_parts <= plan->batch;
    plan->batch = std::min<int64_t>(plan->batch, std::max<int64_t>(plan->split ? n_parts : n_groups, 1));
    plan->scratch_bytes = (size_t)plan->batch * per_sg;
    plan->batch_begin.clear();
    for (int64_t k = 0; k < n_groups; k += plan->batch) plan->batch_begin.push_back(plan->grp_begin[k]);
    plan->batch_begin.push_back(nsg);

    hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
    hipError_t e = hipGetDevice(&plan->device);
    if (e != hipSuccess) {
      delete plan;
      return hip_fail(e, "hipGetDevice");
    }
    int pools = 0;
    plan->async_mem = hipDeviceGetAttribute(&pools, hipDeviceAttributeMemoryPoolsSupported, plan->device) ==
                          hipSuccess && pools != 0 && release_stream(plan->device) != nullptr;
    (void)hipGetLastError();
    // on failure after the first allocation: let the creation stream finish, then free
    auto abandon = [&]() {
      (void)hipStreamSynchronize(stream);
      (void)hipGetLastError();
      plan->release();
      delete plan;
    };
    if ((st = dalloc(&plan->d_sg, dev.size() * sizeof(SubgridDev), plan, "subgrid table", stream)) ||
        (st = dalloc(&plan->d_uvw, uvw_dev.size() * sizeof(double), plan, "uvw", stream)) ||
        (st = dalloc(&plan->d_fc, fc.size() * sizeof(double), plan, "frequencies", stream)) ||
        (st = dalloc(&plan->d_aterms, plan->aterm_bytes, plan, "A-terms", stream)) ||
        (st = dalloc(&plan->d_tables, tables.size(), plan, "tables", stream)) ||
        (st = dalloc(&plan->d_excl, pr.excluded.size() * sizeof(int64_t), plan, "excluded list", stream)) ||
        (st = dalloc(&plan->d_grp, index.size() * sizeof(int64_t), plan, "group index", stream)) ||
        (st = dalloc(&plan->d_scratch, plan->scratch_bytes, plan, "subgrid workspace", stream)) ||
        (st = dalloc(&plan->d_args, sizeof(KernelArgs), plan, "launch parameters", stream)) ||
        (plan->img_ok &&
         ((st = dalloc(&plan->d_img_tw, (size_t)g.N * plan->elem, plan, "image twiddles", stream)) ||
          (st = dalloc(&plan->d_img_itaper, (size_t)g.N * sizeof(double), plan, "image taper", stream)))) ||
        (g.amode &&
         ((st = dalloc(&plan->d_ainvh, plan->aterm_bytes, plan, "inverse A-terms", stream)) ||
          (st = dalloc(&plan->d_npairs, pairs.size() * sizeof(int32_t), plan, "A-term pairs", stream)) ||
          (st = dalloc(&plan->d_ncount, pair_count.size() * sizeof(double), plan, "pair counts", stream)) ||
          (st = dalloc(&plan->d_npartial, (size_t)plan->n_chunks * L * L * sizeof(double), plan,
                       "normalisation partial sums", stream)) ||
          (st = dalloc(&plan->d_nmap, (size_t)L * L * sizeof(double), plan, "normalisation map", stream))))) {
      abandon();
      return st;
    }
    const KernelArgs host_args = plan->args();
    struct Copy {
      void* dst;
      const void* src;
      size_t n;
      hipMemcpyKind kind;
    } copies[] = {
        {plan->d_sg, dev.data(), dev.size() * sizeof(SubgridDev), hipMemcpyHostToDevice},
        {plan->d_uvw, uvw_dev.data(), uvw_dev.size() * sizeof(double), hipMemcpyHostToDevice},
        {plan->d_fc, fc.data(), fc.size() * sizeof(double), hipMemcpyHostToDevice},
        {plan->d_aterms, aterms, plan->aterm_bytes, hipMemcpyDeviceToDevice},
        {plan->d_tables, tables.data(), tables.size(), hipMemcpyHostToDevice},
        {plan->d_excl, pr.excluded.data(), pr.excluded.size() * sizeof(int64_t), hipMemcpyHostToDevice},
        {plan->d_grp, index.data(), index.size() * sizeof(int64_t), hipMemcpyHostToDevice},
        {plan->d_args, &host_args, sizeof(KernelArgs), hipMemcpyHostToDevice},
        {plan->d_img_tw, f32 ? (const void*)img_twf.data() : (const void*)img_tw.data(),
         plan->img_ok ? (size_t)g.N * plan->elem : 0, hipMemcpyHostToDevice},
        {plan->d_img_itaper, img_t.data(), plan->img_ok ? (size_t)g.N * sizeof(double) : 0,
         hipMemcpyHostToDevice},
        {plan->d_npairs, pairs.data(), pairs.size() * sizeof(int32_t), hipMemcpyHostToDevice},
        {plan->d_ncount, pair_count.data(), pair_count.size() * sizeof(double), hipMemcpyHostToDevice},
    };
    for (const Copy& c : copies) {
      if (!c.n) continue;
      e = hipMemcpyAsync(c.dst, c.src, c.n, c.kind, stream);
      if (e != hipSuccess) {
        abandon();
        return hip_fail(e, "hipMemcpyAsync (plan upload)");
      }
    }
    if ((st = refresh_inverse_aterms(plan, stream)) != AIDG_OK) {
      abandon();
      return st;
    }
    if ((e = hipEventCreateWithFlags(&plan->last, hipEventDisableTiming)) != hipSuccess ||
        (e = hipEventRecord(plan->last, stream)) != hipSuccess ||
        (e = hipStreamSynchronize(stream)) != hipSuccess) {
      abandon();
      return hip_fail(e, "plan upload");
    }
    *out = plan;
    return AIDG_OK;
  } catch (const std::bad_alloc&) {
    if (plan) {
      if (plan->async_mem && plan->d_sg) (void)hipDeviceSynchronize();  // allocations in flight
      plan->release();
      delete plan;
    }
    return fail(AIDG_E_NOMEM, "host allocation failed");
  }
}

aidg_status aidg_plan_info_get(const aidg_plan* plan, aidg_plan_info* info) {
  if (!plan || !info) return fail(AIDG_E_INVALID, "NULL plan or info");
  std::memset(info, 0, sizeof(*info));
  info->n_subgrids = (int64_t)plan->table.size();
  info->n_vis = (int64_t)plan->nbl * plan->nt * plan->nc;
  info->n_excluded = plan->n_excluded;
  info->n_wlayers = plan->W;
  info->subgrid_size = plan->g.L;
  info->w_step = plan->g.w_step;
  info->device_bytes = (int64_t)plan->device_bytes;
  info->workspace_bytes = (int64_t)plan->scratch_bytes;
  info->grid_bytes = (int64_t)plan->W * plan->g.npol * plan->g.N * plan->g.N * (int64_t)plan->elem;
  info->vis_bytes = info->n_vis * 4 * (int64_t)plan->elem;
  info->n_batches = plan->batch_begin.empty() ? 0 : (int64_t)plan->batch_begin.size() - 1;
  info->n_groups = plan->grp_begin.empty() ? 0 : (int64_t)plan->grp_begin.size() - 1;
  info->max_subgrid_vis = plan->max_nv;
  info->n_subgrids_pervis = plan->n_pervis;
  info->n_subgrids_direct = plan->n_direct;
  return AIDG_OK;
}

aidg_status aidg_plan_kernels(const aidg_plan* plan, aidg_plan_kernel_info* info) {
  if (!plan || !info) return fail(AIDG_E_INVALID, "NULL plan or info");
  static_assert(kMatrixNone == AIDG_KERNEL_GENERAL && kMatrixPlain == AIDG_KERNEL_MATRIX &&
                    kMatrixWide == AIDG_KERNEL_MATRIX_WIDE, "one numbering");
  *info = {plan->matrix_grid, plan->matrix_degrid, plan->w_terms, 0, plan->n_split};
  return AIDG_OK;
}

aidg_status aidg_plan_subgrids(const aidg_plan* plan, aidg_subgrid* out, int64_t cap) {
  if (!plan || (!out && cap > 0)) return fail(AIDG_E_INVALID, "NULL plan or output");
  const int64_t n = std::min<int64_t>(cap, (int64_t)plan->table.size());
  if (n > 0) std::memcpy(out, plan->table.data(), (size_t)n * sizeof(aidg_subgrid));
  return AIDG_OK;
}

aidg_status aidg_plan_wlayers(const aidg_plan* plan, double* w0, int32_t cap) {
  if (!plan || (!w0 && cap > 0)) return fail(AIDG_E_INVALID, "NULL plan or output");
  for (int j = 0; j < std::min(cap, (int32_t)plan->W); ++j) w0[j] = plan->w0[j];
  return AIDG_OK;
}

aidg_status aidg_plan_set_aterms(aidg_plan* plan, const void* aterms, void* hip_stream) {
  if (!plan || !aterms) return fail(AIDG_E_INVALID, "NULL plan or A-terms");
  BusyGuard guard(plan);
  if (!guard.ok) return fail(AIDG_E_BUSY, "plan in use by another thread");
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  hipError_t e = hipStreamWaitEvent(st, plan->last, 0);
  if (e == hipSuccess)
    e = hipMemcpyAsync(plan->d_aterms, aterms, plan->aterm_bytes, hipMemcpyDeviceToDevice, st);
  if (e != hipSuccess) return hip_fail(e, "A-term copy");
  const aidg_status r = refresh_inverse_aterms(plan, st);
  if (r != AIDG_OK) return r;
  e = hipEventRecord(plan->last, st);
  return e == hipSuccess ? AIDG_OK : hip_fail(e, "hipEventRecord");
}

aidg_status aidg_plan_aterm_norm(aidg_plan* plan, double* out, int64_t cap) {
  if (!plan || (!out && cap > 0)) return fail(AIDG_E_INVALID, "NULL plan or output");
  if (!plan->g.amode) return fail(AIDG_E_INVALID, "the plan is in the adjoint A-term mode (no normalisation)");
  BusyGuard guard(plan);
  if (!guard.ok) return fail(AIDG_E_BUSY, "plan in use by another thread");
  hipError_t e = hipEventSynchronize(plan->last);
  const int64_t n = std::min<int64_t>(cap, (int64_t)plan->g.L * plan->g.L);
  if (e == hipSuccess && n > 0) e = hipMemcpy(out, plan->d_nmap, (size_t)n * sizeof(double), hipMemcpyDeviceToHost);
  return e == hipSuccess ? AIDG_OK : hip_fail(e, "normalisation map copy");
}

aidg_status aidg_grid(aidg_plan* plan, const void* vis, void* grid, void* hip_stream) {
  return grid_calls(plan, vis, grid, hip_stream, 0);
}

aidg_status aidg_grid_adjoint(aidg_plan* plan, const void* vis, void* grid, void* hip_stream) {
  if (plan && plan->g.amode) return fail(AIDG_E_INVALID, "inverse A-term mode: gridding has no adjoint pair");
  return grid_calls(plan, vis, grid, hip_stream, 1);
}

aidg_status aidg_degrid(aidg_plan* plan, const void* grid, void* vis_out, void* hip_stream) {
  return degrid_calls(plan, grid, vis_out, hip_stream, 0);
}

aidg_status aidg_degrid_adjoint(aidg_plan* plan, const void* grid, void* vis_out, void* hip_stream) {
  if (plan && plan->g.amode) return fail(AIDG_E_INVALID, "inverse A-term mode: gridding has no adjoint pair");
  return degrid_calls(plan, grid, vis_out, hip_stream, 1);
}

aidg_status aidg_footprint_estimate(const aidg_geometry* geo, int32_t n_stations, int32_t n_baselines,
                                    int32_t n_times, int32_t n_chans, const double* uvw_m,
                                    const double* freqs_hz, aidg_footprint* out) {
  if (!out) return fail(AIDG_E_INVALID, "out is NULL");
  std::memset(out, 0, sizeof(*out));
  try {
    Geometry g;
    std::string err;
    aidg_status st = validate_geometry(geo, &g, &err);
    if (st != AIDG_OK) return fail(st, err);
    if (n_stations < 1 || n_baselines < 0 || n_times < 0 || n_chans < 0 ||
        (n_baselines && n_times && !uvw_m) || (n_chans && !freqs_hz))
      return fail(AIDG_E_INVALID, "bad observation sizes or NULL host arrays");
    for (int c = 1; c < n_chans; ++c)
      if (!(freqs_hz[c] > freqs_hz[c - 1])) return fail(AIDG_E_INVALID, "frequencies must be strictly increasing");
    ShapeEstimate se;
    estimate_shape(g, n_baselines, n_times, n_chans, uvw_m, freqs_hz, &se);
    const int64_t elem = g.precision == AIDG_FP32 ? 8 : 16;
    const int64_t L = g.L, N = g.N;
    const int64_t n_vis = (int64_t)n_baselines * n_times * n_chans;
    const int64_t n_int = n_times ? (n_times + g.aterm_interval - 1) / g.aterm_interval : 0;
    const int64_t n_sg = se.n_subgrids;
    out->n_wlayers = (int32_t)(se.jmax - se.jmin + 1);
    out->n_pol = g.npol;
    out->w_step = g.w_step > 0 ? g.w_step : 0.0;
    out->n_subgrids = n_sg;
    out->n_groups = se.n_groups;
    out->n_excluded = se.n_excluded;
    out->grid_bytes = (int64_t)out->n_wlayers * g.npol * N * N * elem;
    out->vis_bytes = n_vis * 4 * elem;
    out->aterm_bytes = n_int * n_stations * L * L * 4 * elem * (g.amode ? 2 : 1);
    // what aidg_plan_create allocates, each allocation at least 256 bytes
    auto al = [](int64_t b) { return std::max<int64_t>(b, 256); };
    const int64_t per_image = 4 * L * L * elem;
    const int64_t parts = estimate_parts(g, se);
    int64_t batch = std::max<int64_t>(1, std::min<int64_t>(g.workspace / per_image, 65535));
    batch = std::min(batch, std::max<int64_t>(1, se.n_groups + (se.n_groups + parts <= batch ? parts : 0)));
    int64_t b = al(n_sg * (int64_t)sizeof(SubgridDev)) + al((int64_t)n_baselines * n_times * 24 * (g.fold ? 2 : 1)) +
                al((int64_t)n_chans * 8) + out->aterm_bytes + al((int64_t)TableLayout(g.L, (size_t)elem).bytes) +
                al(se.n_excluded * 8) + al((n_sg + 1) * 8 * (parts ? 2 : 1)) + al(batch * per_image) + al(sizeof(KernelArgs));
    if (N <= kMaxImageN) b += al(N * elem) + al(N * 8);
    if (g.amode) {
      const int64_t pairs = std::min<int64_t>(n_sg, (int64_t)n_int * n_baselines);
      // the normalisation map's partial sums: one chunk per about 64 pairs, at most 64
      const int64_t chunks = std::max<int64_t>(1, std::min<int64_t>(64, (pairs + 63) / 64));
      b += al(pairs * 8) + al(pairs * 8) + al(chunks * L * L * 8) + al(L * L * 8);
    }
    out->plan_bytes = b;
    return AIDG_OK;
  } catch (const std::bad_alloc&) {
    return fail(AIDG_E_NOMEM, "host allocation failed");
  }
}

aidg_status aidg_image_workspace_bytes(const aidg_plan* plan, int64_t* bytes) {
  if (!plan || !bytes) return fail(AIDG_E_INVALID, "NULL plan or output");
  if (!plan->img_ok)
    return fail(AIDG_E_UNSUPPORTED, "image-level transforms need N = 2^a 3^b 5^c <= 8192 with a row of N "
                                    "complex values within 64 KB");
  *bytes = 2 * (int64_t)plan->g.N * plan->g.N * (int64_t)plan->elem;
  return AIDG_OK;
}

aidg_status aidg_invert(aidg_plan* plan, const void* grid, void* image, void* workspace,
                        int64_t workspace_bytes, void* hip_stream) {
  aidg_status r = image_args(plan, grid, image, workspace, workspace_bytes);
  if (r != AIDG_OK) return r;
  BusyGuard guard(plan);
  if (!guard.ok) return fail(AIDG_E_BUSY, "plan in use by another thread");
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  hipError_t e = hipStreamWaitEvent(st, plan->last, 0);
  if (e != hipSuccess) return hip_fail(e, "hipStreamWaitEvent");
  const int N = plan->g.N, prec = plan->g.precision;
  const size_t plane = (size_t)N * N * plan->elem;
  const double dl = plan->g.dl, inv_l2 = 1.0 / ((double)plan->g.L * plan->g.L);
  for (int pol = 0; pol < plan->g.npol && r == AIDG_OK; pol += 2) {  // the workspace holds two planes
    const int n = std::min(2, plan->g.npol - pol);
    char* img = static_cast<char*>(image) + pol * plane;
    for (int w = 0; w < plan->W && r == AIDG_OK; ++w) {
      const char* G = static_cast<const char*>(grid) + ((size_t)w * plan->g.npol + pol) * plane;
      // rows G[gv][gu] -> A[X][gv]; its rows into img[Y][X].  Or rows -> A[gv][X]; columns, in
      // place, then into img[Y][X]
      auto pass = [&](KernelClass k, ImagePass what, const void* in, void* out) {
        if (r != AIDG_OK) return;
        r = image_step(plan, st, k, [&] {
          return launch_image_pass(prec, what, in, out, n, N, plan->img_fr, plan->d_img_tw, plan->d_img_itaper, dl,
                                   plan->w0[w], inv_l2, w == 0, w == plan->W - 1 ? plan->d_nmap : nullptr, plan->g.L,
                                   st);
        });
      };
      pass(kImageFft, kInvertRows, G, workspace);
      if (!image_strips(N)) pass(kImageFft, kInvertColumns, workspace, workspace);
      pass(kImageWstack, kInvertStack, workspace, img);
    }
  }
  if (r != AIDG_OK) return r;
  e = hipEventRecord(plan->last, st);
  return e == hipSuccess ? AIDG_OK : hip_fail(e, "hipEventRecord");
}

aidg_status aidg_predict(aidg_plan* plan, const void* image, void* grid, void* workspace,
                         int64_t workspace_bytes, void* hip_stream) {
  aidg_status r = image_args(plan, image, grid, workspace, workspace_bytes);
  if (r != AIDG_OK) return r;
  BusyGuard guard(plan);
  if (!guard.ok) return fail(AIDG_E_BUSY, "plan in use by another thread");
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
  hipError_t e = hipStreamWaitEvent(st, plan->last, 0);
  if (e != hipSuccess) return hip_fail(e, "hipStreamWaitEvent");
  const int N = plan->g.N, prec = plan->g.precision;
  const size_t plane = (size_t)N * N * plan->elem;
  const double dl = plan->g.dl, inv_l2 = 1.0 / ((double)plan->g.L * plan->g.L);
  for (int w = 0; w < plan->W && r == AIDG_OK; ++w) {
    for (int pol = 0; pol < plan->g.npol && r == AIDG_OK; pol += 2) {  // the workspace holds two planes
      const int n = std::min(2, plan->g.npol - pol);
      const char* img = static_cast<const char*>(image) + pol * plane;
      char* G = static_cast<char*>(grid) + ((size_t)w * plan->g.npol + pol) * plane;
      // rows of img[Y][X] times the w-term -> A[gu][Y]; its rows -> G[gv][gu].  Or rows ->
      // A[Y][gu]; columns, in place, then -> G[gv][gu]
      auto pass = [&](ImagePass what, const void* in, void* out) {
        if (r != AIDG_OK) return;
        r = image_step(plan, st, kImageFft, [&] {
          return launch_image_pass(prec, what, in, out, n, N, plan->img_fr, plan->d_img_tw, plan->d_img_itaper, dl,
                                   plan->w0[w], inv_l2, 1, nullptr, plan->g.L, st);
        });
      };
      pass(kPredictRows, img, workspace);
      if (!image_strips(N)) pass(kPredictColumns, workspace, workspace);
      pass(kPredictGrid, workspace, G);
    }
  }
  if (r != AIDG_OK) return r;
  e = hipEventRecord(plan->last, st);
  return e == hipSuccess ? AIDG_OK : hip_fail(e, "hipEventRecord");
}

aidg_status aidg_plan_set_profiling(aidg_plan* plan, int32_t enable) {
  if (!plan) return fail(AIDG_E_INVALID, "NULL plan");
  BusyGuard guard(plan);
  if (!guard.ok) return fail(AIDG_E_BUSY, "plan in use by another thread");
  if (enable && plan->pool.empty()) {
    const size_t n = 2 * 4096;
    plan->pool.reserve(n);
    for (size_t i = 0; i < n; ++i) {
      hipEvent_t e;
      const hipError_t err = hipEventCreate(&e);
      if (err != hipSuccess) return hip_fail(err, "hipEventCreate");
      plan->pool.push_back(e);
    }
  }
  plan->profiling = enable != 0;
  return AIDG_OK;
}

aidg_status aidg_plan_kernel_times(aidg_plan* plan, aidg_kernel_times* out) {
  if (!plan || !out) return fail(AIDG_E_INVALID, "NULL plan or output");
  BusyGuard guard(plan);
  if (!guard.ok) return fail(AIDG_E_BUSY, "plan in use by another thread");
  std::memset(out, 0, sizeof(*out));
  for (const auto& t : plan->timed) {
    hipError_t e = hipEventSynchronize(t.b);
    float ms = 0.0f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, t.a, t.b);
    if (e != hipSuccess) return hip_fail(e, "reading kernel timers");
    out->ms[t.kind] += ms;
    out->launches[t.kind] += 1;
    out->vis_pixels[t.kind] += t.vp;
    out->subgrids[t.kind] += t.nsg;
  }
  plan->timed.clear();
  plan->pool_next = 0;
  return AIDG_OK;
}

aidg_status aidg_executor_create(int64_t workspace_bytes, aidg_executor** out) {
  if (!out || workspace_bytes < 0) return fail(AIDG_E_INVALID, "NULL output or negative size");
  *out = nullptr;
  aidg_executor* ex = new (std::nothrow) aidg_executor();
  if (!ex) return fail(AIDG_E_NOMEM, "host allocation failed");
  ex->bytes = workspace_bytes ? workspace_bytes : kWorkspaceDefault;
  hipError_t e = hipGetDevice(&ex->device);
  if (e == hipSuccess) e = hipMalloc(&ex->d_scratch, (size_t)ex->bytes);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&ex->last, hipEventDisableTiming);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    if (ex->d_scratch) (void)hipFree(ex->d_scratch);
    delete ex;
    return fail(e == hipErrorOutOfMemory ? AIDG_E_NOMEM : AIDG_E_DEVICE,
                std::string("executor workspace: ") + hipGetErrorString(e));
  }
  *out = ex;
  return AIDG_OK;
}

aidg_status aidg_execute(aidg_executor* ex, const aidg_work* items, int32_t n_items, void* hip_stream) {
  if (!ex) return fail(AIDG_E_INVALID, "NULL executor");
  bool expected = false;
  if (!ex->busy.compare_exchange_strong(expected, true)) return fail(AIDG_E_BUSY, "executor in use");
  const aidg_status r = execute_items(ex->d_scratch, ex->bytes, ex->last, items, n_items, hip_stream);
  ex->busy.store(false);
  return r;
}

aidg_status aidg_execute_static(const aidg_work* items, int32_t n_items, int64_t workspace_bytes,
                                void* hip_stream) {
  if (workspace_bytes < 0 || workspace_bytes > kStaticWorkspaceBytes)
    return fail(AIDG_E_INVALID, "workspace_bytes " + std::to_string(workspace_bytes) +
                                    " outside 0.." + std::to_string(kStaticWorkspaceBytes) +
                                    " (the static workspace's size, AIDG_STATIC_WORKSPACE_BYTES)");
  if ((n_items > 0 && !items) || n_items < 0) return fail(AIDG_E_INVALID, "bad items");
  if (n_items == 0) return AIDG_OK;
  int device = 0;
  const hipError_t e = hipGetDevice(&device);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  std::string err;
  void* ws = static_workspace(device, &err);
  if (!ws) return fail(AIDG_E_DEVICE, err);
  return execute_items(ws, workspace_bytes ? workspace_bytes : kStaticWorkspaceBytes, nullptr, items, n_items,
                       hip_stream);
}

void aidg_executor_destroy(aidg_executor* ex) {
  if (!ex) return;
  if (ex->last) {
    (void)hipEventSynchronize(ex->last);
    (void)hipEventDestroy(ex->last);
  }
  if (ex->d_scratch) (void)hipFree(ex->d_scratch);
  delete ex;
}

void aidg_plan_destroy(aidg_plan* plan) {
  if (!plan) return;
  if (plan->last) (void)hipEventSynchronize(plan->last);
  plan->release();
  delete plan;
}

}  // extern "C"
