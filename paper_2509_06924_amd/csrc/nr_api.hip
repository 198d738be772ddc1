// C ABI of the reflectivity log-likelihood library: argument validation, plan
// construction (work list, record offsets, quadrature rule) and launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "nr.h"
#include "nr_internal.hpp"

using namespace nr;

namespace {

thread_local std::string g_last_hip_error;

nr_status hip_fail(hipError_t e, const char* what) {
  g_last_hip_error = std::string(what) + ": " + hipGetErrorString(e);
  return NR_EHIP;
}

// Workspace of nr_loglik_grad_noalloc: a file-scope device array, one copy
// per GPU, held until the process ends.  Host code must not pass the array's
// name to a kernel or a copy (on the host it is only a stand-in symbol): the
// device address of each GPU's copy is looked up once, with that GPU
// current, and kept in scratch_addr.  Every call on one GPU shares its copy.
__device__ __align__(256) unsigned char scratch[NR_NOALLOC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_addr[kMaxDevices] = {};

// The device address of `dev`'s scratch copy (dev must be current).
nr_status scratch_addr(int dev, void** out) {
  if (dev < 0 || dev >= kMaxDevices) return NR_EINVAL;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_addr[dev]) {
    void* ptr = nullptr;
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr) return hip_fail(e, "scratch symbol address");
    g_scratch_addr[dev] = ptr;
  }
  *out = g_scratch_addr[dev];
  return NR_OK;
}

// 17-point Gauss-Legendre rule on [-1, 1]: Newton iteration on P_17 from
// Tricomi's asymptotic initial guesses, in long double, weights
// 2 / ((1 - x^2) P'_17(x)^2).  Nodes ascending; the centre node is exactly 0.
void legendre_rule(int n, double* x_out, double* u_out) {
  const long double pi = 3.141592653589793238462643383279502884L;
  for (int k = 1; k <= n; ++k) {
    const long double th = pi * (4.0L * k - 1.0L) / (4.0L * n + 2.0L);
    long double x = (1.0L - (n - 1.0L) / (8.0L * n * n * n)) * std::cos(th);
    long double dp = 0.0L;
    for (int it = 0; it < 60; ++it) {
      long double pm1 = 1.0L, p = x;
      for (int m = 2; m <= n; ++m) {
        const long double pn = ((2.0L * m - 1.0L) * x * p - (m - 1.0L) * pm1) / m;
        pm1 = p;
        p = pn;
      }
      dp = n * (pm1 - x * p) / (1.0L - x * x);
      const long double step = p / dp;
      x -= step;
      if (std::fabs(step) <= 1e-32L) break;
    }
    {
      long double pm1 = 1.0L, p = x;
      for (int m = 2; m <= n; ++m) {
        const long double pn = ((2.0L * m - 1.0L) * x * p - (m - 1.0L) * pm1) / m;
        pm1 = p;
        p = pn;
      }
      dp = n * (pm1 - x * p) / (1.0L - x * x);
    }
    // k = 1 is the largest root
    x_out[n - k] = (double)x;
    u_out[n - k] = (double)(2.0L / ((1.0L - x * x) * dp * dp));
  }
  if (n % 2) x_out[n / 2] = 0.0;
}

// Normalised Gaussian smearing weights over nodes 3.5 x_k (units of sigma_Q).
void smearing_rule(double* t, double* w) {
  double x[kSmearNodes], u[kSmearNodes];
  legendre_rule(kSmearNodes, x, u);
  long double g[kSmearNodes], total = 0.0L;
  for (int k = 0; k < kSmearNodes; ++k) {
    t[k] = 3.5 * x[k];
    const long double tk = t[k];
    g[k] = (long double)u[k] * std::exp(-tk * tk / 2.0L);
    total += g[k];
  }
  for (int k = 0; k < kSmearNodes; ++k) w[k] = (double)(g[k] / total);
}

// Tables for the device exp and sincos, correctly rounded from long double:
// (sin, cos)(k pi/64) for k = 0..127, interleaved, then 2^(j/64) for j = 0..63.
void append_math_tables(std::vector<double>& v) {
  const long double pi = 3.141592653589793238462643383279502884L;
  for (int k = 0; k < 128; ++k) {
    v.push_back((double)std::sin(pi * k / 64.0L));
    v.push_back((double)std::cos(pi * k / 64.0L));
  }
  for (int j = 0; j < 64; ++j) v.push_back((double)std::exp2((long double)j / 64.0L));
}

// One kernel launch: a work list for one layer-count bucket.  Full units
// cover 64 consecutive points of one item; tail units pack the trailing
// partial groups of several items of equal depth, lane by lane.
struct Launch {
  int bucket = 0;
  int form = kFormRecompute;  // gradient: the kernel form (resolution calls take their own)
  bool tail = false;
  bool split = false;  // split tail units (one item's partial group, lanes over node groups)
  bool one[2] = {};    // split units whose one node is counted per lane: plain, resolution
  int scan_ch = 0;     // deep lists: the largest levels-per-lane of its items at 64 lanes
  int side = 0;        // 0: the caller's stream, k: the plan's side stream k - 1
  double est = 0.0;    // gradient: estimated time, us (see launch_estimate)
  int n_wu = 0;
  int32_t* item = nullptr;      // [n_wu]: the unit's item (first item for tails)
  int32_t* split_code = nullptr;  // [n_wu] split units: points | node groups << 16
  int32_t* p0 = nullptr;        // [n_wu]: first point (full units)
  int64_t* rec = nullptr;       // [n_wu]: record offset (full units)
  int32_t* lane_item = nullptr; // [n_wu * 64] (tail units)
  int32_t* lane_pt = nullptr;   // [n_wu * 64]
  int64_t* lane_rec = nullptr;  // [n_wu * 64], -1 for idle lanes
};

// Per-item lists of record offsets summed by the reduction kernels.
struct RecordLists {
  int64_t* first = nullptr;
  int32_t* count = nullptr;
  int64_t* offs = nullptr;
};

// Workgroups are dispatched to the 8 XCDs round-robin (block b -> XCD b % 8)
// and each XCD has its own L2.  Block b takes entry xcd_order(b, n, run) of
// the cost-sorted unit list: within each chunk of 8 x run blocks, one XCD
// gets a run of `run` consecutive entries, while the chunks keep the
// longest-first order: where equal costs leave the units of one item together
// (see make_full), its layer records are fetched into one L2.  The last partial
// chunk maps to itself.
constexpr int kXcds = 8;
size_t xcd_order(size_t b, size_t n, size_t run) {
  const size_t chunk = kXcds * run;
  const size_t c0 = (b / chunk) * chunk;
  if (c0 + chunk > n) return b;
  const size_t r = b - c0;
  return c0 + (r % kXcds) * run + r / kXcds;
}

// The order of units by `key`, ascending, equal keys as they are: counting passes
// over the keys' bytes, without those that all keys share.  Comparing the units of
// 4096 draws (57 000 in two lists of seven costs and places) took 0.4 ms of a plan's
// 1.65, those of 16384 ragged items 10 of 16 ms.
std::vector<uint32_t> order_by(const std::vector<uint64_t>& key) {
  const size_t n = key.size();
  std::vector<uint32_t> idx(n), next(n);
  uint32_t count[8][256] = {};
  for (size_t i = 0; i < n; ++i) {
    idx[i] = (uint32_t)i;
    for (int b = 0; b < 8; ++b) ++count[b][key[i] >> (8 * b) & 0xff];
  }
  for (int b = 0; b < 8 && n > 0; ++b) {
    if (count[b][key[0] >> (8 * b) & 0xff] == n) continue;
    uint32_t at = 0;
    for (uint32_t& c : count[b]) {
      const uint32_t here = c;
      c = at;
      at += here;
    }
    for (const uint32_t i : idx) next[count[b][key[i] >> (8 * b) & 0xff]++] = i;
    idx.swap(next);
  }
  return idx;
}

// Device copies of host arrays, in one allocation and one copy: a plan has dozens of
// small ones, at some 15 us each (64 items of 400 points 626 us a plan one by one, 295
// so; 400 ragged items 1535 / 609).
template <class T>
struct Part {
  T** dst;  // null for an empty array
  const std::vector<T>& src;
  size_t bytes() const { return (src.size() * sizeof(T) + 255) / 256 * 256; }
  void stage(unsigned char* host, unsigned char* device, size_t& at) const {
    if (src.empty()) return;
    std::memcpy(host + at, src.data(), src.size() * sizeof(T));
    *dst = reinterpret_cast<T*>(device + at);
    at += bytes();
  }
};
template <class T>
Part<T> part(T** dst, const std::vector<T>& src) {
  *dst = nullptr;
  return {dst, src};
}
template <class... T>
hipError_t upload(std::vector<void*>& owned, Part<T>... parts) {
  const size_t total = (parts.bytes() + ...);
  if (total == 0) return hipSuccess;
  void* device = nullptr;
  const hipError_t e = hipMalloc(&device, total);
  if (e != hipSuccess) return e;
  owned.push_back(device);
  std::vector<unsigned char> host(total);
  size_t at = 0;
  (parts.stage(host.data(), static_cast<unsigned char*>(device), at), ...);
  return hipMemcpy(device, host.data(), total, hipMemcpyHostToDevice);
}

// Streams beside the caller's for the gradient's launches (four in all, the
// hardware queues of a process).
constexpr int kSideStreams = 3;

// The side streams of eager calls, one set per device, counted by the device's
// plans and given back with the last of them.  A set per plan would put the
// streams of several plans on one hardware queue, a plan's side stream on its
// caller's (three live plans of 2048 ragged items in FP32: 3.1 -> 3.5 ms).
// A set that another caller's stream may still be working on is left to it, and
// the call keeps to its own stream: calls on two streams never wait for each
// other's side work (40 small items issued beside 2048 ragged ones: FP32 3.8 ms
// behind the larger plan's join, 3.0 on their own stream; FP64 5.6 / 3.4).  The
// price is overlap where two callers do run at once (two plans of 2048 ragged
// items on two streams: FP32 3.3 -> 4.0 ms a call).  The mutex keeps each fork ... join sequence whole.
// A call under graph capture takes streams of its plan instead: a stream being
// captured must not see other threads' work.
struct ForkJoin {
  hipStream_t st[kSideStreams] = {};
  hipEvent_t fork = nullptr, join[kSideStreams] = {};
};

void fork_join_free(ForkJoin& f) {
  for (hipStream_t s : f.st)
    if (s) (void)hipStreamDestroy(s);
  for (hipEvent_t e : f.join)
    if (e) (void)hipEventDestroy(e);
  if (f.fork) (void)hipEventDestroy(f.fork);
  f = ForkJoin();
}

// Makes what is missing of the first n streams and their events.
hipError_t fork_join_make(ForkJoin& f, int n) {
  hipError_t e = hipSuccess;
  if (!f.fork) e = hipEventCreateWithFlags(&f.fork, hipEventDisableTiming);
  for (int k = 0; k < n && e == hipSuccess; ++k) {
    if (!f.st[k]) e = hipStreamCreateWithFlags(&f.st[k], hipStreamNonBlocking);
    if (!f.join[k] && e == hipSuccess)
      e = hipEventCreateWithFlags(&f.join[k], hipEventDisableTiming);
  }
  return e;
}

// For calls that another thread's capture in global mode would refuse.
struct RelaxedCapture {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

struct SidePool {
  std::mutex mu;
  int users = 0;
  ForkJoin set;
  hipStream_t caller = nullptr;  // of the last call that forked
  int used = 0;                  // streams that it took
};
SidePool g_side_pool[kMaxDevices];

// (All its streams are made together: one made later, after others of the process,
// would share a hardware queue with one of them, and 6 to 20 ragged items would take
// 1.2-1.5 times as long.)
hipError_t side_pool_acquire(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  SidePool& pool = g_side_pool[device];
  std::lock_guard<std::mutex> lock(pool.mu);
  const hipError_t e = fork_join_make(pool.set, kSideStreams);
  if (e == hipSuccess)
    ++pool.users;
  else if (pool.users == 0)
    fork_join_free(pool.set);
  return e;
}
void side_pool_release(int device) {
  SidePool& pool = g_side_pool[device];
  std::lock_guard<std::mutex> lock(pool.mu);
  if (--pool.users > 0) return;
  fork_join_free(pool.set);
  pool.used = 0;
}
// Whether a call on st may fork: the last one that did was on st too (its join
// comes before anything new there), or has ended.  Under pool.mu.
bool side_pool_free(const SidePool& pool, hipStream_t st) {
  if (pool.used == 0 || (st == pool.caller && st != hipStreamPerThread)) return true;
  RelaxedCapture relaxed;
  for (int k = 0; k < pool.used; ++k)
    if (hipEventQuery(pool.set.join[k]) != hipSuccess) {
      // (not this call's error: the launches ask for the last one)
      if (hipPeekAtLastError() == hipErrorNotReady) (void)hipGetLastError();
      return false;
    }
  return true;
}

// The launches of a gradient call and the records they write.
struct GradSchedule {
  std::vector<Launch> launches;
  RecordLists lists;
  int64_t records = 0;  // doubles
  int n_side = 0;       // streams beside the caller's
};

}  // namespace

struct nr_plan {
  int device = 0;
  int32_t n_datasets = 0, n_items = 0, precision = NR_F64;
  nr_plan_options opts;
  int bucket_form[kNumBuckets];  // GradForm of the plain gradient
  bool grad_scaled = false;      // a gradient launch takes the select form
  bool scan_select = false;      // the deep items' launches do
  bool value_forms = false;      // the value kernels take both node forms (FP64)
  std::vector<int64_t> q_off, row_off, out_off;
  std::vector<int32_t> dataset_of_item;
  std::vector<double> dqq;
  int64_t rec_ll_total = 0;
  // device copies
  int32_t* d_dataset_of_item = nullptr;
  int64_t* d_q_off = nullptr;
  int64_t* d_row_off = nullptr;
  double* d_dqq = nullptr;
  int64_t* d_out_off = nullptr;
  RecordLists lists_ll;
  double* d_rule = nullptr;
  hipEvent_t ev_start = nullptr, ev_stop = nullptr;
  std::vector<Launch> launches_fwd;
  // grad_res: of calls with the resolution derivative, where they have their own
  GradSchedule grad, grad_res;
  bool res_own = false;
  const GradSchedule& schedule(bool res) const { return res && res_own ? grad_res : grad; }
  uint8_t* d_row_kind = nullptr;  // 0 fronting, 1 layer, 2 backing, per row
  int uniform_rows = 0;           // rows per item if all items agree, else 0
  int max_rows = 2;               // rows of the deepest item
  double node_t[kSmearNodes], node_w[kSmearNodes];
  std::vector<void*> owned;
  // streams beside the caller's for the gradient's launches (side_stream)
  bool pooled = false;        // holds a use of the device's SidePool
  mutable ForkJoin cap;       // calls under graph capture; made by the first
  mutable std::mutex cap_mu;  // one captured fork ... join sequence at a time
};

namespace {

void plan_free(nr_plan* p) {
  for (void* ptr : p->owned)
    if (ptr) (void)hipFree(ptr);
  p->owned.clear();
  fork_join_free(p->cap);
  if (p->pooled) side_pool_release(p->device);
  p->pooled = false;
}

nr_status validate_desc(const nr_batch_desc* d) {
  if (!d) return NR_EINVAL;
  if (d->n_datasets < 0 || d->n_items < 0) return NR_EINVAL;
  if (d->precision != NR_F64 && d->precision != NR_F32) return NR_EINVAL;
  if (!d->q_off || !d->row_off) return NR_EINVAL;
  if (d->n_datasets > 0 && !d->dq_over_q) return NR_EINVAL;
  if (d->n_items > 0 && !d->dataset_of_item) return NR_EINVAL;
  if (d->q_off[0] != 0 || d->row_off[0] != 0) return NR_EINVAL;
  for (int s = 0; s < d->n_datasets; ++s) {
    if (d->q_off[s + 1] < d->q_off[s]) return NR_EINVAL;
    if (d->q_off[s + 1] - d->q_off[s] > (int64_t)INT32_MAX) return NR_EINVAL;
    const double r = d->dq_over_q[s];
    if (!(r >= 0.0) || !std::isfinite(r)) return NR_EINVAL;
  }
  for (int b = 0; b < d->n_items; ++b) {
    const int64_t rows = d->row_off[b + 1] - d->row_off[b];
    if (rows < 2 || rows > NR_MAX_DEEP_LAYERS + 2) return NR_EINVAL;
    const int32_t s = d->dataset_of_item[b];
    if (s < 0 || s >= d->n_datasets) return NR_EINVAL;
  }
  return NR_OK;
}

nr_status check_call(const nr_plan* p, const nr_values* v, bool need_data) {
  if (!p || !v) return NR_EINVAL;
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != p->device) return NR_EINVAL;
  if (p->n_items == 0) return NR_OK;
  if (!v->layers || !v->scale || !v->bkg) return NR_EINVAL;
  if (p->q_off.back() > 0) {
    if (!v->q) return NR_EINVAL;
    if (need_data && (!v->r_obs || !v->r_err)) return NR_EINVAL;
  }
  return NR_OK;
}

KernelArgs base_args(const nr_plan* p, const nr_values* v) {
  KernelArgs a;
  std::memset(&a, 0, sizeof(a));
  a.dataset_of_item = p->d_dataset_of_item;
  a.q_off = p->d_q_off;
  a.row_off = p->d_row_off;
  a.dq_over_q = p->d_dqq;
  a.out_off = p->d_out_off;
  a.q = v->q;
  a.r_obs = v->r_obs;
  a.r_err = v->r_err;
  a.layers = v->layers;
  a.scale = v->scale;
  a.bkg = v->bkg;
  a.item_status = v->item_status;
  a.dq = v->dq;
  a.dqq_item = v->dqq_item;
  a.rule = p->d_rule;
  return a;
}

// Workspace layout: per-row layer records (6 doubles per row of every item),
// their float copies (8 floats per row), then the per-work-unit partial
// records of the operation.
size_t consts_doubles(const nr_plan* p) {
  return (size_t)p->row_off.back() * (kRecDoubles + kRecFloats / 2);
}
const float* consts_floats(const nr_plan* p, const double* ws) {
  return reinterpret_cast<const float*>(ws + (size_t)p->row_off.back() * kRecDoubles);
}

size_t op_doubles(const nr_plan* p, int op) {
  size_t n = consts_doubles(p);
  if (op == NR_OP_LOGLIK) n += (size_t)p->rec_ll_total;
  if (op == NR_OP_LOGLIK_GRAD) n += (size_t)std::max(p->grad.records, p->grad_res.records);
  return n;
}

// What a gradient launch costs, in us.  A wave runs its nodes and an epilogue (one
// reduction per record field) worth `e` nodes more, `us` per level each; w waves per
// SIMD take f(w) times a wave's share of a full SIMD.  A SIMD with one wave more than
// the others holds up the launch, so f goes in steps: s1 up to one wave (nothing
// hides its latencies), 2 up to two, s3 up to three, then `slope` for each.  Fits of
// calls of uniform items (MI355X, 0.5 to 8 units per SIMD in 1, 2, 3, 4, 6, 9 and 17 node
// groups at every bucket's depth; us a call = 9 + the launch), to 4 % in the mean and
// 10-20 % at worst: 10 layers FP64 at 1.98 / 2.30 / 2.98 / 3.40 / 5.98 units per SIMD 209
// / 285 / 304 / 371 / 610 whole, 120 / 166 / 173 / 210 / 338 in two groups; 36 layers
// whole at 0.98 / 1.20 / 1.98 / 2.30 519 / 852 / 963 / 1324.
struct LaunchCost {
  double us, e;             // per level and node; the epilogue in nodes
  double s1, s3, slope;     // f(w)
  double step(double w) const {
    const double c = std::ceil(w);
    return c <= 1.0 ? s1 : (c <= 2.0 ? 2.0 : s3 + (c - 3.0) * slope) - 0.1 * (c - w);
  }
};
LaunchCost launch_cost(int precision, int lmax, bool res, bool split) {
  const bool f64 = precision == NR_F64;
  const double n = lmax + 1;
  if (grad_waves_per_simd(precision, lmax) == 1)
    return f64 ? LaunchCost{(0.51 + 0.0065 * (lmax - 16)) * (res ? 1.1 : 1.0), res ? 1.25 : 1.55,
                            1.05, 3.0, 0.97}
               : LaunchCost{0.40, res ? 1.85 : 2.1, 0.98, 2.97, 0.96};
  if (f64) {
    // (the whole resolution kernels spill less than the split ones: 0.8 of the time
    // at 14 layers)
    const double whole = split       ? 1.0
                         : lmax <= 2 ? 1.04
                         : res       ? 1.0 - 0.024 * std::max(0, lmax - 6)
                                     : 1.0;
    return {(0.35 + 0.012 * lmax) * (res ? 1.25 : 1.0) * whole, res ? 0.6 + 5.0 / n : 0.85 + 6.5 / n,
            split ? 1.38 : 1.25, lmax <= 2 ? 2.72 : 2.97,
            lmax <= 2 ? 0.8 : split ? 0.86 : res ? 0.93 : 1.0};
  }
  // (16 layers: the split resolution kernel has the SIMD to itself)
  if (res && split && lmax == 16) return {0.38, 2.1, 0.95, 2.98, 0.96};
  const double whole =
      split ? 1.0 : lmax <= 2 ? 1.14 : lmax <= 6 ? 1.1 : lmax <= 20 ? 1.04 : lmax <= 24 ? 0.93 : 0.85;
  return {(0.19 + 0.006 * lmax) * (res && lmax <= 6 ? 1.3 : 1.0) * whole,
          std::min(6.0, std::max(2.0, res ? 0.7 + 12.0 / n : 1.0 + 15.0 / n)),
          split ? 1.42 : 1.34, lmax <= 4 || (lmax == 10 && !res && !split) ? 2.65 : 3.05,
          lmax <= 4 ? 0.73 : 0.86};
}
double launch_estimate(int precision, int lmax, bool split, int64_t waves, double nodes,
                       int64_t simds) {
  const LaunchCost c = launch_cost(precision, lmax, false, split);
  return c.us * (lmax + 1) * (nodes + c.e) * c.step((double)waves / (double)simds);
}

// Whether a gradient launch of one node per lane counts it per lane.  A wave alone
// on its SIMD that runs one node waits for each scalar load of a record it has
// not read yet; the vector loads of a per-lane counter run ahead.  Up to a
// quarter of the SIMDs busy that is the faster one at every depth (us a call per
// wave / per lane, one item of 200 points: 16 layers FP32 30.0 / 27.7, 20 layers 35.7
// / 32.6, 40 layers with resolution 61.5 / 57.4, FP64 79.6 / 77.0; FP32 at 6 layers
// 20.6 / 21.0).  With more waves the scalar loads win in resolution calls (10 items of
// 184 points, 40 layers FP64 93 / 112) and at 14 and 18 layers in FP32 (1.5-3 %), the
// vector loads in the rest: 45 items of 48 points, 16 layers FP32 29.6 / 27.5, 20
// layers 36.8 / 35.5.
bool lane_counter_pays(int precision, int lmax, bool res, int64_t waves, int64_t simds) {
  const bool few = 4 * waves <= simds;
  if (precision == NR_F64) return few || (lmax >= 24 && !res);
  return (few && lmax != 6) || (lmax >= 16 && lmax != 18 && (!res || lmax <= 28));
}

// How a small plan's gradient units are made: node groups per point (1: whole groups
// of 64 points, then tails), and whether the tails of several items share waves.
struct UnitPlan {
  int groups = 1;
  bool pack = false;
  bool operator==(const UnitPlan& o) const { return groups == o.groups && pack == o.pack; }
};

// The units of a small plan whose launches (one per depth bucket, on up to
// 1 + kSideStreams streams) take the least estimated time: [0] plain calls, [1] calls with
// the resolution derivative, the same unless others are 1 % faster.  Units of 400 points,
// 10 layers, us a call at G = 1 / 2 / 3 / 6 / 9 / 17: 112 units 141 / 80 / 62 / 42 / 38 / 51; 672: 146 / 120 / 92 / 94 / 104 / 153; 1344: 212 / 170 / 156 / 166 / 176 /
// 278; 2688: 309 / 268 / 283 / 298 / 328 / 537; 4480: 430 / 445 / 446 / 479 / 535 / 878.
// G = 2048 / units, the rule before, took 53, 92, 211, 309 and 429 us there.  Many short
// items gain from the lanes that groups fill: 2355 of 40 points, 10 layers FP64 with
// resolution 315 us whole, 221 split.
// Tails in waves of their own displace whole units: where the two do not fit the rounds
// that the whole units take, the last of these end as much later as a tail takes (438
// items of 400 points, 36 layers FP32, 2.57 + 0.43 units per SIMD: 966 us, 887 packed;
// 250 items, 1.46 + 0.24: 613, 647).  Launches of other depths cover it, over many rounds
// it does not show (3584 items of 130 to 168 points: 0.93-1.02 of the packed time at nearly
// every depth), and packed units that spill or have a SIMD's other wave to themselves
// give it back, so packing is tried at one wave per SIMD in one-form kernels alone (FP32
// 32-40 layers, FP64 40: 300 items of 400 points 1306 us, 1170 packed).
// Launches of several depths overlap, but not fully: a stream's share of them one after
// the other plus 0.7 of the time that all would take on a full device.  kReduceUs: the
// reduction adds an item's records one by one (in plans of one depth it is hidden in
// the 9 us).
// Over 420 plans of one depth (24 to 900 points, 0.3 to 6 units per SIMD, both precisions)
// the choice is 1.4 % over the best of the eight in the mean, plain, and 1.1 % with
// resolution; 5 % or more in one of ten, 28 % at worst.  Over 88 ragged ones (10 to 600
// items of 100 to 1000 points) 1.6 and 2.0 %, 21 % at worst: 400 of 2 to 40 layers FP64
// 1816 us whole, 1293 / 1306 / 1431 / 1610 in 2 / 3 / 4 / 9 groups.
// More groups write more records.  A plan that the fixed scratch of
// nr_loglik_grad_noalloc held with that rule's records is not pushed over it.
constexpr int kSmallPlanWaves = 6;  // units per SIMD: from here on the plan is not split
constexpr double kReduceUs = 0.08;
std::array<UnitPlan, 2> pick_units(const nr_plan* p, int64_t units, int64_t simds) {
  const int G_fit = (int)std::max<int64_t>(1, std::min<int64_t>(kSmearNodes, 2 * simds / units));
  // per bucket of the shallow items: units; apart from those, units of unsmeared items
  // (one node each) and, at G = 1, the smeared tails of 32 points or fewer, the nodes they
  // run in node groups, and their points per depth
  struct Count {
    int64_t waves = 0, flat = 0, tails = 0;
    int64_t all() const { return waves + flat + tails; }
    double tail_nodes = 0.0;
    std::map<int64_t, int64_t> tail_points;
  };
  Count of[kNumBuckets];
  int64_t most_records = 0;  // of an item
  auto count = [&](int G) {
    size_t doubles = consts_doubles(p);
    most_records = 0;
    for (Count& c : of) c = Count();
    for (int b = 0; b < p->n_items; ++b) {
      const int s = p->dataset_of_item[b];
      const int64_t rows = p->row_off[b + 1] - p->row_off[b];
      const int bk = bucket_of((int)rows - 2);
      const bool deep = bk == kDeepBucket;
      const int64_t nq = p->q_off[s + 1] - p->q_off[s];
      const int64_t npts = deep ? 1 : p->dqq[s] > 0.0 ? kWuPoints / G : kWuPoints;
      const int64_t n = (nq + npts - 1) / npts;
      doubles += (size_t)n * (4 + 4 * (size_t)rows);
      if (deep) continue;
      most_records = std::max(most_records, n);
      Count& c = of[bk];
      if (!(p->dqq[s] > 0.0)) {
        c.flat += n;
        continue;
      }
      const int tail = (int)(nq % kWuPoints);
      const bool part = G == 1 && tail > 0 && tail <= kWuPoints / 2;
      c.waves += part ? n - 1 : n;
      if (part) {
        const int groups = std::min(kWuPoints / tail, (int)kSmearNodes);
        ++c.tails;
        c.tail_nodes += (kSmearNodes + groups - 1) / groups;
        c.tail_points[rows] += tail;
      }
    }
    return sizeof(double) * doubles;
  };
  const size_t limit = std::max<size_t>(count(G_fit), NR_NOALLOC_SCRATCH_BYTES);
  // us, of the counts
  auto estimate = [&](UnitPlan u, bool res) {
    const int nodes = (kSmearNodes + u.groups - 1) / u.groups;
    int launches = 0;
    for (const Count& c : of) launches += c.all() > 0;
    double sum = 0.0, work = 0.0;  // launch by launch, and as one full device
    for (int k = 0; k < kNumBuckets; ++k) {
      const Count& n = of[k];
      if (n.all() == 0) continue;
      const int lmax = kBucketLmax[k];
      const LaunchCost c = launch_cost(p->precision, lmax, res, u.groups > 1);
      const LaunchCost ct = launch_cost(p->precision, lmax, res, true);
      const double wave = c.us * (lmax + 1) * (nodes + c.e);
      const double each =
          n.tails > 0 ? ct.us * (lmax + 1) * (n.tail_nodes / (double)n.tails + ct.e) : 0.0;
      const double w = (double)n.waves / (double)simds, wt = (double)n.tails / (double)simds;
      work += wave * c.slope * w + each * ct.slope * wt;
      if (n.flat > 0) {
        const double one = ct.us * (lmax + 1) * (1.0 + ct.e), wf = (double)n.flat / (double)simds;
        sum += one * ct.step(wf);
        work += one * ct.slope * wf;
      }
      if (u.pack) {
        int64_t packed = 0;
        for (const auto& d : n.tail_points) packed += (d.second + kWuPoints - 9) / (kWuPoints - 8);
        sum += 1.01 * wave * c.step(w + (double)packed / (double)simds);
        continue;
      }
      if (n.waves > 0) sum += wave * c.step(w);
      if (n.tails == 0) continue;
      if (launches > 1 || n.waves == 0)
        sum += each * ct.step(wt);
      else if (w + wt > 0.985 * std::ceil(w))
        sum += (p->precision == NR_F32 || grad_waves_per_simd(NR_F64, lmax) == 1 ? 1.0 : 1.6) * each;
    }
    if (launches <= 1) return std::max(sum, work);
    return std::max(sum / std::min(launches, 1 + kSideStreams) + 0.7 * work, work) +
           kReduceUs * (double)most_records;
  };
  struct Candidate {
    UnitPlan units;
    double us[2];
  };
  std::vector<Candidate> list;
  auto add = [&](UnitPlan u) { list.push_back({u, {estimate(u, false), estimate(u, true)}}); };
  for (int G : {1, 2, 3, 4, 5, 6, 9, 17}) {
    if (count(G) > limit) continue;
    add({G, false});
    if (G == 1 && p->opts.pack_tails) {
      int launches = 0, pack = 0;
      for (int k = 0; k < kNumBuckets; ++k) {
        launches += of[k].all() > 0;
        pack += of[k].tails > 0 && of[k].waves >= simds && p->bucket_form[k] != kFormSelect &&
                grad_waves_per_simd(p->precision, kBucketLmax[k]) == 1;
      }
      if (launches == 1 && pack == 1) add({1, true});
    }
  }
  std::array<UnitPlan, 2> out;
  size_t best = 0;
  for (int res : {0, 1}) {
    for (size_t k = 0; k < list.size(); ++k)
      if (list[k].us[res] < 0.99 * list[best].us[res]) best = k;
    if (!list.empty()) out[res] = list[best].units;
  }
  return out;
}

// The streams of a schedule's launches.  A launch that does not fill the device,
// or the last waves of one that does, leave it idle until the next launch of their
// stream; launches on other streams fill it.  The longest launches come first, each
// on the stream with the least work so far.  Measured on MI355X, two streams in the
// old order -> four in this one, ragged batches of 2..40 layers: 200 items 3.37 ->
// 0.87 ms (with node groups chosen for it), 700: 4.1 -> 2.9, 2048: 6.5 -> 5.0, 2048 in
// FP32 4.2 -> 3.1.  Three exceptions:
//  * A plan of many units per SIMD spends little on such gaps and loses more where
//    kernels of different register budgets mix on a SIMD (16384 items in FP32 22.5 ->
//    23.4 ms, in FP64 36.9 both): it keeps two streams, alternating from bucket to
//    bucket, with the small launches beside them.
//  * Where the whole units of a plan of one depth leave no room in their last round, a
//    split or packed launch of more than three waves per SIMD, which fills the device
//    alone, comes after them (beside / after, us a call: 4096 draws of 10 layers x 400
//    points, 24 and 4 units per SIMD, 2254 / 2225, x 80 points 552 / 518, 28 layers x 90
//    points 2066 / 1993; but 4200 draws of 10 layers FP64 x 80 points 580 / 637, x 90 643
//    / 724, x 209 1312 / 1358, x 400 2398 / 2409, 6500 of 20 layers FP32 x 90 1184 / 1297, and
//    beside is the faster one for 117 of 120 such plans of 4 to 36 layers).
//  * A call that forks takes some 55 us however short its kernels are (events and
//    waits, on the host and across hardware queues), so launches that are done by
//    then in a row stay in a row: two items of 20 and 2 layers 46.6 us in a row, 48-57
//    on two streams; two of 28 and 6 60.5 / 55.3.
constexpr double kForkCallUs = 55.0, kLaunchUs = 5.0;
void assign_streams(GradSchedule& S, bool side, int precision, int64_t simds) {
  std::vector<Launch>& list = S.launches;
  S.n_side = 0;
  if (!side || list.size() < 2) return;
  int64_t total = 0;
  double us = 0.0;
  for (const Launch& L : list) {
    total += L.n_wu;
    us += L.est + kLaunchUs;
  }
  if (us <= kForkCallUs) return;
  if (total > 48 * simds) {
    int full = 0;
    for (Launch& L : list) {
      const bool whole = !L.tail && !L.split;
      L.side = whole ? full++ % 2 : L.n_wu <= 2 * simds ? 1 : 0;
      S.n_side = std::max(S.n_side, L.side);
    }
    return;
  }
  std::stable_sort(list.begin(), list.end(),
                   [](const Launch& x, const Launch& y) { return x.est > y.est; });
  // what the whole units of the one depth leave idle of a wave per SIMD
  int whole = 0;
  double idle = 1.0;
  for (const Launch& L : list) {
    if (L.tail || L.split) continue;
    const double per = L.bucket == kDeepBucket
                           ? 1.0
                           : grad_waves_per_simd(precision, kBucketLmax[L.bucket]);
    const double rounds = (double)L.n_wu / (per * (double)simds);
    ++whole;
    idle = per * (std::ceil(rounds) - rounds);
  }
  double load[1 + kSideStreams] = {};
  for (Launch& L : list) {
    const bool after = (L.tail || L.split) && L.n_wu > 3 * simds && whole == 1 && idle < 0.05;
    L.side = after ? 0 : (int)(std::min_element(load, load + 1 + kSideStreams) - load);
    load[L.side] += L.est;
    S.n_side = std::max(S.n_side, L.side);
  }
}

nr_status run_launches(const nr_plan* p, int op, KernelArgs a, hipStream_t st,
                       bool events = true, bool res = false);

// res: gradient launches take the form that also yields the derivative with
// respect to the relative resolution.
nr_status run_launches(const nr_plan* p, int op, KernelArgs a, hipStream_t st, bool events,
                       bool res) {
  {
    // the select form and the value kernels with node forms read the scaled factors
    const bool grad_scaled = op == kOpLoglikGrad && p->grad_scaled && !res;
    hipError_t e = launch_item_consts(
        p->precision == NR_F32   ? kConstsFloat
        : op != kOpLoglikGrad    ? (p->value_forms ? kConstsScaled : kConstsPlain)
        : !grad_scaled           ? kConstsPlain
        : p->scan_select         ? kConstsScan
                                 : kConstsScaled,
        p->d_row_off,
        a.layers, const_cast<double*>(a.consts), const_cast<float*>(a.constsf), p->n_items, st);
    if (e != hipSuccess) return hip_fail(e, "constants launch");
  }
  if (events && p->ev_start) {
    hipError_t e = hipEventRecord(p->ev_start, st);
    if (e != hipSuccess) return hip_fail(e, "timing event");
  }
  const bool grad = (op == kOpLoglikGrad);
  const GradSchedule& sched = p->schedule(res);
  // fork: the side streams wait for the constants (and everything before
  // them on st); join: st waits for the side streams' launches
  bool fork = grad && sched.n_side > 0;
  std::unique_lock<std::mutex> lock;
  // A call being captured into a graph uses streams and events of its plan, so
  // that none is shared between captured and eager fork/joins.
  const ForkJoin* fj = nullptr;
  if (fork) {
    SidePool& pool = g_side_pool[p->device];
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    hipError_t e = hipStreamIsCapturing(st, &cs);
    const bool capturing = e == hipSuccess && cs != hipStreamCaptureStatusNone;
    lock = std::unique_lock<std::mutex>(capturing ? p->cap_mu : pool.mu);
    if (capturing) {
      fj = &p->cap;
      RelaxedCapture relaxed;
      e = fork_join_make(p->cap, sched.n_side);
    } else if (side_pool_free(pool, st)) {
      fj = &pool.set;
      pool.caller = st;
      pool.used = sched.n_side;
    } else {
      fork = false;
      lock.unlock();
    }
    if (fork) {
      if (e == hipSuccess) e = hipEventRecord(fj->fork, st);
      for (int k = 0; k < sched.n_side && e == hipSuccess; ++k)
        e = hipStreamWaitEvent(fj->st[k], fj->fork, 0);
    }
    if (e != hipSuccess) return hip_fail(e, "side stream fork");
  }
  hipError_t launch_err = hipSuccess;
  for (const Launch& L : grad ? sched.launches : p->launches_fwd) {
    a.wu_item = L.item;
    a.wu_p0 = L.p0;
    a.wu_rec = L.rec;
    a.wu_split = L.split_code;
    a.tail_item = L.lane_item;
    a.tail_pt = L.lane_pt;
    a.tail_rec = L.lane_rec;
    const int form = res ? kFormRecomputeRes : L.form;
    const int mode = L.tail              ? kModeTail
                     : L.one[res]        ? kModeSplitOne
                     : L.split           ? kModeSplit
                                         : kModeFull;
    const hipStream_t ls = (fork && L.side > 0) ? fj->st[L.side - 1] : st;
    if (!grad)
      launch_err = launch_forward(p->precision, op, L.split, p->value_forms, a, L.n_wu, ls);
    else if (L.bucket == kDeepBucket)
      launch_err = form == kFormSelect ? launch_grad_scan_select(L.scan_ch, a, L.n_wu, ls)
                                       : launch_grad_scan(res, L.scan_ch, a, L.n_wu, ls);
    else
      launch_err = launch_grad(p->precision, L.bucket, form, mode, a, L.n_wu, ls);
    if (launch_err != hipSuccess) break;
  }
  if (fork) {
    // joined even after a failed launch, so that a capture stays well formed
    hipError_t e = hipSuccess;
    for (int k = 0; k < sched.n_side; ++k) {
      hipError_t ek = hipEventRecord(fj->join[k], fj->st[k]);
      if (ek == hipSuccess) ek = hipStreamWaitEvent(st, fj->join[k], 0);
      if (e == hipSuccess) e = ek;
    }
    if (e != hipSuccess && launch_err == hipSuccess) return hip_fail(e, "side stream join");
  }
  if (launch_err != hipSuccess) return hip_fail(launch_err, "kernel launch");
  if (events && p->ev_stop) {
    hipError_t e = hipEventRecord(p->ev_stop, st);
    if (e != hipSuccess) return hip_fail(e, "timing event");
  }
  return NR_OK;
}

// Enqueues the whole logL + gradient evaluation (validated arguments); with
// seed set, the vector-Jacobian product of R_hat instead.
nr_status enqueue_grad(const nr_plan* p, const nr_values* v, double* logL, double* g_rows,
                       double* g_inst, void* ws, hipStream_t s, bool events,
                       const double* seed = nullptr, double* g_res = nullptr) {
  KernelArgs a = base_args(p, v);
  a.seed = seed;
  a.consts = static_cast<double*>(ws);
  a.constsf = consts_floats(p, a.consts);
  a.rec = static_cast<double*>(ws) + consts_doubles(p);
  nr_status st = run_launches(p, kOpLoglikGrad, a, s, events, g_res != nullptr);
  if (st != NR_OK) return st;
  ReduceArgs r;
  std::memset(&r, 0, sizeof(r));
  r.n_items = p->n_items;
  const RecordLists& lists = p->schedule(g_res != nullptr).lists;
  r.item_wu_first = lists.first;
  r.item_wu_count = lists.count;
  r.rec_of_wu = lists.offs;
  r.rec = a.rec;
  r.row_off = p->d_row_off;
  r.layers = v->layers;
  r.logL = logL;
  r.g_rows = g_rows;
  r.g_inst = g_inst;
  r.g_res = g_res;
  r.max_rows = p->max_rows;
  hipError_t e = launch_reduce(kOpLoglikGrad, r, s);
  return e == hipSuccess ? NR_OK : hip_fail(e, "reduce launch");
}

nr_status check_hmc(const nr_plan* p, const nr_values* data, const nr_hmc_state* st, double dt,
                    int32_t n_steps, void* ws, size_t ws_bytes) {
  if (!p || !data || !st || n_steps < 0 || !std::isfinite(dt)) return NR_EINVAL;
  nr_values v = *data;
  v.layers = st->layers;
  v.scale = st->scale;
  v.bkg = st->bkg;
  nr_status s = check_call(p, &v, true);
  if (s != NR_OK) return s;
  if (p->n_items == 0) return NR_OK;
  if (!st->mom_rows || !st->mom_inst || !st->logL || !st->g_rows || !st->g_inst)
    return NR_EINVAL;
  const size_t need = sizeof(double) * op_doubles(p, NR_OP_LOGLIK_GRAD);
  if (need > 0 && (!ws || ws_bytes < need)) return NR_EWORKSPACE;
  return NR_OK;
}

nr_status enqueue_leapfrog(const nr_plan* p, const nr_values* data, const nr_hmc_state* st,
                           double dt, int32_t n_steps, void* ws, hipStream_t s, bool events) {
  if (p->n_items == 0) return NR_OK;
  nr_values v = *data;
  v.layers = st->layers;
  v.scale = st->scale;
  v.bkg = st->bkg;
  const int64_t nre = p->row_off.back() * 4;
  const int64_t ni = p->n_items;
  for (int32_t k = 0; k < n_steps; ++k) {
    hipError_t e = launch_kick(nre, 2 * ni, st->mom_rows, st->g_rows, st->mom_inst, st->g_inst,
                               0.5 * dt, s);
    if (e != hipSuccess) return hip_fail(e, "kick launch");
    e = launch_drift(nre, ni, p->d_row_kind, st->layers, st->scale, st->bkg, st->mom_rows,
                     st->mom_inst, st->inv_mass_rows, st->inv_mass_inst, dt, s);
    if (e != hipSuccess) return hip_fail(e, "drift launch");
    nr_status r = enqueue_grad(p, &v, st->logL, st->g_rows, st->g_inst, ws, s, events);
    if (r != NR_OK) return r;
    e = launch_kick(nre, 2 * ni, st->mom_rows, st->g_rows, st->mom_inst, st->g_inst, 0.5 * dt, s);
    if (e != hipSuccess) return hip_fail(e, "kick launch");
  }
  return NR_OK;
}

}  // namespace

struct nr_graph {
  hipStream_t stream = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

struct nr_hmc {
  const nr_plan* plan = nullptr;
  nr_hmc_config cfg;
  int64_t n_entries = 0;  // 4 x rows + 2 x items
  double* buf = nullptr;  // r, z0, g0, wmean, wm2 (n_entries each), then the chain scalars
  uint64_t* iter = nullptr;
};

namespace {

bool chains_complete(const nr_hmc_chains* ch) {
  const void* need[] = {ch->z_rows, ch->z_inst, ch->kind_rows, ch->kind_inst, ch->a_rows,
                        ch->b_rows, ch->a_inst, ch->b_inst, ch->inv_mass_rows,
                        ch->inv_mass_inst, ch->step, ch->layers, ch->scale, ch->bkg,
                        ch->logL, ch->g_rows, ch->g_inst, ch->potential, ch->accept_prob,
                        ch->energy_error, ch->n_accept, ch->n_divergent};
  for (const void* q : need)
    if (!q) return false;
  return true;
}

nr_status check_chains(const nr_hmc* h, const nr_values* data, const nr_hmc_chains* ch, void* ws,
                       size_t ws_bytes) {
  if (!h || !data || !ch) return NR_EINVAL;
  nr_values v = *data;
  v.layers = ch->layers;
  v.scale = ch->scale;
  v.bkg = ch->bkg;
  nr_status s = check_call(h->plan, &v, true);
  if (s != NR_OK) return s;
  if (h->plan->n_items == 0) return NR_OK;
  if (!chains_complete(ch)) return NR_EINVAL;
  const size_t bytes = sizeof(double) * op_doubles(h->plan, NR_OP_LOGLIK_GRAD);
  if (bytes > 0 && (!ws || ws_bytes < bytes)) return NR_EWORKSPACE;
  return NR_OK;
}

HmcArgs hmc_args(const nr_hmc* h, const nr_hmc_chains* ch) {
  const nr_plan* p = h->plan;
  HmcArgs a;
  std::memset(&a, 0, sizeof(a));
  a.n_items = p->n_items;
  a.n_row_entries = p->row_off.back() * 4;
  a.row_off = p->d_row_off;
  a.row_kind = p->d_row_kind;
  a.z_rows = ch->z_rows;
  a.z_inst = ch->z_inst;
  a.kind_rows = ch->kind_rows;
  a.kind_inst = ch->kind_inst;
  a.a_rows = ch->a_rows;
  a.b_rows = ch->b_rows;
  a.a_inst = ch->a_inst;
  a.b_inst = ch->b_inst;
  a.im_rows = ch->inv_mass_rows;
  a.im_inst = ch->inv_mass_inst;
  a.step = ch->step;
  a.layers = ch->layers;
  a.scale = ch->scale;
  a.bkg = ch->bkg;
  a.logL = ch->logL;
  a.g_rows = ch->g_rows;
  a.g_inst = ch->g_inst;
  a.U = ch->potential;
  a.accept_prob = ch->accept_prob;
  a.energy_error = ch->energy_error;
  a.n_accept = ch->n_accept;
  a.n_divergent = ch->n_divergent;
  const int64_t n = h->n_entries;
  a.r = h->buf;
  a.z0 = h->buf + n;
  a.g0 = h->buf + 2 * n;
  a.wmean = h->buf + 3 * n;
  a.wm2 = h->buf + 4 * n;
  a.cs = h->buf + 5 * n;
  a.iter = h->iter;
  a.seed = h->cfg.seed;
  a.max_energy_error = h->cfg.max_energy_error;
  a.target_accept = h->cfg.target_accept;
  return a;
}

}  // namespace

struct nr_vi_mvn {
  const nr_plan* plan = nullptr;
  nr_vi_mvn_config cfg;
  int32_t P = 0, rows = 0;
  double* buf = nullptr;  // eps, z, h, f, layers, scale, bkg, logL, g_rows, g_inst, adam m, v
  uint64_t* iter = nullptr;
  MvnArgs args;           // driver-owned pointers and configuration
};

namespace {

nr_status check_mvn(const nr_vi_mvn* m, const nr_values* data, const nr_vi_mvn_params* prm,
                    void* ws, size_t ws_bytes) {
  if (!m || !data || !prm) return NR_EINVAL;
  const void* need[] = {prm->kind, prm->a, prm->b, prm->theta_fixed, prm->mu, prm->omega,
                        prm->lam, prm->elbo, prm->grad_mu, prm->grad_omega, prm->grad_lam};
  for (const void* q : need)
    if (!q) return NR_EINVAL;
  nr_values v = *data;
  v.layers = m->args.layers;
  v.scale = m->args.scale;
  v.bkg = m->args.bkg;
  nr_status s = check_call(m->plan, &v, true);
  if (s != NR_OK) return s;
  const size_t bytes = sizeof(double) * op_doubles(m->plan, NR_OP_LOGLIK_GRAD);
  if (bytes > 0 && (!ws || ws_bytes < bytes)) return NR_EWORKSPACE;
  return NR_OK;
}

MvnArgs mvn_args(const nr_vi_mvn* m, const nr_vi_mvn_params* prm) {
  MvnArgs a = m->args;
  a.kind = prm->kind;
  a.a = prm->a;
  a.b = prm->b;
  a.theta_fixed = prm->theta_fixed;
  a.mu = prm->mu;
  a.omega = prm->omega;
  a.lam = prm->lam;
  a.grad_mu = prm->grad_mu;
  a.grad_omega = prm->grad_omega;
  a.grad_lam = prm->grad_lam;
  a.elbo = prm->elbo;
  return a;
}

// One step: draws, logL + gradient of every draw, the z-gradients, the
// per-restart ELBO and gradient, Adam (optional), the iteration tick.
nr_status enqueue_mvn_step(const nr_vi_mvn* m, const nr_values* data,
                           const nr_vi_mvn_params* prm, bool adam, void* ws, hipStream_t s,
                           bool events) {
  const MvnArgs a = mvn_args(m, prm);
  nr_values v = *data;
  v.layers = a.layers;
  v.scale = a.scale;
  v.bkg = a.bkg;
  hipError_t e = launch_mvn(kMvnSample, a, s);
  if (e != hipSuccess) return hip_fail(e, "mvn sample");
  nr_status r = enqueue_grad(m->plan, &v, a.logL, a.g_rows, a.g_inst, ws, s, events);
  if (r != NR_OK) return r;
  e = launch_mvn(kMvnChain, a, s);
  if (e == hipSuccess) e = launch_mvn(kMvnReduce, a, s);
  if (e == hipSuccess && adam) e = launch_mvn(kMvnAdam, a, s);
  if (e == hipSuccess) e = launch_mvn(kMvnTick, a, s);
  return e == hipSuccess ? NR_OK : hip_fail(e, "mvn launch");
}

nr_values chain_values(const nr_values* data, const nr_hmc_chains* ch) {
  nr_values v = *data;
  v.layers = ch->layers;
  v.scale = ch->scale;
  v.bkg = ch->bkg;
  return v;
}

// One transition (Sec. 2.3): begin (momentum, first half kick), then per
// leapfrog step drift, logL + gradient, kick (a full kick where two half
// kicks meet), then the accept.
nr_status enqueue_transition(const nr_hmc* h, const nr_values* data, const nr_hmc_chains* ch,
                             int32_t adapt, void* ws, hipStream_t s, bool events) {
  const nr_plan* p = h->plan;
  if (p->n_items == 0) return NR_OK;
  const HmcArgs a = hmc_args(h, ch);
  const nr_values v = chain_values(data, ch);
  hipError_t e = launch_hmc(kHmcBegin, a, 0, 0.0, s);
  if (e != hipSuccess) return hip_fail(e, "hmc begin");
  const int L = h->cfg.n_leapfrog;
  for (int k = 0; k < L; ++k) {
    e = launch_hmc(kHmcDrift, a, 0, 0.0, s);
    if (e != hipSuccess) return hip_fail(e, "hmc drift");
    nr_status r = enqueue_grad(p, &v, ch->logL, ch->g_rows, ch->g_inst, ws, s, events);
    if (r != NR_OK) return r;
    e = launch_hmc(kHmcKick, a, 0, (k + 1 < L) ? 1.0 : 0.5, s);
    if (e != hipSuccess) return hip_fail(e, "hmc kick");
  }
  e = launch_hmc(kHmcEnd, a, adapt, 0.0, s);
  return e == hipSuccess ? NR_OK : hip_fail(e, "hmc end");
}

}  // namespace

extern "C" {

int32_t nr_version(void) { return NR_VERSION; }

const char* nr_status_string(nr_status s) {
  switch (s) {
    case NR_OK:
      return "ok";
    case NR_EINVAL:
      return "invalid argument";
    case NR_EWORKSPACE:
      return "workspace missing or too small";
    case NR_EHIP:
      return g_last_hip_error.empty() ? "HIP error" : g_last_hip_error.c_str();
    case NR_ENOMEM:
      return "device allocation failed";
    case NR_ESCRATCH:
      return "the plan's workspace exceeds the fixed scratch of nr_loglik_grad_noalloc "
             "(NR_NOALLOC_SCRATCH_BYTES); use nr_loglik_grad with a workspace";
    default:
      return "unknown status";
  }
}

nr_status nr_smearing_rule(double* t, double* w) {
  if (!t || !w) return NR_EINVAL;
  smearing_rule(t, w);
  return NR_OK;
}

nr_status nr_plan_options_default(nr_plan_options* o) {
  if (!o) return NR_EINVAL;
  for (int k = 0; k < NR_NUM_BUCKETS; ++k) o->grad_variant[k] = NR_VARIANT_AUTO;
  o->xcd_run = 8;
  o->pack_tails = 1;
  o->split_tails = NR_TAILS_LONE | NR_TAILS_SPLIT | NR_SPLIT_SMALL;
  o->side_stream = 1;
  o->node_groups = 0;
  return NR_OK;
}

int32_t nr_bucket_lmax(int32_t k) { return (k < 0 || k >= kNumBuckets) ? -1 : kBucketLmax[k]; }

int32_t nr_store_max_layers(int32_t precision) {
  if (precision != NR_F64 && precision != NR_F32) return -1;
  return store_max_layers(precision);
}

nr_status nr_plan_create(const nr_batch_desc* d, nr_plan** out) {
  return nr_plan_create_ex(d, nullptr, out);
}

nr_status nr_plan_create_ex(const nr_batch_desc* d, const nr_plan_options* opts, nr_plan** out) {
  if (!out) return NR_EINVAL;
  *out = nullptr;
  nr_status st = validate_desc(d);
  if (st != NR_OK) return st;
  nr_plan_options o;
  nr_plan_options_default(&o);
  if (opts) o = *opts;
  if (o.xcd_run < 1 || o.xcd_run > 64 || (o.pack_tails != 0 && o.pack_tails != 1) ||
      (o.split_tails & ~(NR_TAILS_LONE | NR_TAILS_SPLIT | NR_SPLIT_SMALL)) ||
      (o.side_stream != 0 && o.side_stream != 1) ||
      !(o.node_groups == 0 || (o.node_groups >= 2 && o.node_groups <= kSmearNodes)))
    return NR_EINVAL;
  // buckets deeper than kSelectMaxLayers that the batch uses
  bool used[kNumBuckets + 1] = {};
  for (int b = 0; b < d->n_items; ++b)
    used[bucket_of((int)(d->row_off[b + 1] - d->row_off[b]) - 2)] = true;
  int deep_kinds = 0;
  for (int k = 0; k < kNumBuckets; ++k) deep_kinds += used[k] && kBucketLmax[k] > kSelectMaxLayers;
  const int select_max = deep_kinds == 1 ? kSelectAloneLayers : kSelectMaxLayers;
  int bucket_form[kNumBuckets];
  for (int k = 0; k < kNumBuckets; ++k) {
    const int v = o.grad_variant[k];
    const bool can_store = kBucketLmax[k] <= store_max_layers(d->precision);
    if (v == NR_VARIANT_AUTO) {
      bucket_form[k] = kBucketLmax[k] <= default_store_layers(d->precision) ? kFormStore
                       : d->precision == NR_F64 && kBucketLmax[k] >= kSelectMinLayers &&
                               kBucketLmax[k] <= select_max
                           ? kFormSelect
                           : kFormRecompute;
    } else if (v == NR_VARIANT_STORE) {
      if (!can_store) return NR_EINVAL;
      bucket_form[k] = kFormStore;
    } else if (v == NR_VARIANT_RECOMPUTE) {
      bucket_form[k] = kFormRecompute;
    } else {
      return NR_EINVAL;
    }
  }
  nr_plan* p = new nr_plan();
  p->opts = o;
  for (int k = 0; k < kNumBuckets; ++k) p->bucket_form[k] = bucket_form[k];
  if (hipGetDevice(&p->device) != hipSuccess) {
    delete p;
    return NR_EHIP;
  }
  p->n_datasets = d->n_datasets;
  p->n_items = d->n_items;
  p->precision = d->precision;
  p->q_off.assign(d->q_off, d->q_off + d->n_datasets + 1);
  p->row_off.assign(d->row_off, d->row_off + d->n_items + 1);
  p->dataset_of_item.assign(d->dataset_of_item, d->dataset_of_item + d->n_items);
  p->dqq.assign(d->dq_over_q, d->dq_over_q + d->n_datasets);
  smearing_rule(p->node_t, p->node_w);

  // ---- work lists -------------------------------------------------------
  // Forward ops: one unit per item x 64 points (the last may be partial),
  // one record (a logL partial) per unit.  Gradient op: full units as above
  // plus tail units that pack the trailing partial groups of items with the
  // same depth and node count; a full unit writes one record, and so does
  // each item's group of lanes in a tail unit.  Every item's records are
  // listed contiguously.
  const int nI = d->n_items;
  p->out_off.assign(nI + 1, 0);
  struct Wu {
    int32_t item, p0;
    int64_t rec;
    uint32_t cost;      // lanes x nodes x levels, or nodes x levels
    int32_t split = 0;  // split tail units: points | node groups << 16
  };
  struct Tail {
    int32_t item, p0, count;
    int64_t rec0;  // record of its first point
  };
  // gradient: one list per bucket, then three deep lists (kDeepBucket + c), by
  // the levels per lane an item needs at 64 lanes (c = 0: up to 8, 1: up to 16,
  // 2: more), which set the waves per data point of the scan kernel (1, 2, 4), so
  // that shallower deep items do not run with the idle lanes of the deepest one
  constexpr int kDeepClasses = 3;
  std::vector<Wu> fwd_units;
  int scan_ch[kDeepClasses] = {0, 0, 0};
  std::vector<int64_t> ll_first(nI), ll_offs;
  std::vector<int32_t> ll_count(nI);
  int64_t rec_ll = 0;
  // Small problems (NR_SPLIT_SMALL): one wave per 64 points leaves most of the
  // device idle, or its last round nearly empty, for as long as a wave takes
  // over the 17 nodes of its points; splitting the nodes of every point group
  // over G lanes gives G times the waves, each running 17 / G nodes.  The
  // value kernels (nr_loglik, nr_reflectivity) take the same split, with their
  // own unit count (deep items included: they have no scan form).
  int64_t simds = 0;
  {
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, p->device) ==
        hipSuccess)
      simds = 4 * (int64_t)cus;
  }
  simds = std::max<int64_t>(simds, 1);
  UnitPlan small, small_res;  // of the gradient calls
  int small_G_fwd = 1;
  if (p->opts.split_tails & NR_SPLIT_SMALL) {
    int64_t units = 0, units_fwd = 0, levels_fwd = 0;
    for (int b = 0; b < nI; ++b) {
      const int s = p->dataset_of_item[b];
      const int N = (int)(p->row_off[b + 1] - p->row_off[b]) - 2;
      const int64_t u = (p->q_off[s + 1] - p->q_off[s] + kWuPoints - 1) / kWuPoints;
      units_fwd += u;
      levels_fwd += u * (N + 1);
      if (bucket_of(N) != kDeepBucket) units += u;
    }
    // The resolution form's split kernels spend more registers on the derivative: a
    // choice of their own, and a schedule where it is another (us a call, split like
    // the plain gradient / whole: 2000 items of 96 points, 14 layers FP64 632 / 553, 16
    // layers FP32 447 / 353, but 2355 of 40 points, 10 layers FP64 221 / 315).
    if (units > 0 && units < kSmallPlanWaves * simds) {
      const std::array<UnitPlan, 2> pick = pick_units(p, units, simds);
      small = pick[0];
      small_res = pick[1];
    }
    // Value units, by how many each SIMD would get unsplit.  Measured on MI355X
    // (10 layers x 400 points, us a call at G = 1 / 2 / 6 / 9): 224 units 72 /
    // 47 / 32 / 29; 448: 74 / 48 / 40 / 41; 1344: 114 / 87 / 80 / 83; 1792:
    // 113 / 92 / 98 / 102; 2688: 147 / 130 / 137 / 139; 3584: 152 / 160 / 174 /
    // 178.  G = 4 leaves nodes over and is never the best.  G = 17 (one node per
    // lane) is the best up to 64 units of 64 points in FP64 (64 units at G = 9 /
    // 17: 12 layers 19.1 / 18.6, 20 layers 24.2 / 22.4, 40 layers 36.3 / 32.0; 96:
    // 19.6 / 22.5, 24.2 / 27.0, 36.7 / 41.5) and 100 in FP32 (96 units: 17.5 / 18.0,
    // 21.9 / 21.6, 33.9 / 31.8; 140: 19.7 / 20.4, 25.7 / 25.1, 41.8 / 38.3).  Deep FP32
    // items keep G = 9 longer (339 units at G = 6 / 9: 6 layers 17.7 / 18.2, 16 layers
    // 30.1 / 27.9, 28 layers 44.6 / 39.8, 40 layers 59.2 / 51.4; 312: 4 layers 17.6 / 19.4,
    // 12 layers 26.9 / 27.1).
    const bool f32 = p->precision == NR_F32;
    const bool f32_deep = f32 && levels_fwd >= 14 * units_fwd;
    if (units_fwd > 0)
      small_G_fwd = (f32 ? 10 : 16) * units_fwd <= simds  ? 17
                    : (f32_deep ? 2 : 4) * units_fwd < simds ? 9
                    : 2 * units_fwd < 3 * simds              ? 6
                    : units_fwd < 3 * simds                  ? 2
                                                             : 1;
  }
  // a tiling given by the caller: every point group split over node_groups
  if (p->opts.node_groups >= 2) small = small_res = UnitPlan{p->opts.node_groups, false};
  // Where every lane runs one node, the two node forms do not pay for their
  // costlier constants and the scalar record loads that a wave waits for at its
  // first node: the one-form kernels.  us a call, two forms / one: 10 smeared items
  // of 180 points, 6 layers 24.6 / 23.1, 18 layers 39.3 / 36.7, 36 layers 76.5 /
  // 68.6; unsmeared, 10 items of 180 points, 10 layers 24.8 / 23.6, 4000 of 400
  // 264 / 261, 1000 of 400, 32 layers 341 / 323, 3544 of 784, 21 layers 1394 / 1353.
  // The scan kernel of deep items likewise, up to two points per SIMD: 6 items of
  // 96 points, 306 layers 31.7 / 29.0, 22 of 84, 459 layers 63.7 / 61.1, but 100
  // of 300, 200 layers 207.6 / 235.0.
  bool one_node = true, scan_one_node = true;
  int64_t scan_points = 0;
  for (int b = 0; b < nI; ++b) {
    const int s = p->dataset_of_item[b];
    const bool smeared = p->dqq[s] > 0.0;
    if (bucket_of((int)(p->row_off[b + 1] - p->row_off[b]) - 2) == kDeepBucket) {
      scan_one_node &= !smeared;
      scan_points += p->q_off[s + 1] - p->q_off[s];
    } else {
      one_node &= !smeared || small.groups == kSmearNodes;
    }
  }
  scan_one_node &= scan_points <= 2 * simds;
  if (one_node)
    for (int& form : p->bucket_form)
      if (form == kFormSelect) form = kFormRecompute;
  for (int b = 0; b < nI; ++b) {
    const int s = p->dataset_of_item[b];
    const int64_t nq = p->q_off[s + 1] - p->q_off[s];
    const int N = (int)(p->row_off[b + 1] - p->row_off[b]) - 2;
    const int K = p->dqq[s] > 0.0 ? kSmearNodes : 1;
    p->out_off[b + 1] = p->out_off[b] + nq;
    ll_first[b] = (int64_t)ll_offs.size();
    {
      // value units: groups of npts points, the last one of what is left; a
      // smeared group of np points runs G = 64 / np node groups side by side
      const int npts = K > 1 ? kWuPoints / small_G_fwd : kWuPoints;
      for (int64_t p0 = 0; p0 < nq; p0 += npts) {
        const int np = (int)std::min<int64_t>(npts, nq - p0);
        const int G = std::min(kWuPoints / np, K);
        Wu u{b, (int32_t)p0, rec_ll, (uint32_t)((K + G - 1) / G * (N + 1))};
        u.split = np | (G << 16);
        fwd_units.push_back(u);
        ll_offs.push_back(rec_ll++);
      }
      ll_count[b] = (int32_t)(ll_offs.size() - (size_t)ll_first[b]);
    }
    p->max_rows = std::max(p->max_rows, N + 2);
  }
  p->rec_ll_total = rec_ll;

  hipError_t e = hipSuccess;
  {
    std::vector<uint8_t> kind((size_t)p->row_off.back(), 1);
    p->uniform_rows = nI > 0 ? (int)(p->row_off[1] - p->row_off[0]) : 0;
    for (int b = 0; b < nI; ++b) {
      kind[(size_t)p->row_off[b]] = 0;
      kind[(size_t)p->row_off[b + 1] - 1] = 2;
      if (p->row_off[b + 1] - p->row_off[b] != p->uniform_rows) p->uniform_rows = 0;
    }
    std::vector<double> rule(p->node_t, p->node_t + kSmearNodes);
    rule.insert(rule.end(), p->node_w, p->node_w + kSmearNodes);
    append_math_tables(rule);
    e = upload(p->owned, part(&p->d_dataset_of_item, p->dataset_of_item),
               part(&p->d_q_off, p->q_off), part(&p->d_row_off, p->row_off),
               part(&p->d_dqq, p->dqq), part(&p->d_out_off, p->out_off),
               part(&p->d_row_kind, kind), part(&p->lists_ll.first, ll_first),
               part(&p->lists_ll.count, ll_count), part(&p->lists_ll.offs, ll_offs),
               part(&p->d_rule, rule));
  }

  // full-unit launches: one per non-empty bucket, deepest first, LPT order
  auto make_full = [&](int op, std::vector<std::vector<Wu>>& units,
                       std::vector<Launch>& out_list, bool split) {
    for (int bk = (int)units.size() - 1; bk >= 0; --bk) {
      auto& v = units[bk];
      if (v.empty() || e != hipSuccess) continue;
      // Equal costs: where the kernel chooses between node forms, by the place
      // in the item's data set (low q first, as data are usually kept): units
      // in flight together then run the same form, whose code they share in
      // the instruction cache, and the units with many general nodes, the
      // longer ones, come first (10 layers 2 % faster, 16-20 layers 4-5 %).
      // Elsewhere the units of one item stay together.
      const bool forms = op == kOpLoglik ? p->precision == NR_F64
                                         : bk < kNumBuckets && p->bucket_form[bk] == kFormSelect;
      std::vector<uint64_t> key(v.size());
      for (size_t k = 0; k < v.size(); ++k) {
        const int s = p->dataset_of_item[v[k].item];
        // (a float's bits order as the number does, from zero up)
        const float at = forms ? (float)v[k].p0 / (float)(p->q_off[s + 1] - p->q_off[s]) : 0.0f;
        uint32_t bits;
        std::memcpy(&bits, &at, sizeof(bits));
        key[k] = (uint64_t)~v[k].cost << 32 | bits;
      }
      const std::vector<uint32_t> order = order_by(key);
      std::vector<int32_t> it(v.size()), p0(v.size()), sc(v.size());
      std::vector<int64_t> rc(v.size());
      for (size_t k = 0; k < v.size(); ++k) {
        const size_t src = order[xcd_order(k, v.size(), (size_t)p->opts.xcd_run)];
        it[k] = v[src].item;
        p0[k] = v[src].p0;
        rc[k] = v[src].rec;
        sc[k] = v[src].split;
      }
      Launch L;
      L.bucket = std::min(bk, kDeepBucket);
      // (deep items: the scan kernel that the deepest bucket's option names;
      // the records of an FP32 plan have no room for the scaled factors)
      const bool scan_select = p->precision == NR_F64 && !scan_one_node &&
                               p->opts.grad_variant[kNumBuckets - 1] == NR_VARIANT_AUTO;
      L.form = bk < kNumBuckets ? p->bucket_form[bk] : scan_select ? kFormSelect : kFormRecompute;
      L.scan_ch = bk >= kDeepBucket ? std::max(scan_ch[bk - kDeepBucket], 1) : 0;
      L.split = split;
      L.n_wu = (int)v.size();
      // (deep units: one to four waves of up to eight levels, 1.5 times the work)
      int nodes = 1;
      for (const Wu& u : v) {
        const int K = p->dqq[p->dataset_of_item[u.item]] > 0.0 ? kSmearNodes : 1;
        const int G = std::max(1, u.split >> 16);
        nodes = std::max(nodes, (K + G - 1) / G);
      }
      for (bool res : {false, true})
        L.one[res] = op == kOpLoglikGrad && split && nodes == 1 && L.bucket != kDeepBucket &&
                     (res || L.form != kFormSelect) &&
                     lane_counter_pays(p->precision, kBucketLmax[L.bucket], res, L.n_wu, simds);
      L.est = L.bucket == kDeepBucket
                  ? 0.68 * 8 * nodes * L.n_wu * std::max(1, L.scan_ch / 8) / (double)simds
                  : launch_estimate(p->precision, kBucketLmax[L.bucket], split, L.n_wu, nodes, simds);
      if (!split) sc.clear();
      e = upload(p->owned, part(&L.item, it), part(&L.p0, p0), part(&L.rec, rc),
                 part(&L.split_code, sc));
      out_list.push_back(L);
    }
  };
  {
    // the value kernels take any depth: one launch
    std::vector<std::vector<Wu>> all{std::move(fwd_units)};
    bool split = false;
    for (const Wu& u : all[0]) split |= (u.split >> 16) > 1;
    // The node forms save per level and node and their constants cost per item, so
    // items of little work in a launch of many waves take the one form.  us a call,
    // two forms / one, by points x levels of an unsmeared item: 3783 items of 182
    // 19.9 / 17.1, 546 27.6 / 25.8, 819 33.7 / 32.9, 1183 42.0 / 41.8, 4000 of 800
    // 38.3 / 33.9; 3094 86.3 / 92; in two waves per SIMD or fewer (whose kernel warms
    // the records) 1000 of 832 14.8 / 15.8.
    int64_t steps = 0;
    for (int b = 0; b < nI; ++b)
      steps += (p->out_off[b + 1] - p->out_off[b]) * (p->row_off[b + 1] - p->row_off[b] - 1) *
               (p->dqq[p->dataset_of_item[b]] > 0.0 ? kSmearNodes : 1);
    p->value_forms = p->precision == NR_F64 &&
                     (split || (int64_t)all[0].size() <= 2 * simds || steps >= 1300 * (int64_t)nI);
    make_full(kOpLoglik, all, p->launches_fwd, split);
  }
  // the gradient's schedule with every smeared point group split over the plan's node
  // groups (1: whole groups of 64 points and tails)
  auto build_grad = [&](UnitPlan unit_plan, GradSchedule& S) {
    const int small_G = unit_plan.groups;
    const int own_tails = unit_plan.pack ? 0 : p->opts.split_tails;
    std::vector<std::vector<Wu>> grad_units(kNumBuckets + kDeepClasses);
    std::vector<std::vector<Wu>> split_units(kNumBuckets);
    std::map<std::pair<int, int>, std::vector<Tail>> tails;  // (depth, nodes)
    std::vector<int64_t> gr_first(nI), gr_offs;
    std::vector<int32_t> gr_count(nI);
    int64_t rec_gr = 0;
    for (int b = 0; b < nI; ++b) {
      const int s = p->dataset_of_item[b];
      const int64_t nq = p->q_off[s + 1] - p->q_off[s];
      const int N = (int)(p->row_off[b + 1] - p->row_off[b]) - 2;
      const int K = p->dqq[s] > 0.0 ? kSmearNodes : 1;
      const int bk = bucket_of(N);
      const int64_t rsz = 4 + 4 * (N + 2);
      if (bk == kDeepBucket) {
        // one unit per data point; its lanes split the layers
        gr_first[b] = (int64_t)gr_offs.size();
        gr_count[b] = (int32_t)nq;
        const int ch64 = (N + 1 + 63) / 64;
        const int cls = ch64 <= 8 ? 0 : ch64 <= 16 ? 1 : 2;
        scan_ch[cls] = std::max(scan_ch[cls], ch64);
        for (int64_t k = 0; k < nq; ++k) {
          grad_units[kDeepBucket + cls].push_back(
              {b, (int32_t)k, rec_gr, (uint32_t)(K * (N + 1) * 64)});
          gr_offs.push_back(rec_gr);
          rec_gr += rsz;
        }
        continue;
      }
      if (K > 1 && small_G >= 2) {
        // every point group split over small_G node groups (lane = g npts + p)
        const int npts = kWuPoints / small_G;
        gr_first[b] = (int64_t)gr_offs.size();
        int32_t cnt = 0;
        for (int64_t p0 = 0; p0 < nq; p0 += npts) {
          const int np = (int)std::min<int64_t>(npts, nq - p0);
          Wu u{b, (int32_t)p0, rec_gr, (uint32_t)(np * K * (N + 1))};
          u.split = np | (small_G << 16);
          split_units[bk].push_back(u);
          gr_offs.push_back(rec_gr);
          rec_gr += rsz;
          ++cnt;
        }
        gr_count[b] = cnt;
        continue;
      }
      const int nfull = (int)(nq / kWuPoints);
      const int ntail = (int)(nq % kWuPoints);
      gr_first[b] = (int64_t)gr_offs.size();
      gr_count[b] = nfull + (ntail > 0 ? 1 : 0);
      for (int k = 0; k < nfull; ++k) {
        grad_units[bk].push_back({b, k * kWuPoints, rec_gr, (uint32_t)(kWuPoints * K * (N + 1))});
        gr_offs.push_back(rec_gr);
        rec_gr += rsz;
      }
      if (ntail > 0) {
        // A smeared tail gets a wave of its own: of 32 points or fewer with
        // node groups x points over the lanes, else with idle lanes.  Its
        // item stays wave-uniform, and no wave runs all 17 nodes for a few
        // points.  Packing tails of several items into one wave (per-lane
        // layer records, up to 1 KB of spill in the deep kernels, and launches
        // of few waves that each take as long as a full unit) was the rule
        // beyond 10 layers: 2048 ragged items 8.9 -> 6.6 ms, 200 items 5.3 ->
        // 3.4 ms, 16384 items 38.0 -> 37.0 ms, FP32 5.6 -> 4.2 ms for 2048.
        // Unsmeared tails, one node each, are still packed.
        const int G = std::min(kWuPoints / ntail, K);
        if ((p->opts.split_tails & NR_TAILS_LONE) && (ntail >= 48 || (K > 1 && G == 1))) {
          grad_units[bk].push_back({b, nfull * kWuPoints, rec_gr, (uint32_t)(ntail * K * (N + 1))});
        } else if ((own_tails & NR_TAILS_SPLIT) && G >= 2) {
          Wu u{b, nfull * kWuPoints, rec_gr, (uint32_t)(ntail * K * (N + 1))};
          u.split = ntail | (G << 16);
          split_units[bk].push_back(u);
        } else {
          tails[{N, K}].push_back({b, nfull * kWuPoints, ntail, rec_gr});
        }
        gr_offs.push_back(rec_gr);
        rec_gr += rsz;
      }
    }
    S.records = rec_gr;
    if (e == hipSuccess)
      e = upload(p->owned, part(&S.lists.first, gr_first), part(&S.lists.count, gr_count),
                 part(&S.lists.offs, gr_offs));

    std::vector<Launch> tail_launches;  // after the full units
    // tail launches: per (depth, nodes) group, largest tails first, first fit
    // into 64-lane units; then one launch per bucket over all its groups (the
    // units holding a single item join the full units below)
    {
      std::vector<std::vector<int32_t>> b_item(kNumBuckets), b_litem(kNumBuckets), b_lpt(kNumBuckets);
      std::vector<std::vector<int64_t>> b_lrec(kNumBuckets);
      int b_nodes[kNumBuckets] = {};
      for (auto& kv : tails) {
        const int bk = bucket_of(kv.first.first);
        b_nodes[bk] = std::max(b_nodes[bk], kv.first.second);
        auto& v = kv.second;
        std::stable_sort(v.begin(), v.end(),
                         [](const Tail& x, const Tail& y) { return x.count > y.count; });
        std::vector<int> fill;                   // lanes used per unit of this group
        std::vector<std::vector<size_t>> units;  // the tails of each unit
        for (size_t t = 0; t < v.size(); ++t) {
          size_t u = p->opts.pack_tails ? 0 : fill.size();
          while (u < fill.size() && fill[u] + v[t].count > kWuPoints) ++u;
          if (u == fill.size()) {
            fill.push_back(0);
            units.emplace_back();
          }
          units[u].push_back(t);
          fill[u] += v[t].count;
        }
        for (const auto& un : units) {
          if (un.size() == 1) {
            // a unit of one item is a full unit with idle lanes (its layer
            // records stay scalar loads)
            const Tail& t = v[un[0]];
            grad_units[bk].push_back(
                {t.item, t.p0, t.rec0, (uint32_t)(t.count * kv.first.second * (kv.first.first + 1))});
            continue;
          }
          const size_t base = b_item[bk].size() * kWuPoints;
          b_item[bk].push_back(v[un[0]].item);
          b_litem[bk].insert(b_litem[bk].end(), kWuPoints, -1);
          b_lpt[bk].insert(b_lpt[bk].end(), kWuPoints, 0);
          b_lrec[bk].insert(b_lrec[bk].end(), kWuPoints, -1);
          int f = 0;
          for (size_t ti : un) {
            const Tail& t = v[ti];
            for (int l = 0; l < t.count; ++l) {
              b_litem[bk][base + f + l] = t.item;
              b_lpt[bk][base + f + l] = t.p0 + l;
              b_lrec[bk][base + f + l] = t.rec0;
            }
            f += t.count;
          }
        }
      }
      for (int bk = kNumBuckets - 1; bk >= 0; --bk) {
        if (b_item[bk].empty() || e != hipSuccess) continue;
        // idle lanes repeat lane 0 of their unit (a valid point, result unused)
        for (size_t u = 0; u < b_item[bk].size(); ++u)
          for (int l = 0; l < kWuPoints; ++l)
            if (b_litem[bk][u * kWuPoints + l] < 0) {
              b_litem[bk][u * kWuPoints + l] = b_litem[bk][u * kWuPoints];
              b_lpt[bk][u * kWuPoints + l] = b_lpt[bk][u * kWuPoints];
            }
        Launch L;
        L.bucket = bk;
        L.form = p->bucket_form[bk] == kFormSelect ? kFormRecompute : p->bucket_form[bk];
        L.tail = true;
        L.n_wu = (int)b_item[bk].size();
        L.est = launch_estimate(p->precision, kBucketLmax[bk], true, L.n_wu, b_nodes[bk], simds);
        e = upload(p->owned, part(&L.item, b_item[bk]), part(&L.lane_item, b_litem[bk]),
                   part(&L.lane_pt, b_lpt[bk]), part(&L.lane_rec, b_lrec[bk]));
        tail_launches.push_back(L);
      }
    }

    make_full(kOpLoglikGrad, grad_units, S.launches, false);
    make_full(kOpLoglikGrad, split_units, S.launches, true);
    S.launches.insert(S.launches.end(), tail_launches.begin(), tail_launches.end());
    for (const Launch& L : S.launches) {
      p->grad_scaled |= L.form == kFormSelect;
      p->scan_select |= L.form == kFormSelect && L.bucket == kDeepBucket;
    }
    assign_streams(S, p->opts.side_stream != 0, p->precision, simds);
  };
  build_grad(small, p->grad);
  p->res_own = !(small_res == small);
  if (p->res_own) build_grad(small_res, p->grad_res);
  if (std::max(p->grad.n_side, p->grad_res.n_side) > 0 && e == hipSuccess) {
    e = side_pool_acquire(p->device);
    p->pooled = e == hipSuccess;
  }
  for (int c = 0; c < kDeepClasses && e == hipSuccess; ++c)
    if (scan_ch[c] > 0) e = prepare_grad_scan(scan_ch[c]);
  if (e == hipSuccess) e = prepare_reduce(p->max_rows);

  if (e != hipSuccess) {
    plan_free(p);
    delete p;
    g_last_hip_error = std::string("plan upload: ") + hipGetErrorString(e);
    return (e == hipErrorOutOfMemory) ? NR_ENOMEM : NR_EHIP;
  }
  *out = p;
  return NR_OK;
}

nr_status nr_leapfrog(const nr_plan* p, const nr_values* data, const nr_hmc_state* st, double dt,
                      int32_t n_steps, void* ws, size_t ws_bytes, void* stream) {
  nr_status s = check_hmc(p, data, st, dt, n_steps, ws, ws_bytes);
  if (s != NR_OK) return s;
  return enqueue_leapfrog(p, data, st, dt, n_steps, ws, (hipStream_t)stream, true);
}

nr_status nr_leapfrog_graph_create(const nr_plan* p, const nr_values* data, const nr_hmc_state* st,
                                   double dt, int32_t n_steps, void* ws, size_t ws_bytes,
                                   nr_graph** out) {
  if (!out) return NR_EINVAL;
  *out = nullptr;
  nr_status s = check_hmc(p, data, st, dt, n_steps, ws, ws_bytes);
  if (s != NR_OK) return s;
  nr_graph* g = new nr_graph();
  hipError_t e = hipStreamCreateWithFlags(&g->stream, hipStreamNonBlocking);
  if (e != hipSuccess) {
    delete g;
    return hip_fail(e, "graph stream");
  }
  e = hipStreamBeginCapture(g->stream, hipStreamCaptureModeThreadLocal);
  if (e == hipSuccess) {
    s = enqueue_leapfrog(p, data, st, dt, n_steps, ws, g->stream, false);
    hipError_t e2 = hipStreamEndCapture(g->stream, &g->graph);
    if (s == NR_OK && e2 != hipSuccess) s = hip_fail(e2, "end capture");
  } else {
    s = hip_fail(e, "begin capture");
  }
  if (s == NR_OK) {
    e = hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0);
    if (e != hipSuccess) s = hip_fail(e, "graph instantiate");
  }
  if (s != NR_OK) {
    nr_graph_destroy(g);
    return s;
  }
  *out = g;
  return NR_OK;
}

nr_status nr_hmc_create(const nr_plan* p, const nr_hmc_config* cfg, nr_hmc** out) {
  if (!out) return NR_EINVAL;
  *out = nullptr;
  if (!p || !cfg || cfg->n_leapfrog < 1 || !(cfg->max_energy_error > 0.0) ||
      !(cfg->target_accept > 0.0 && cfg->target_accept < 1.0))
    return NR_EINVAL;
  nr_hmc* h = new nr_hmc();
  h->plan = p;
  h->cfg = *cfg;
  h->n_entries = p->row_off.back() * 4 + 2 * (int64_t)p->n_items;
  const size_t nd = (size_t)(5 * h->n_entries + (int64_t)kChainScalars * p->n_items);
  hipError_t e = hipSuccess;
  if (nd > 0) {
    e = hipMalloc(reinterpret_cast<void**>(&h->buf), nd * sizeof(double));
    if (e == hipSuccess) e = hipMemset(h->buf, 0, nd * sizeof(double));
  }
  if (e == hipSuccess && p->n_items > 0) {
    e = hipMalloc(reinterpret_cast<void**>(&h->iter), p->n_items * sizeof(uint64_t));
    if (e == hipSuccess) e = hipMemset(h->iter, 0, p->n_items * sizeof(uint64_t));
  }
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    nr_hmc_destroy(h);
    (void)hip_fail(e, "hmc state");
    return (e == hipErrorOutOfMemory) ? NR_ENOMEM : NR_EHIP;
  }
  *out = h;
  return NR_OK;
}

nr_status nr_hmc_destroy(nr_hmc* h) {
  if (!h) return NR_OK;
  if (h->buf) (void)hipFree(h->buf);
  if (h->iter) (void)hipFree(h->iter);
  delete h;
  return NR_OK;
}

nr_status nr_hmc_init(nr_hmc* h, const nr_values* data, const nr_hmc_chains* ch,
                      int32_t from_theta, void* ws, size_t ws_bytes, void* stream) {
  nr_status s = check_chains(h, data, ch, ws, ws_bytes);
  if (s != NR_OK) return s;
  if (h->plan->n_items == 0) return NR_OK;
  hipStream_t st = (hipStream_t)stream;
  const HmcArgs a = hmc_args(h, ch);
  hipError_t e = launch_hmc(kHmcTheta, a, from_theta ? 1 : 0, 0.0, st);
  if (e != hipSuccess) return hip_fail(e, "hmc theta");
  const nr_values v = chain_values(data, ch);
  s = enqueue_grad(h->plan, &v, ch->logL, ch->g_rows, ch->g_inst, ws, st, true);
  if (s != NR_OK) return s;
  e = launch_hmc(kHmcPotential, a, 0, 0.0, st);
  return e == hipSuccess ? NR_OK : hip_fail(e, "hmc potential");
}

nr_status nr_hmc_transition(nr_hmc* h, const nr_values* data, const nr_hmc_chains* ch,
                            int32_t adapt, void* ws, size_t ws_bytes, void* stream) {
  nr_status s = check_chains(h, data, ch, ws, ws_bytes);
  if (s != NR_OK) return s;
  if (adapt & ~(NR_HMC_ADAPT_MASS | NR_HMC_ADAPT_STEP)) return NR_EINVAL;
  return enqueue_transition(h, data, ch, adapt, ws, (hipStream_t)stream, true);
}

nr_status nr_hmc_graph_create(nr_hmc* h, const nr_values* data, const nr_hmc_chains* ch,
                              int32_t adapt, int32_t n_transitions, void* ws, size_t ws_bytes,
                              nr_graph** out) {
  if (!out) return NR_EINVAL;
  *out = nullptr;
  nr_status s = check_chains(h, data, ch, ws, ws_bytes);
  if (s != NR_OK) return s;
  if (n_transitions < 0 || (adapt & ~(NR_HMC_ADAPT_MASS | NR_HMC_ADAPT_STEP))) return NR_EINVAL;
  nr_graph* g = new nr_graph();
  hipError_t e = hipStreamCreateWithFlags(&g->stream, hipStreamNonBlocking);
  if (e != hipSuccess) {
    delete g;
    return hip_fail(e, "graph stream");
  }
  e = hipStreamBeginCapture(g->stream, hipStreamCaptureModeThreadLocal);
  if (e == hipSuccess) {
    for (int32_t t = 0; t < n_transitions && s == NR_OK; ++t)
      s = enqueue_transition(h, data, ch, adapt, ws, g->stream, false);
    hipError_t e2 = hipStreamEndCapture(g->stream, &g->graph);
    if (s == NR_OK && e2 != hipSuccess) s = hip_fail(e2, "end capture");
  } else {
    s = hip_fail(e, "begin capture");
  }
  if (s == NR_OK) {
    e = hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0);
    if (e != hipSuccess) s = hip_fail(e, "graph instantiate");
  }
  if (s != NR_OK) {
    nr_graph_destroy(g);
    return s;
  }
  *out = g;
  return NR_OK;
}

nr_status nr_hmc_adapt(nr_hmc* h, const nr_hmc_chains* ch, int32_t actions, void* stream) {
  if (!h || !ch) return NR_EINVAL;
  if (actions & ~(NR_HMC_MASS_WINDOW_END | NR_HMC_STEP_RESTART | NR_HMC_STEP_FINAL))
    return NR_EINVAL;
  if (h->plan->n_items == 0 || actions == 0) return NR_OK;
  if (!chains_complete(ch)) return NR_EINVAL;
  hipError_t e = launch_hmc(kHmcAdapt, hmc_args(h, ch), actions, 0.0, (hipStream_t)stream);
  return e == hipSuccess ? NR_OK : hip_fail(e, "hmc adapt");
}

nr_status nr_vi_mvn_create(const nr_plan* p, const nr_vi_mvn_config* cfg, nr_vi_mvn** out) {
  if (!out) return NR_EINVAL;
  *out = nullptr;
  if (!p || !cfg || cfg->n_restarts < 1 || cfg->n_draws < 1 ||
      (int64_t)cfg->n_restarts * cfg->n_draws != p->n_items || p->uniform_rows < 2 ||
      p->uniform_rows > kMaxLayers + 2 ||
      !(cfg->lr > 0.0) || !(cfg->beta1 >= 0.0 && cfg->beta1 < 1.0) ||
      !(cfg->beta2 >= 0.0 && cfg->beta2 < 1.0) || !(cfg->adam_eps > 0.0))
    return NR_EINVAL;
  nr_vi_mvn* m = new nr_vi_mvn();
  m->plan = p;
  m->cfg = *cfg;
  m->rows = p->uniform_rows;
  m->P = 4 * m->rows + 2;
  const int64_t items = p->n_items, P = m->P, R = cfg->n_restarts;
  const int64_t n_adam = R * (2 * P + P * P);
  const int64_t sizes[] = {items * P, items * P, items * P, items, items * 4 * m->rows,
                           items, items, items, items * 4 * m->rows, items * 2, n_adam, n_adam};
  int64_t total = 0;
  for (int64_t v : sizes) total += v;
  hipError_t e = hipMalloc(reinterpret_cast<void**>(&m->buf), (size_t)total * sizeof(double));
  if (e == hipSuccess) e = hipMemset(m->buf, 0, (size_t)total * sizeof(double));
  if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void**>(&m->iter), sizeof(uint64_t));
  if (e == hipSuccess) e = hipMemset(m->iter, 0, sizeof(uint64_t));
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e != hipSuccess) {
    nr_vi_mvn_destroy(m);
    (void)hip_fail(e, "mvn state");
    return (e == hipErrorOutOfMemory) ? NR_ENOMEM : NR_EHIP;
  }
  double* ptrs[12];
  double* q = m->buf;
  for (int k = 0; k < 12; ++k) {
    ptrs[k] = q;
    q += sizes[k];
  }
  MvnArgs& a = m->args;
  std::memset(&a, 0, sizeof(a));
  a.R = cfg->n_restarts;
  a.S = cfg->n_draws;
  a.P = m->P;
  a.rows = m->rows;
  a.eps = ptrs[0];
  a.z = ptrs[1];
  a.h = ptrs[2];
  a.f = ptrs[3];
  a.layers = ptrs[4];
  a.scale = ptrs[5];
  a.bkg = ptrs[6];
  a.logL = ptrs[7];
  a.g_rows = ptrs[8];
  a.g_inst = ptrs[9];
  a.adam_m = ptrs[10];
  a.adam_v = ptrs[11];
  a.iter = m->iter;
  a.seed = cfg->seed;
  a.lr = cfg->lr;
  a.beta1 = cfg->beta1;
  a.beta2 = cfg->beta2;
  a.adam_eps = cfg->adam_eps;
  *out = m;
  return NR_OK;
}

nr_status nr_vi_mvn_destroy(nr_vi_mvn* m) {
  if (!m) return NR_OK;
  if (m->buf) (void)hipFree(m->buf);
  if (m->iter) (void)hipFree(m->iter);
  delete m;
  return NR_OK;
}

nr_status nr_vi_mvn_step(nr_vi_mvn* m, const nr_values* data, const nr_vi_mvn_params* prm,
                         int32_t adam, void* ws, size_t ws_bytes, void* stream) {
  nr_status s = check_mvn(m, data, prm, ws, ws_bytes);
  if (s != NR_OK) return s;
  return enqueue_mvn_step(m, data, prm, adam != 0, ws, (hipStream_t)stream, true);
}

nr_status nr_vi_mvn_graph_create(nr_vi_mvn* m, const nr_values* data, const nr_vi_mvn_params* prm,
                                 int32_t n_steps, void* ws, size_t ws_bytes, nr_graph** out) {
  if (!out) return NR_EINVAL;
  *out = nullptr;
  nr_status s = check_mvn(m, data, prm, ws, ws_bytes);
  if (s != NR_OK) return s;
  if (n_steps < 0) return NR_EINVAL;
  nr_graph* g = new nr_graph();
  hipError_t e = hipStreamCreateWithFlags(&g->stream, hipStreamNonBlocking);
  if (e != hipSuccess) {
    delete g;
    return hip_fail(e, "graph stream");
  }
  e = hipStreamBeginCapture(g->stream, hipStreamCaptureModeThreadLocal);
  if (e == hipSuccess) {
    for (int32_t t = 0; t < n_steps && s == NR_OK; ++t)
      s = enqueue_mvn_step(m, data, prm, true, ws, g->stream, false);
    hipError_t e2 = hipStreamEndCapture(g->stream, &g->graph);
    if (s == NR_OK && e2 != hipSuccess) s = hip_fail(e2, "end capture");
  } else {
    s = hip_fail(e, "begin capture");
  }
  if (s == NR_OK) {
    e = hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0);
    if (e != hipSuccess) s = hip_fail(e, "graph instantiate");
  }
  if (s != NR_OK) {
    nr_graph_destroy(g);
    return s;
  }
  *out = g;
  return NR_OK;
}

nr_status nr_graph_launch(nr_graph* g, void* stream) {
  if (!g || !g->exec) return NR_EINVAL;
  hipError_t e = hipGraphLaunch(g->exec, (hipStream_t)stream);
  return e == hipSuccess ? NR_OK : hip_fail(e, "graph launch");
}

nr_status nr_graph_destroy(nr_graph* g) {
  if (!g) return NR_OK;
  if (g->exec) (void)hipGraphExecDestroy(g->exec);
  if (g->graph) (void)hipGraphDestroy(g->graph);
  if (g->stream) (void)hipStreamDestroy(g->stream);
  delete g;
  return NR_OK;
}

nr_status nr_vi_elbo_grad(const nr_plan* p, const nr_values* data, const nr_vi_args* vi,
                          void* ws, size_t ws_bytes, void* stream) {
  if (!p || !data || !vi) return NR_EINVAL;
  if (p->n_items == 0) return NR_EINVAL;
  const int rows = p->uniform_rows;
  if (rows < 2) return NR_EINVAL;
  if (!vi->mu || !vi->omega || !vi->mask || !vi->eps || !vi->layers || !vi->scale ||
      !vi->bkg || !vi->logL || !vi->g_rows || !vi->g_inst || !vi->grad_mu ||
      !vi->grad_omega || !vi->elbo)
    return NR_EINVAL;
  nr_values v = *data;
  v.layers = vi->layers;
  v.scale = vi->scale;
  v.bkg = vi->bkg;
  nr_status s = check_call(p, &v, true);
  if (s != NR_OK) return s;
  const size_t need = sizeof(double) * op_doubles(p, NR_OP_LOGLIK_GRAD);
  if (need > 0 && (!ws || ws_bytes < need)) return NR_EWORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  const int P = rows * 4 + 2;
  hipError_t e = launch_vi_sample(p->n_items, P, rows, vi->mu, vi->omega, vi->mask, vi->eps,
                                  vi->layers, vi->scale, vi->bkg, st);
  if (e != hipSuccess) return hip_fail(e, "sampler launch");
  s = enqueue_grad(p, &v, vi->logL, vi->g_rows, vi->g_inst, ws, st, true);
  if (s != NR_OK) return s;
  e = launch_vi_reduce(p->n_items, P, rows, vi->omega, vi->mask, vi->eps, vi->logL, vi->g_rows,
                       vi->g_inst, vi->grad_mu, vi->grad_omega, vi->elbo, st);
  return e == hipSuccess ? NR_OK : hip_fail(e, "reduction launch");
}

nr_status nr_tie_sum(int64_t n_out, const int64_t* first, const int64_t* src, const double* in,
                     double* out, void* stream) {
  if (n_out < 0) return NR_EINVAL;
  if (n_out == 0) return NR_OK;
  if (!first || !src || !in || !out) return NR_EINVAL;
  hipError_t e = launch_tie_sum(n_out, first, src, in, out, (hipStream_t)stream);
  return e == hipSuccess ? NR_OK : hip_fail(e, "tie-sum launch");
}

nr_status nr_scale_gradient(const nr_plan* p, const double* g_rows, const double* g_inst,
                            const double* seed, int64_t seed_stride, double* out_rows,
                            double* out_inst, void* stream) {
  int dev = -1;
  if (!p || seed_stride < 0 || hipGetDevice(&dev) != hipSuccess || dev != p->device)
    return NR_EINVAL;
  if (p->n_items == 0) return NR_OK;
  if (!g_rows || !g_inst || !seed || !out_rows || !out_inst) return NR_EINVAL;
  hipError_t e = launch_scale_gradient(p->n_items, p->d_row_off, g_rows, g_inst, seed, seed_stride,
                                       out_rows, out_inst, (hipStream_t)stream);
  return e == hipSuccess ? NR_OK : hip_fail(e, "gradient scaling launch");
}

nr_status nr_plan_set_timing_events(nr_plan* p, void* start, void* stop) {
  if (!p || ((start == nullptr) != (stop == nullptr))) return NR_EINVAL;
  p->ev_start = static_cast<hipEvent_t>(start);
  p->ev_stop = static_cast<hipEvent_t>(stop);
  return NR_OK;
}

nr_status nr_plan_destroy(nr_plan* p) {
  if (!p) return NR_OK;
  plan_free(p);
  delete p;
  return NR_OK;
}

nr_status nr_workspace_size(const nr_plan* p, int32_t op, size_t* bytes) {
  if (!p || !bytes) return NR_EINVAL;
  if (op != NR_OP_REFLECTIVITY && op != NR_OP_LOGLIK && op != NR_OP_LOGLIK_GRAD) return NR_EINVAL;
  *bytes = sizeof(double) * op_doubles(p, op);
  return NR_OK;
}

nr_status nr_output_offsets(const nr_plan* p, int64_t* out_off) {
  if (!p || !out_off) return NR_EINVAL;
  std::memcpy(out_off, p->out_off.data(), sizeof(int64_t) * p->out_off.size());
  return NR_OK;
}

nr_status nr_plan_launches(const nr_plan* p, int32_t op, int32_t capacity, nr_launch_info* out,
                           int32_t* n_out) {
  if (!p || !n_out || (capacity > 0 && !out) || op < NR_OP_REFLECTIVITY || op > NR_OP_LOGLIK_GRAD)
    return NR_EINVAL;
  static_assert(NR_FORM_RECOMPUTE == kFormRecompute && NR_FORM_STORE == kFormStore &&
                    NR_FORM_SELECT == kFormSelect && NR_MODE_FULL == kModeFull &&
                    NR_MODE_PACKED == kModeTail && NR_MODE_SPLIT == kModeSplit,
                "the header's launch kinds and the kernels' disagree");
  static_assert(NR_NUM_BUCKETS == kDeepBucket, "the deep stacks' launches follow the buckets");
  const bool grad = op == NR_OP_LOGLIK_GRAD;
  const std::vector<Launch>& list = grad ? p->grad.launches : p->launches_fwd;
  *n_out = (int32_t)list.size();
  for (int32_t k = 0; k < capacity && k < *n_out; ++k) {
    const Launch& L = list[k];
    out[k].bucket = grad ? L.bucket : -1;
    out[k].form = grad ? L.form : p->value_forms ? NR_FORM_SELECT : NR_FORM_RECOMPUTE;
    out[k].mode = L.tail ? kModeTail : L.split ? kModeSplit : kModeFull;
    out[k].units = L.n_wu;
    out[k].stream = grad ? L.side : 0;
  }
  return NR_OK;
}

nr_status nr_reflectivity(const nr_plan* p, const nr_values* v, double* r_hat, void* ws,
                          size_t ws_bytes, void* stream) {
  nr_status st = check_call(p, v, false);
  if (st != NR_OK) return st;
  if (p->n_items == 0 || p->out_off.back() == 0) return NR_OK;
  if (!r_hat) return NR_EINVAL;
  if (!ws || ws_bytes < sizeof(double) * op_doubles(p, NR_OP_REFLECTIVITY)) return NR_EWORKSPACE;
  KernelArgs a = base_args(p, v);
  a.out = r_hat;
  a.consts = static_cast<double*>(ws);
  a.constsf = consts_floats(p, a.consts);
  return run_launches(p, kOpReflectivity, a, (hipStream_t)stream);
}

nr_status nr_loglik(const nr_plan* p, const nr_values* v, double* logL, void* ws,
                    size_t ws_bytes, void* stream) {
  nr_status st = check_call(p, v, true);
  if (st != NR_OK) return st;
  if (p->n_items == 0) return NR_OK;
  if (!logL) return NR_EINVAL;
  const size_t need = sizeof(double) * op_doubles(p, NR_OP_LOGLIK);
  if (need > 0 && (!ws || ws_bytes < need)) return NR_EWORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  KernelArgs a = base_args(p, v);
  a.consts = static_cast<double*>(ws);
  a.constsf = consts_floats(p, a.consts);
  a.rec = static_cast<double*>(ws) + consts_doubles(p);
  st = run_launches(p, kOpLoglik, a, s);
  if (st != NR_OK) return st;
  ReduceArgs r;
  std::memset(&r, 0, sizeof(r));
  r.n_items = p->n_items;
  r.item_wu_first = p->lists_ll.first;
  r.item_wu_count = p->lists_ll.count;
  r.rec_of_wu = p->lists_ll.offs;
  r.rec = a.rec;
  r.logL = logL;
  hipError_t e = launch_reduce(kOpLoglik, r, s);
  return e == hipSuccess ? NR_OK : hip_fail(e, "reduce launch");
}

nr_status nr_reflectivity_vjp(const nr_plan* p, const nr_values* v, const double* seed,
                              double* dot, double* g_rows, double* g_inst, void* ws,
                              size_t ws_bytes, void* stream) {
  nr_status st = check_call(p, v, false);
  if (st != NR_OK) return st;
  if (p->n_items == 0) return NR_OK;
  if (!dot || !g_rows || !g_inst) return NR_EINVAL;
  if (p->out_off.back() > 0 && !seed) return NR_EINVAL;
  const size_t need = sizeof(double) * op_doubles(p, NR_OP_LOGLIK_GRAD);
  if (need > 0 && (!ws || ws_bytes < need)) return NR_EWORKSPACE;
  return enqueue_grad(p, v, dot, g_rows, g_inst, ws, (hipStream_t)stream, true, seed);
}

nr_status nr_loglik_grad_res(const nr_plan* p, const nr_values* v, double* logL, double* g_rows,
                             double* g_inst, double* g_res, void* ws, size_t ws_bytes,
                             void* stream) {
  nr_status st = check_call(p, v, true);
  if (st != NR_OK) return st;
  if (p->n_items == 0) return NR_OK;
  if (!logL || !g_rows || !g_inst || !g_res) return NR_EINVAL;
  const size_t need = sizeof(double) * op_doubles(p, NR_OP_LOGLIK_GRAD);
  if (need > 0 && (!ws || ws_bytes < need)) return NR_EWORKSPACE;
  return enqueue_grad(p, v, logL, g_rows, g_inst, ws, (hipStream_t)stream, true, nullptr, g_res);
}

nr_status nr_loglik_grad(const nr_plan* p, const nr_values* v, double* logL, double* g_rows,
                         double* g_inst, void* ws, size_t ws_bytes, void* stream) {
  nr_status st = check_call(p, v, true);
  if (st != NR_OK) return st;
  if (p->n_items == 0) return NR_OK;
  if (!logL || !g_rows || !g_inst) return NR_EINVAL;
  const size_t need = sizeof(double) * op_doubles(p, NR_OP_LOGLIK_GRAD);
  if (need > 0 && (!ws || ws_bytes < need)) return NR_EWORKSPACE;
  return enqueue_grad(p, v, logL, g_rows, g_inst, ws, (hipStream_t)stream, true);
}

nr_status nr_loglik_grad_noalloc(const nr_plan* p, const nr_values* v, double* logL,
                                 double* g_rows, double* g_inst, void* stream) {
  nr_status st = check_call(p, v, true);
  if (st != NR_OK) return st;
  if (p->n_items == 0) return NR_OK;
  if (!logL || !g_rows || !g_inst) return NR_EINVAL;
  const size_t need = sizeof(double) * op_doubles(p, NR_OP_LOGLIK_GRAD);
  if (need > (size_t)NR_NOALLOC_SCRATCH_BYTES) return NR_ESCRATCH;
  void* ws = nullptr;
  st = scratch_addr(p->device, &ws);
  if (st != NR_OK) return st;
  return enqueue_grad(p, v, logL, g_rows, g_inst, ws, (hipStream_t)stream, true);
}

}  // extern "C"
