// Host runtime behind the C ABI in include/brmppi.h: arena sub-allocation,
// controller slots (resident path, warm start, plant state), the plain,
// batched (persistent kernels in a HIP graph) and closed-loop solves, and the
// served form (a request thread doing continuous batching over the streams).
#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <fstream>
#include <map>
#include <memory>
#include <mutex>
#include <sstream>
#include <string>
#include <thread>
#include <unordered_map>
#include <vector>

#include <rocprofiler-sdk-roctx/roctx.h>

#include "brmppi_internal.h"
#include "launch_plan.h"
#include "served_core.h"

using namespace brm;

static __device__ __align__(256) char scratch[BRMPPI_NOALLOC_MAX_BYTES];

namespace {

thread_local std::string g_err;

int fail(int code, const std::string& msg) {
  g_err = msg;
  return code;
}

#define HIPCHK(x)                                                                            \
  do {                                                                                       \
    hipError_t e_ = (x);                                                                     \
    if (e_ != hipSuccess) return fail(BRMPPI_EDEVICE, std::string(#x) + ": " + hipGetErrorString(e_)); \
  } while (0)


// ---------------------------------------------------------------------------
// static scratch of brmppi_solve_noalloc
// ---------------------------------------------------------------------------
// One array per GPU the library runs on, held until the process ends.  On the
// host the array's name is only a stand-in for the symbol, never a device
// address: brmppi_create looks up the array's address on its device with
// hipGetSymbolAddress (once per device, that device current), and every host
// use (kernel arguments through the descriptors, copies) goes through that
// address.
constexpr int kMaxDevices = 64;
std::mutex g_static_mu;                        // guards g_static_ptr
char* g_static_ptr[kMaxDevices] = {};          // the array's address on each device
std::mutex g_static_call_mu[kMaxDevices];      // one no-alloc call at a time per device

// a roctx range over a scope (rocprofv3 --marker-trace shows it)
struct TraceRange {
  explicit TraceRange(const char* name) { roctxRangePushA(name); }
  ~TraceRange() { roctxRangePop(); }
  TraceRange(const TraceRange&) = delete;
  TraceRange& operator=(const TraceRange&) = delete;
};

// pinned host staging buffer (allocated at create; re-allocated only when a
// call needs more, which `grows` counts)
constexpr size_t kPinnedInit = size_t(1) << 20;
struct Pinned {
  char* ptr = nullptr;
  size_t bytes = 0;
  uint64_t grows = 0;
  int ensure(size_t n) {
    if (n <= bytes) return 0;
    if (ptr) {
      (void)hipHostFree(ptr);
      ++grows;
    }
    ptr = nullptr;
    bytes = 0;
    n = round_up(std::max<size_t>(n, 4096), 4096);
    HIPCHK(hipHostMalloc((void**)&ptr, n, hipHostMallocDefault));
    bytes = n;
    return 0;
  }
  void release() {
    if (ptr) (void)hipHostFree(ptr);
    ptr = nullptr;
    bytes = 0;
  }
};

// (busy: a served request is in flight; warm_T: length of the resident warm
// start, 0 = none)
struct Controller : SlotState, Resident {
  Block mem;                  // unom (3*MAX_T floats) + plant (8 doubles)
  Block path_blk;
  bool plant_set = false;
};

// one instance's uploaded inputs: [descriptor | reduce counter (zero) | nominal
// sequence], staged together in pinned memory
struct InputBlock {
  size_t counter, unom, bytes;
};

InputBlock input_block(uint32_t T, bool with_unom, uint32_t n_groups) {
  InputBlock b;
  b.counter = (sizeof(SolveDesc) + 255) / 256 * 256;
  b.unom = b.counter + counter_bytes(n_groups);
  b.bytes = b.unom + (with_unom ? sizeof(float) * 3 * T : 0);
  return b;
}

const brmppi_params& params_of(const brmppi_ctx* ctx, const brmppi_problem& p);

// obstacle rows of a problem: one per (footprint disc, obstacle)
uint32_t obstacle_rows(const brmppi_ctx* ctx, const brmppi_problem& p) {
  return p.n_obs * n_discs(params_of(ctx, p));
}

// normals per (sample, step): 3 inputs, 2 hitch rows, one per obstacle row
uint32_t normals_per_step(const brmppi_ctx* ctx, const brmppi_problem& p) {
  return (p.flags & BRMPPI_GUIDANCE_OFF) ? 3u : 5u + obstacle_rows(ctx, p);
}

// rows of one reduce work item, per instance, for a launch over these
// instances.  An item costs about kRedItemPasses 8-row passes of fixed work
// (its costs, weights, row merge and publish) plus one per pass of rows, and
// the reduce blocks the chip holds take the items in rounds, so the launch
// lasts about (rounds) x (fixed + passes of the longest item).  The passes per
// item are chosen to minimise that (ties: fewer, longer items), and each
// (instance, group) splits its rows evenly over its items.  When every item
// fits one round, the fewest passes that keep it there win; beyond one round
// longer items cut the fixed work, and plan_fill queues them longest first.
void reduce_rows(const brmppi_problem* const* ps, uint32_t n, int n_cu, uint32_t* rows) {
  constexpr uint32_t kRedItemPasses = 5;
  const size_t slots = (size_t)std::max(1, n_cu) * kRedBlocksPerCU;
  const uint32_t max_pp = kMaxRowsPerItem / kRowsPerPass;
  auto passes = [&](uint32_t i) { return (3 * ps[i]->T + kRowsPerPass - 1) / kRowsPerPass; };
  uint32_t best_pp = max_pp;
  size_t best = SIZE_MAX;
  for (uint32_t pp = 1; pp <= max_pp; ++pp) {
    size_t items = 0;
    uint32_t longest = 0;
    for (uint32_t i = 0; i < n; ++i) {
      const uint32_t P = passes(i), nrg = (P + pp - 1) / pp;
      items += (size_t)((ps[i]->S + kWChunk - 1) / kWChunk) * nrg;
      longest = std::max(longest, (P + nrg - 1) / nrg);
    }
    const size_t cost = ((items + slots - 1) / slots) * (kRedItemPasses + longest);
    if (cost <= best) {
      best = cost;
      best_pp = pp;
    }
  }
  for (uint32_t i = 0; i < n; ++i) {
    const uint32_t P = passes(i), nrg = (P + best_pp - 1) / best_pp;
    rows[i] = kRowsPerPass * ((P + nrg - 1) / nrg);
  }
}

// largest precomputed-noise buffer a plain solve may take; it is also held to
// half of the context's arena.  Beyond it, and where the arena has no room for them,
// the solve draws its normals in the rollout kernel (variant_in_kernel).
constexpr size_t kMaxNoiseBytes = size_t(2) << 30;
// closed loop: normals of up to this many bytes are drawn per noise launch,
// and at most this many updates share one descriptor upload and noise launch
constexpr size_t kClosedLoopNoiseBytes = size_t(256) << 20;
constexpr uint32_t kLoopChunk = 16;

struct Profile {
  double ms[5] = {0, 0, 0, 0, 0};
  double n[5] = {0, 0, 0, 0, 0};
};

struct TimedLaunch {
  int kind;
  hipEvent_t a, b;
};

// Device side of the served form (the queue, admission and the request
// thread are served_core.h's): a batch's packed device block, its outputs in
// the slot's pinned staging, its completion event and its trace range.
struct HipServed {
  brmppi_ctx* ctx = nullptr;
  struct BatchState {
    Block mem;                      // descs + tiles + items + per-instance scratch
    size_t out_off = 0;             // offset of the packed outputs in the slot's pinned staging
    std::vector<size_t> out_pos;    // float offset of each request's [stats(4) | u(3T)]
    size_t out_floats = 0;
    hipEvent_t done_ev = nullptr;
    roctx_range_id_t range = 0;     // launch to completion
  };
  template <class B> int launch(B& b);
  template <class B> int query(B& b);
  template <class B> void retire(B& b);
  template <class B> void abandon(B& b);
  SlotState& controller(uint32_t id);
  bool fits(size_t bytes);
  template <class B> void on_launch(B& b) {
    b.state.range = roctxRangeStartA("brmppi batch");
  }
  template <class B> void on_complete(B& b) {
    roctxRangeStop(b.state.range);
  }
  void trace_push(const char* name) { roctxRangePushA(name); }
  void trace_pop() { roctxRangePop(); }
};

constexpr int kBuckets[5] = {0, 2, 8, 16, 32};
int bucket_index(int bucket) {
  for (int i = 0; i < 5; ++i)
    if (kBuckets[i] == bucket) return i;
  return 4;
}
// sample-count classes of the launch table: <= 2048, <= 8192, <= 32768, larger
int s_class(uint32_t S) { return S <= 2048 ? 0 : (S <= 8192 ? 1 : (S <= 32768 ? 2 : 3)); }

}  // namespace

struct brmppi_ctx {
  int device = 0;
  Arena arena;
  hipStream_t streams[4] = {nullptr, nullptr, nullptr, nullptr};
  uint32_t n_streams = 1;
  uint32_t flags = 0;
  int n_cu = 256;
  std::string tune_path;
  std::vector<Controller> ctrl;
  LaunchShape shape[5][4];      // plain-path table, tuned entries: [bucket index][S class]
  LaunchShape forced{0, 0};     // block 0 = not forced
  Block counters_blk;           // BatchCounters per stream + spare
  BatchCounters* counters = nullptr;
  uint32_t* drawn_ctr = nullptr;   // completion counters of k_rollout_drawn (zero again when it ends)

  // blocking-path scratch (cached; re-allocated only when a call needs more)
  Block scratch;
  // the device's static scratch (brmppi_solve_noalloc), its address on this
  // context's device
  char* static_scratch = nullptr;
  bool no_events = false;       // set while a no-alloc call enqueues: no HIP events are taken
  uint64_t scratch_grows = 0;
  Pinned pin;                   // blocking staging
  hipEvent_t loop_ev[2] = {nullptr, nullptr};   // closed loop: completion of each staging half
  // the last batched solve's plan (type-erased: defined with the batch code)
  std::shared_ptr<void> plan_cache;
  // graph cache for the batched form
  hipGraphExec_t graph_exec = nullptr;
  hipGraph_t graph = nullptr;
  std::vector<uint64_t> graph_key;
  // profiling
  Profile prof;
  std::vector<hipEvent_t> ev_pool;
  std::vector<TimedLaunch> pending_timing;

  // served form: the request queue and thread of served_core.h over HIP
  HipServed served_dev;
  ServedCore<HipServed> srv;
  std::mutex& mu = srv.mu;      // guards the whole context and every device enqueue
  Pinned slot_pin[4];

  // host resources (also on a failed create); device memory is the caller's
  ~brmppi_ctx() {
    pin.release();
    for (auto& p : slot_pin) p.release();
    for (auto& e : loop_ev) {
      if (e) (void)hipEventDestroy(e);
      e = nullptr;
    }
  }
};

namespace {

// Defaults of every tuning parameter (the paper's tuned values are
// unpublished): the Sec. V input bounds j in [-2, 2] m/s^3 and omega in
// [-0.9, 0.9] rad/s; a 4 m / 0.5 m / 10 m tractor-trailer with the hitch limit
// 0.7 - 0.05 v rad and a 1 m footprint disc; Ts = 0.05 s; sampling noise
// (1.0, 0.3, 0.5) for (j, omega, nu) and 0.2 for the auxiliary inputs; W the
// inverse sampling covariance, rho = 0.1; barrier rates starting at 0.5 within
// [-1, 1]; contouring weights Qc = Ql = 2, heading weights 1, effort 0.05,
// progress weight 0.5 toward 2 m/s; collision-penalty weight 1000; hitch QP
// with Q_h = W's input block and alpha_h = 0.5.
brmppi_params default_params() {
  brmppi_params P{};
  P.Ts = 0.05f; P.l1 = 4.0f; P.lh = 0.5f; P.l2 = 10.0f; P.dtheta_max = 0.7f; P.kappa = 0.05f; P.r_disc = 1.0f;
  P.Qc = 2.0f; P.Ql = 2.0f; P.Qth1 = 1.0f; P.Qth2 = 1.0f; P.R_j = 0.05f; P.R_w = 0.05f; P.mu = 0.5f;
  P.nu_bar = 2.0f;
  P.sigma_j = 1.0f; P.sigma_w = 0.3f; P.sigma_nu = 0.5f; P.sigma_a = 0.2f;
  P.W_j = (float)(1.0 / (1.0 * 1.0)); P.W_w = (float)(1.0 / (0.3 * 0.3));
  P.W_a = (float)(1.0 / (0.2 * 0.2)); P.rho = 0.1f;
  P.j_lo = -2.0f; P.j_hi = 2.0f; P.w_lo = -0.9f; P.w_hi = 0.9f;
  P.alpha0 = 0.5f; P.alpha_lo = -1.0f; P.alpha_hi = 1.0f;
  P.h_eps = 1e-5f; P.w_col = 1000.0f;
  P.qh_j = P.W_j; P.qh_w = P.W_w; P.alpha_h = 0.5f;
  P.n_disc_tractor = 1; P.disc_tractor[0] = 0.0f;   // the rear axle, eq. (16)
  P.n_disc_trailer = 0;
  return P;
}

// the parameters a problem runs with: its own, or its controller's
const brmppi_params& params_of(const brmppi_ctx* ctx, const brmppi_problem& p) {
  return p.params ? *p.params : ctx->ctrl[p.controller].params;
}

// ---------------------------------------------------------------------------
// validation
// ---------------------------------------------------------------------------
bool finite_params(const brmppi_params& p) {
  const float* f = reinterpret_cast<const float*>(&p);   // every float field precedes the disc counts
  for (size_t i = 0; i < offsetof(brmppi_params, n_disc_tractor) / sizeof(float); ++i)
    if (!std::isfinite(f[i])) return false;
  return true;
}

int validate_params(const brmppi_params& P) {
  if (!finite_params(P)) return fail(BRMPPI_EINVAL, "non-finite parameter");
  if (!(P.Ts > 0) || !(P.l1 > 0) || !(P.l2 > 0) || !(P.h_eps > 0))
    return fail(BRMPPI_EINVAL, "Ts, l1, l2 and h_eps must be positive");
  if (!(P.W_j + P.rho > 0) || !(P.W_w + P.rho > 0) || !(P.W_a + P.rho > 0) || P.rho < 0 || P.W_j < 0 ||
      P.W_w < 0 || P.W_a < 0)
    return fail(BRMPPI_EINVAL, "projection weights must be >= 0 with W + rho > 0");
  if (P.n_disc_tractor > BRMPPI_MAX_DISCS || P.n_disc_trailer > BRMPPI_MAX_DISCS || n_discs(P) < 1)
    return fail(BRMPPI_EINVAL, "footprint: 1..4 discs per body, at least one disc");
  return BRMPPI_OK;
}

int validate(brmppi_ctx* ctx, const brmppi_problem* p) {
  if (!ctx || !p) return fail(BRMPPI_EINVAL, "null context or problem");
  if (p->controller >= ctx->ctrl.size()) return fail(BRMPPI_EINVAL, "controller id out of range");
  if (p->S < 1 || p->S > BRMPPI_MAX_S) return fail(BRMPPI_EINVAL, "S out of range");
  if (p->T < 1 || p->T > BRMPPI_MAX_T) return fail(BRMPPI_EINVAL, "T out of range");
  if (p->n_obs > BRMPPI_MAX_OBS) return fail(BRMPPI_EINVAL, "too many obstacles");
  if (p->n_obs > 0 && !p->obs) return fail(BRMPPI_EINVAL, "obstacles pointer is NULL");
  if (p->flags & ~(BRMPPI_GUIDANCE_OFF | BRMPPI_HITCH_OFF | BRMPPI_X0_RESIDENT | BRMPPI_ADVANCE_PLANT |
                   BRMPPI_COLLISION_PENALTY | BRMPPI_HITCH_QP))
    return fail(BRMPPI_EINVAL, "unknown flags");
  if ((p->flags & BRMPPI_HITCH_QP) && !(p->flags & BRMPPI_ADVANCE_PLANT))
    return fail(BRMPPI_EINVAL, "BRMPPI_HITCH_QP acts on the plant step (BRMPPI_ADVANCE_PLANT)");
  if ((p->flags & BRMPPI_ADVANCE_PLANT) && !(p->flags & BRMPPI_X0_RESIDENT))
    return fail(BRMPPI_EINVAL, "BRMPPI_ADVANCE_PLANT needs BRMPPI_X0_RESIDENT");
  const brmppi_params& P = params_of(ctx, *p);
  if (int rc = validate_params(P)) return rc;
  if (!(p->lambda > 0) || !std::isfinite(p->lambda)) return fail(BRMPPI_EINVAL, "lambda must be positive");
  if ((p->flags & BRMPPI_HITCH_QP) && (!(P.qh_j > 0) || !(P.qh_w > 0) || !(P.alpha_h > 0)))
    return fail(BRMPPI_EINVAL, "BRMPPI_HITCH_QP needs qh_j, qh_w and alpha_h positive");
  if (!std::isfinite(p->t0)) return fail(BRMPPI_EINVAL, "t0 must be finite");
  if ((size_t)p->n_obs * n_discs(P) > BRMPPI_MAX_OBS)
    return fail(BRMPPI_EINVAL, "obstacles times footprint discs exceed BRMPPI_MAX_OBS");
  for (uint32_t i = 0; i < p->n_obs; ++i) {
    const brmppi_obstacle& o = p->obs[i];
    if (o.e != 2.0f && o.e != 4.0f) return fail(BRMPPI_EINVAL, "obstacle exponent e must be 2 or 4");
    const float v[8] = {o.cx, o.cy, o.mx, o.my, o.heading, o.e, o.vx, o.vy};
    for (float x : v)
      if (!std::isfinite(x)) return fail(BRMPPI_EINVAL, "non-finite obstacle field");
    if (!(o.mx + P.r_disc > 0) || !(o.my + P.r_disc > 0))
      return fail(BRMPPI_EINVAL, "inflated semi-axes must be positive");
  }
  const Controller& c = ctx->ctrl[p->controller];
  if (!c.path) return fail(BRMPPI_ESTATE, "controller has no path (brmppi_set_path)");
  if (!p->u_nom && c.warm_T != p->T)
    return fail(BRMPPI_ESTATE, "no resident warm start of length T for this controller");
  if ((p->flags & BRMPPI_X0_RESIDENT) && !c.plant_set)
    return fail(BRMPPI_ESTATE, "no resident plant state (brmppi_set_state)");
  return BRMPPI_OK;
}

// dynamic LDS of the fused epilogue for a plain launch, 0 when the tiles are
// not whole units or do not fit (k_reduce then reduces from HBM)
size_t fused_lds(const brmppi_problem& p, const LaunchShape& sh) {
  const uint32_t per_tile = sh.block / (uint32_t)variant_lanes(sh.variant);
  if (!fused_tile_ok(per_tile)) return 0;
  const size_t b = fused_lds_bytes(per_tile, p.T, (p.S + kWChunk - 1) / kWChunk);
  return b <= kFusedLdsMax ? b : 0;
}

size_t normals_bytes(const brmppi_ctx* ctx, const brmppi_problem& p) {
  return (size_t)normals_per_step(ctx, p) * p.T * round_up(p.S, 256) * sizeof(float);
}
size_t normals_limit(const brmppi_ctx* ctx) { return std::min(kMaxNoiseBytes, ctx->arena.size() / 2); }

// the shape that the caller forced or tuned, if any (block 0: none)
LaunchShape set_shape(const brmppi_ctx* ctx, const brmppi_problem& p) {
  if (ctx->forced.block) return ctx->forced;
  return ctx->shape[bucket_index(bucket_for(obstacle_rows(ctx, p), p.flags))][s_class(p.S)];
}

// Bytes of normals in the scratch that brmppi_solve_noalloc is stated to need: the
// same whichever launch draws them, so that a new default shape does not move the
// limit.
size_t stated_normals(const brmppi_ctx* ctx, const brmppi_problem& p) {
  const LaunchShape s = set_shape(ctx, p);
  const bool counted = s.block ? variant_pre(s.variant) : p.S <= ((p.flags & BRMPPI_GUIDANCE_OFF) ? 8192u : 32768u);
  const size_t n = normals_bytes(ctx, p);
  return counted && n <= normals_limit(ctx) ? n : 0;
}

// launch shape of a plain (single-instance) rollout
LaunchShape plain_shape(brmppi_ctx* ctx, const brmppi_problem& p) {
  const int bucket = bucket_for(obstacle_rows(ctx, p), p.flags);
  LaunchShape s = set_shape(ctx, p);
  const size_t noise = normals_bytes(ctx, p);
  if (s.block == 0)
    s = default_shape(bucket, p.S, noise, (p.flags & BRMPPI_COLLISION_PENALTY) != 0, footprint_is_rear_axle(params_of(ctx, p)));
  if (drawn_fits(ctx->n_cu, bucket, s, p.S, p.T, fused_lds(p, s))) s.variant = kDrawnVariant;
  if (variant_pre(s.variant) && noise > normals_limit(ctx))
    s.variant = variant_in_kernel(bucket);
  return s;
}

// (without normals: see Normals)
ScratchLayout plain_layout(const brmppi_ctx* ctx, const brmppi_problem& p) {
  const brmppi_problem* pp = &p;
  uint32_t rows = kRowsPerPass;
  reduce_rows(&pp, 1, ctx->n_cu, &rows);
  return scratch_layout(p.S, p.T, 0u, rows);
}

hipEvent_t take_event(brmppi_ctx* ctx) {
  if (!ctx->ev_pool.empty()) {
    hipEvent_t e = ctx->ev_pool.back();
    ctx->ev_pool.pop_back();
    return e;
  }
  // timing only (read after a stream sync): no system-scope fence at the
  // record, whose cache write-back and invalidation would otherwise land in
  // the measured interval and slow the next kernel
  hipEvent_t e = nullptr;
  if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) return nullptr;
  return e;
}

// launch with optional timing (kind: 0 rollout, 1 weights, 2 reduce, 3 plant, 4 noise)
template <typename F>
int timed(brmppi_ctx* ctx, hipStream_t st, int kind, F&& launch) {
  const bool prof = !ctx->no_events && ((ctx->flags & BRMPPI_CTX_PROFILE) != 0 ||
                    ((ctx->flags & BRMPPI_CTX_PROFILE_ROLLOUT) != 0 && (kind == 0 || kind == 4)));
  TimedLaunch tl{kind, nullptr, nullptr};
  if (prof) {
    tl.a = take_event(ctx);
    tl.b = take_event(ctx);
    if (tl.a) HIPCHK(hipEventRecord(tl.a, st));
  }
  HIPCHK(launch());
  if (prof && tl.b) {
    HIPCHK(hipEventRecord(tl.b, st));
    ctx->pending_timing.push_back(tl);
  }
  return 0;
}

// after a stream sync: fold recorded kernel timings into the profile
void collect_timing(brmppi_ctx* ctx) {
  for (auto& t : ctx->pending_timing) {
    float ms = 0.0f;
    if (t.a && t.b && hipEventElapsedTime(&ms, t.a, t.b) == hipSuccess) {
      ctx->prof.ms[t.kind] += ms;
      ctx->prof.n[t.kind] += 1.0;
    }
    if (t.a) ctx->ev_pool.push_back(t.a);
    if (t.b) ctx->ev_pool.push_back(t.b);
  }
  ctx->pending_timing.clear();
}

// the normals of `count` updates from the one of descriptor h on, buffers
// `stride` floats apart, and the upload of their inputs, in one launch
int enqueue_noise(brmppi_ctx* ctx, hipStream_t st, const SolveDesc& h, uint32_t count, size_t stride,
                  const Upload& up) {
  if (!h.noise) return fail(BRMPPI_EINVAL, "internal: noise buffer missing");
  const NoiseArgs a{h.noise, stride, (uint64_t)h.seed_hi << 32 | h.seed_lo, h.S_pad, h.n_normals, h.instance};
  return timed(ctx, st, 4, [&] { return launch_noise(a, count, h.T, up, st); });
}

// An update by k_rollout_drawn: its inputs as the launch's arguments, the nominal
// sequence among them when the caller gives one.
int enqueue_drawn(brmppi_ctx* ctx, hipStream_t st, SolveArgs& a, const float* u_nom, size_t lds) {
  if (u_nom) {
    a.d.u_nom_in = nullptr;
    std::memcpy(a.unom, u_nom, sizeof(float) * 3 * a.d.T);
  }
  const uint32_t grid = (a.d.S + kDrawnTile - 1) / kDrawnTile;
  const int rc = timed(ctx, st, 0, [&] { return launch_rollout_drawn((int)a.d.bucket, a, grid, lds, st); });
  // normals drawn apart from the rollout's lanes, in no time of their own
  if (!rc && !ctx->no_events && (ctx->flags & (BRMPPI_CTX_PROFILE | BRMPPI_CTX_PROFILE_ROLLOUT))) ctx->prof.n[4] += 1.0;
  return rc;
}

Upload upload(const char* src, char* dst, size_t bytes) { return Upload{src, dst, (bytes + 15) / 16}; }

// rollout + weights + reduce (+ plant) of one instance whose normals, if the
// shape reads them, are already in its noise buffer (or ordered before on st);
// lds > 0: the rollout reduces its own tiles (fused epilogue, no k_reduce)
int enqueue_rollout_reduce(brmppi_ctx* ctx, hipStream_t st, const SolveDesc* d_desc, const brmppi_problem& p,
                           const ScratchLayout& L, const LaunchShape& sh, size_t lds) {
  const int bucket = bucket_for(obstacle_rows(ctx, p), p.flags);
  const uint32_t per_tile = sh.block / variant_lanes(sh.variant);
  const uint32_t grid = (p.S + per_tile - 1) / per_tile;
  int rc = timed(ctx, st, 0, [&] {
    return launch_rollout(bucket, sh.variant, d_desc, grid, sh.block, lds, st);
  });
  if (rc || lds) return rc;
  const uint32_t nr = L.n_wchunk * L.n_rgroup;
  return timed(ctx, st, 1, [&] { return launch_reduce(d_desc, nullptr, nr, nullptr, nr, st); });
}

int ensure_scratch(brmppi_ctx* ctx, size_t bytes) {
  if (ctx->scratch.bytes >= bytes) return 0;
  if (ctx->scratch.ptr) ++ctx->scratch_grows;
  ctx->arena.release(ctx->scratch);
  ctx->scratch = ctx->arena.alloc(bytes);
  if (!ctx->scratch.ptr) return fail(BRMPPI_ENOMEM, "solve scratch does not fit in the arena");
  return 0;
}

// Room for the precomputed normals of a call: behind the first `used` bytes of the
// kept scratch where they fit, else in free memory of the arena, which no one else can
// take while the call holds the context's lock.  Nothing is kept, so that normals never
// take what a later batch or request could use.  take() fails where there is no room:
// the call then draws its normals in the rollout.
class Normals {
 public:
  explicit Normals(brmppi_ctx* ctx) : ctx_(ctx) {}
  ~Normals() {
    // a call that failed may have left work on its stream that still uses the memory
    if (lent_) (void)hipStreamSynchronize(ctx_->streams[0]);
  }
  Normals(const Normals&) = delete;
  Normals& operator=(const Normals&) = delete;
  char* take(size_t used, size_t bytes) {
    used = round_up(used, 256);
    if (ctx_->scratch.bytes >= used + bytes) return ctx_->scratch.ptr + used;
    char* p = ctx_->arena.lend(bytes);
    lent_ = p != nullptr;
    return p;
  }
  void idle() { lent_ = false; }   // the call's stream has been waited for

 private:
  brmppi_ctx* ctx_;
  bool lent_ = false;
};

// ---------------------------------------------------------------------------
// plain solve
// ---------------------------------------------------------------------------
// Costs of up to this size are written to pinned host memory by the rollout
// itself: the transfer runs while the samples do.
constexpr size_t kDirectCostBytes = size_t(1) << 20;
// Larger results come in pieces of this size through two halves of the pinned
// buffer: the device fills one while the host empties the other.
// (3001 applied sequences of 37 steps, 1.4 MB: 191 us for the update and its
// download; by a pitched copy to the caller's pageable memory 890 us).  The pitched
// copy's cost is by the row, so rows of a piece and longer are left to it (the update,
// its costs and sequences of 4 steps, pieces / pitched copy: 32768 samples 179 / 212 us,
// 50000 255 / 252, 65536 305 / 290, 130000 562 / 459, 300000 1330 / 1226).
constexpr size_t kPieceBytes = size_t(256) << 10;

// n_rows rows of `row` floats, `pitch` apart at src on the device, to dense rows at dst
int download_rows(brmppi_ctx* ctx, hipStream_t s, float* dst, size_t row, const char* src, size_t pitch, size_t n_rows,
                  const char* piece) {
  if (row * sizeof(float) >= kPieceBytes) {
    HIPCHK(hipMemcpy2D(dst, row * sizeof(float), src, pitch * sizeof(float), row * sizeof(float), n_rows, hipMemcpyDeviceToHost));
    return 0;
  }
  constexpr size_t kPiece = kPieceBytes / sizeof(float);
  const size_t total = (n_rows - 1) * pitch + row;
  const size_t n_pieces = (total + kPiece - 1) / kPiece;
  auto half = [&](size_t k) { return const_cast<char*>(piece) + (k % 2) * kPieceBytes; };
  auto fetch = [&](size_t k) -> int {
    const size_t a = k * kPiece, n = std::min(kPiece, total - a);
    HIPCHK(hipMemcpyAsync(half(k), src + a * sizeof(float), n * sizeof(float), hipMemcpyDeviceToHost, s));
    HIPCHK(hipEventRecord(ctx->loop_ev[k % 2], s));
    return 0;
  };
  if (int rc = fetch(0)) return rc;
  for (size_t k = 0; k < n_pieces; ++k) {
    if (k + 1 < n_pieces)
      if (int rc = fetch(k + 1)) return rc;
    HIPCHK(hipEventSynchronize(ctx->loop_ev[k % 2]));
    const float* got = reinterpret_cast<const float*>(half(k));
    const size_t a = k * kPiece, b = std::min(total, a + kPiece);
    for (size_t at = a; at < b;) {
      const size_t r = at / pitch, c = at - r * pitch;   // c past the row: its padding
      const size_t end = std::min(b, r * pitch + (c < row ? row : pitch));
      if (c < row) std::memcpy(dst + r * row + c, got + (at - a), (end - at) * sizeof(float));
      at = end;
    }
  }
  return 0;
}

// fixed != nullptr: the scratch is that block of fixed_bytes (the device's
// static scratch), and the call allocates nothing: no arena block, no pinned
// staging growth, no HIP events (sizes beyond either are ENOMEM)
int solve_locked(brmppi_ctx* ctx, const brmppi_problem* p, const brmppi_outputs* out, brmppi_stats* st,
                 char* fixed = nullptr, size_t fixed_bytes = 0) {
  const auto t_start = Clock::now();
  int rc = validate(ctx, p);
  if (rc) return rc;
  if (!out || !out->u_out) return fail(BRMPPI_EINVAL, "u_out is NULL");
  Controller& c = ctx->ctrl[p->controller];
  LaunchShape sh = plain_shape(ctx, *p);
  const ScratchLayout L = plain_layout(ctx, *p);
  // device: [scratch | input block]
  const bool drawn = sh.variant == kDrawnVariant;   // the inputs are the launch's arguments
  const InputBlock IB = drawn ? InputBlock{} : input_block(p->T, p->u_nom != nullptr, L.n_wchunk);
  const size_t in_off = L.bytes;
  const size_t need = in_off + round_up(IB.bytes, 256);
  char* base;
  float* noise = nullptr;
  Normals normals(ctx);
  if (fixed) {
    const size_t asked = L.bytes + round_up(input_block(p->T, p->u_nom != nullptr, L.n_wchunk).bytes, 256) +
                         stated_normals(ctx, *p);
    if (asked > fixed_bytes)
      return fail(BRMPPI_ENOMEM, "the update needs " + std::to_string(asked) + " bytes of scratch, more than the " +
                                     std::to_string(fixed_bytes) + " of the static scratch");
    base = fixed;
    if (variant_pre(sh.variant)) {
      if (need + normals_bytes(ctx, *p) <= fixed_bytes) noise = reinterpret_cast<float*>(fixed + need);
      else sh.variant = variant_in_kernel(bucket_for(obstacle_rows(ctx, *p), p->flags));
    }
  } else {
    if ((rc = ensure_scratch(ctx, need))) return rc;
    base = ctx->scratch.ptr;
    if (variant_pre(sh.variant)) {
      noise = reinterpret_cast<float*>(normals.take(need, normals_bytes(ctx, *p)));
      if (!noise) sh.variant = variant_in_kernel(bucket_for(obstacle_rows(ctx, *p), p->flags));
    }
  }
  const size_t lds = fused_lds(*p, sh);
  // pinned: [input block | stats, sequence | costs | two pieces of the sequences];
  // the kernels read the first and write the next two themselves
  const size_t out_off = round_up(IB.bytes, 256);
  const size_t J_off = out_off + round_up((4 + 3 * (size_t)p->T) * sizeof(float), 256);
  const bool J_direct = out->J_out && lds > 0 && p->S * sizeof(float) <= kDirectCostBytes;
  const size_t piece_off = J_off + (J_direct ? round_up(p->S * sizeof(float), 256) : 0);
  const bool rows_out = out->useq_out || (out->J_out && !J_direct);
  const size_t pin_need = piece_off + (rows_out ? 2 * kPieceBytes : 0);
  if (fixed) {
    if (pin_need > ctx->pin.bytes) return fail(BRMPPI_ENOMEM, "inputs larger than the pinned staging buffer");
  } else if ((rc = ctx->pin.ensure(pin_need))) {
    return rc;
  }
  SolveDesc* d_desc = reinterpret_cast<SolveDesc*>(base + in_off);
  hipStream_t s = ctx->streams[0];
  char* pin = ctx->pin.ptr;
  SolveDesc* h_desc = reinterpret_cast<SolveDesc*>(pin);
  float* pin_out = reinterpret_cast<float*>(pin + out_off);
  float* pin_J = reinterpret_cast<float*>(pin + J_off);

  ctx->no_events = fixed != nullptr;
  if (drawn) {
    SolveArgs a;
    fill_desc(a.d, *p, c, L, base, 0, nullptr, ctx->drawn_ctr, pin_out, true, out->useq_out != nullptr);
    if (J_direct) a.d.J = pin_J;
    rc = enqueue_drawn(ctx, s, a, p->u_nom, lds);
  } else {
    fill_desc(*h_desc, *p, c, L, base, 0, reinterpret_cast<const float*>(base + in_off + IB.unom),
              reinterpret_cast<uint32_t*>(base + in_off + IB.counter), pin_out, lds > 0, out->useq_out != nullptr);
    h_desc->noise = noise;
    if (J_direct) h_desc->J = pin_J;
    std::memset(pin + IB.counter, 0, IB.unom - IB.counter);
    if (p->u_nom) std::memcpy(pin + IB.unom, p->u_nom, sizeof(float) * 3 * p->T);
    const Upload up = upload(pin, base + in_off, IB.bytes);
    if (variant_pre(sh.variant)) {
      rc = enqueue_noise(ctx, s, *h_desc, 1, 0, up);
    } else {
      const hipError_t e = launch_upload(up, s);
      rc = e == hipSuccess ? 0 : fail(BRMPPI_EDEVICE, std::string("upload: ") + hipGetErrorString(e));
    }
    if (!rc) rc = enqueue_rollout_reduce(ctx, s, d_desc, *p, L, sh, lds);
  }
  ctx->no_events = false;
  if (rc) {
    (void)hipStreamSynchronize(s);   // nothing of this call may still run on the scratch
    return rc;
  }
  HIPCHK(hipStreamSynchronize(s));
  normals.idle();
  collect_timing(ctx);
  if (J_direct) std::memcpy(out->J_out, pin_J, sizeof(float) * p->S);
  else if (out->J_out && (rc = download_rows(ctx, s, out->J_out, p->S, base + L.off_J, L.S_pad, 1, pin + piece_off))) return rc;
  if (out->useq_out && (rc = download_rows(ctx, s, out->useq_out, p->S, base + L.off_ustar, L.S_pad, 3 * (size_t)p->T,
                                           pin + piece_off)))
    return rc;
  const int status = (int)pin_out[3];
  std::memcpy(out->u_out, pin_out + 4, sizeof(float) * 3 * p->T);
  if (status == BRMPPI_OK) c.warm_T = p->T;   // the shifted result is resident
  if (st) {
    st->J_min = pin_out[0];
    st->Z = pin_out[1];
    st->ess = pin_out[2];
    st->status = status;
    st->latency_us = std::chrono::duration<double, std::micro>(Clock::now() - t_start).count();
  }
  if (status != BRMPPI_OK) return fail(status, "every rollout cost was non-finite");
  return BRMPPI_OK;
}

// ---------------------------------------------------------------------------
// batched solve: descriptor table + tile list + work lists, persistent kernels
// ---------------------------------------------------------------------------
struct BatchPlan {
  std::vector<SolveDesc> descs;
  std::vector<Tile> tiles;
  std::vector<Item> ritems;
  std::vector<ScratchLayout> layouts;
  std::vector<size_t> scratch_off;   // offset of each instance's scratch inside the block
  std::vector<size_t> unom_off;      // offset of each caller nominal sequence (header), or 0
  std::vector<size_t> out_pos;       // float offset of each [stats(4) | u_new(3T)] in the outputs
  // block layout: header [descs | tiles | ritems | nominals | counters]
  // (one upload), then every instance's scratch; the outputs go to pinned memory
  size_t off_descs = 0, off_tiles = 0, off_ritems = 0, off_counters = 0, header_bytes = 0;
  size_t out_floats = 0, total = 0;
  uint32_t block = 256;              // of the rollout launch
  bool guided = false;               // some instance is
};

// samples of a tile of this instance in a batched launch of `block` threads
uint32_t batch_tile(const brmppi_ctx* ctx, const brmppi_problem& p, uint32_t block) {
  return block / (uint32_t)variant_lanes(variant_in_kernel(bucket_for(obstacle_rows(ctx, p), p.flags)));
}

void plan_layout(brmppi_ctx* ctx, const brmppi_problem* const* ps, uint32_t n, BatchPlan& bp) {
  bp.layouts.resize(n);
  bp.block = ctx->forced.block ? ctx->forced.block : 256;
  bp.guided = std::any_of(ps, ps + n, [](const brmppi_problem* p) { return !(p->flags & BRMPPI_GUIDANCE_OFF); });
  size_t n_tiles = 0, n_r = 0;
  std::vector<uint32_t> rows_item(n);
  reduce_rows(ps, n, ctx->n_cu, rows_item.data());
  for (uint32_t i = 0; i < n; ++i) {
    bp.layouts[i] = batch_scratch(ps[i]->S, ps[i]->T, rows_item[i]);
    const uint32_t per = batch_tile(ctx, *ps[i], bp.block);
    n_tiles += (ps[i]->S + per - 1) / per;
    n_r += (size_t)bp.layouts[i].n_wchunk * bp.layouts[i].n_rgroup;
  }
  size_t o = 0;
  bp.off_descs = o;
  o = round_up(o + sizeof(SolveDesc) * n, 256);
  bp.off_tiles = o;
  o = round_up(o + sizeof(Tile) * n_tiles, 256);
  bp.off_ritems = o;
  o = round_up(o + sizeof(Item) * n_r, 256);
  // caller-supplied nominal sequences travel with the header
  bp.unom_off.assign(n, 0);
  for (uint32_t i = 0; i < n; ++i) {
    if (!ps[i]->u_nom) continue;
    bp.unom_off[i] = o;
    o = round_up(o + sizeof(float) * 3 * ps[i]->T, 256);
  }
  bp.off_counters = o;                        // uploaded as zeros
  o = round_up(o + sizeof(uint32_t) * n, 256);
  bp.header_bytes = o;
  bp.out_pos.resize(n);
  size_t nf = 0;
  for (uint32_t i = 0; i < n; ++i) {
    bp.out_pos[i] = nf;
    nf += 4 + 3 * (size_t)ps[i]->T;
  }
  bp.out_floats = nf;
  bp.scratch_off.resize(n);
  for (uint32_t i = 0; i < n; ++i) {
    bp.scratch_off[i] = o;
    o += bp.layouts[i].bytes;
  }
  bp.total = o;
}

// the descriptors of a batch (every call: they hold its inputs)
void plan_descs(brmppi_ctx* ctx, const brmppi_problem* const* ps, uint32_t n, char* base, BatchPlan& bp) {
  bp.descs.resize(n);
  for (uint32_t i = 0; i < n; ++i) {
    const brmppi_problem& p = *ps[i];
    const float* unom_dev = p.u_nom ? reinterpret_cast<const float*>(base + bp.unom_off[i]) : nullptr;
    uint32_t* counter = reinterpret_cast<uint32_t*>(base + bp.off_counters) + i;
    fill_desc(bp.descs[i], p, ctx->ctrl[p.controller], bp.layouts[i], base + bp.scratch_off[i], 0, unom_dev,
              counter, nullptr);   // the outputs' place follows when it is staged
  }
}

// the tiles and reduce items of a batch, in launch order (they depend only on
// its composition: see batch_signature)
void plan_work(brmppi_ctx* ctx, const brmppi_problem* const* ps, uint32_t n, BatchPlan& bp) {
  bp.tiles.clear();
  bp.ritems.clear();
  struct TC {
    double cost;
    Tile t;
  };
  std::vector<TC> tc;
  for (uint32_t i = 0; i < n; ++i) {
    const brmppi_problem& p = *ps[i];
    const uint32_t per = batch_tile(ctx, p, bp.block);
    // instructions of a tile's wave, about: 150 a step, and its share of the
    // rows (45 each) and of the Philox blocks of four normals (100 each)
    const double share = (double)per / bp.block;
    const bool guided = !(p.flags & BRMPPI_GUIDANCE_OFF);
    const double rows = guided ? 2.0 + obstacle_rows(ctx, p) : 0.0;
    const double cost = (double)p.T * (150.0 + share * (45.0 * rows + 25.0 * (3.0 + rows)));
    for (uint32_t s0 = 0; s0 < p.S; s0 += per) tc.push_back({cost, Tile{i, s0}});
    for (uint32_t k = 0; k < bp.layouts[i].n_wchunk * bp.layouts[i].n_rgroup; ++k) bp.ritems.push_back(Item{i, k});
  }
  // tiles longest first (stable: instance order breaks ties)
  std::stable_sort(tc.begin(), tc.end(), [](const TC& a, const TC& b) { return a.cost > b.cost; });
  bp.tiles.reserve(tc.size());
  for (const TC& c : tc) bp.tiles.push_back(c.t);
  // reduce items longest first (stable), for when they outnumber the blocks
  auto item_rows = [&](const Item& it) {
    const ScratchLayout& L = bp.layouts[it.inst];
    const uint32_t r0 = (it.idx % L.n_rgroup) * L.rows_item;
    return std::min(L.rows_item, 3 * ps[it.inst]->T - r0);
  };
  std::stable_sort(bp.ritems.begin(), bp.ritems.end(),
                   [&](const Item& a, const Item& b) { return item_rows(a) > item_rows(b); });
}

void plan_fill(brmppi_ctx* ctx, const brmppi_problem* const* ps, uint32_t n, char* base, BatchPlan& bp) {
  plan_descs(ctx, ps, n, base, bp);
  plan_work(ctx, ps, n, bp);
}

// What plan_layout and plan_work depend on: the launch table and, per
// instance, S, T, the constraint rows, the flags and whether a nominal
// sequence comes with the call.  A batched solve with the signature of the
// previous one reuses its layout, tiles and reduce items (a control loop
// that re-solves the same set of problems every tick), and only refills the
// descriptors.
void batch_signature(brmppi_ctx* ctx, const brmppi_problem* const* ps, uint32_t n, std::vector<uint64_t>& sig) {
  sig.clear();
  sig.reserve(8 + 3 * (size_t)n);
  sig.push_back(n);
  sig.push_back(ctx->forced.block);
  for (uint32_t i = 0; i < n; ++i) {
    sig.push_back(((uint64_t)ps[i]->S << 32) | ps[i]->T);
    sig.push_back(((uint64_t)obstacle_rows(ctx, *ps[i]) << 32) | ps[i]->flags);
    sig.push_back(ps[i]->u_nom ? 1u : 0u);
  }
}

struct BatchPlanCache {
  std::vector<uint64_t> sig;   // empty: no valid plan
  BatchPlan bp;
};

BatchPlanCache& plan_cache(brmppi_ctx* ctx) {
  if (!ctx->plan_cache)
    ctx->plan_cache = std::shared_ptr<void>(new BatchPlanCache, [](void* q) { delete static_cast<BatchPlanCache*>(q); });
  return *static_cast<BatchPlanCache*>(ctx->plan_cache.get());
}

uint32_t persistent_grid(brmppi_ctx* ctx, uint32_t block, bool guided, size_t n_tiles) {
  const int per_cu = rollout_batch_blocks_per_cu(block, guided);
  const size_t g = (size_t)ctx->n_cu * (size_t)std::max(per_cu, 1);
  return (uint32_t)std::max<size_t>(1, std::min(g, n_tiles));
}

// a persistent rollout over every instance's tiles, then the persistent reduce
// (weights, update, shift, plant steps) over every instance's items (a launch's
// work counters are zero again when it ends)
int enqueue_batch(brmppi_ctx* ctx, hipStream_t st, char* base, const BatchPlan& bp, BatchCounters* ctr,
                  bool timing) {
  const SolveDesc* descs = reinterpret_cast<const SolveDesc*>(base + bp.off_descs);
  const Tile* tiles = reinterpret_cast<const Tile*>(base + bp.off_tiles);
  const Item* ri = reinterpret_cast<const Item*>(base + bp.off_ritems);
  const uint32_t nr = (uint32_t)bp.ritems.size();
  const uint32_t g_r = std::max<uint32_t>(1, std::min<uint32_t>(nr, (uint32_t)ctx->n_cu * 8));
  const uint32_t nt = (uint32_t)bp.tiles.size();
  const uint32_t g_roll = persistent_grid(ctx, bp.block, bp.guided, nt);
  auto L0 = [&] { return launch_rollout_batch(descs, tiles, nt, ctr, g_roll, bp.block, bp.guided, st); };
  if (timing) {
    if (int rc = timed(ctx, st, 0, L0)) return rc;
  } else {
    HIPCHK(L0());
  }
  auto L1 = [&] { return launch_reduce(descs, ri, nr, ctr, g_r, st); };
  if (timing) return timed(ctx, st, 1, L1);
  HIPCHK(L1());
  return 0;
}

// write the header of a batch into pinned memory (uploaded to the batch's block
// by one launch); the outputs follow it there, written by the kernels
void stage_batch(const BatchPlan& bp, const brmppi_problem* const* ps, char* pin) {
  std::memcpy(pin + bp.off_descs, bp.descs.data(), sizeof(SolveDesc) * bp.descs.size());
  std::memcpy(pin + bp.off_tiles, bp.tiles.data(), sizeof(Tile) * bp.tiles.size());
  std::memcpy(pin + bp.off_ritems, bp.ritems.data(), sizeof(Item) * bp.ritems.size());
  float* outs = reinterpret_cast<float*>(pin + bp.header_bytes);
  for (size_t i = 0; i < bp.descs.size(); ++i) {
    SolveDesc& d = reinterpret_cast<SolveDesc*>(pin + bp.off_descs)[i];
    d.stats = outs + bp.out_pos[i];
    d.u_new = d.stats + 4;
  }
  for (size_t i = 0; i < bp.descs.size(); ++i)
    if (ps[i]->u_nom) std::memcpy(pin + bp.unom_off[i], ps[i]->u_nom, sizeof(float) * 3 * ps[i]->T);
  std::memset(pin + bp.off_counters, 0, bp.header_bytes - bp.off_counters);
}

// enqueue the upload and the kernels (or a graph of them) of a batch whose block
// starts at `base`; `pin` holds header_bytes + out_floats floats
int run_batch(brmppi_ctx* ctx, hipStream_t s, char* base, const BatchPlan& bp, BatchCounters* ctr, char* pin,
              bool use_graph);

void drop_graph(brmppi_ctx* ctx) {
  if (ctx->graph_exec) (void)hipGraphExecDestroy(ctx->graph_exec);
  if (ctx->graph) (void)hipGraphDestroy(ctx->graph);
  ctx->graph_exec = nullptr;
  ctx->graph = nullptr;
  ctx->graph_key.clear();
}

int run_batch(brmppi_ctx* ctx, hipStream_t s, char* base, const BatchPlan& bp, BatchCounters* ctr, char* pin,
              bool use_graph) {
  HIPCHK(launch_upload(upload(pin, base, bp.header_bytes), s));
  int rc;
  if (!use_graph) {
    if ((rc = enqueue_batch(ctx, s, base, bp, ctr, true))) return rc;
  } else {
    // the captured launches bake in every pointer and count: key on them
    std::vector<uint64_t> key = {(uint64_t)(uintptr_t)base, bp.tiles.size(), bp.ritems.size(),
                                 (uint64_t)(uintptr_t)s, bp.descs.size(), (uint64_t)(uintptr_t)ctr, bp.block, bp.guided};
    if (key != ctx->graph_key || !ctx->graph_exec) {
      drop_graph(ctx);
      HIPCHK(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
      rc = enqueue_batch(ctx, s, base, bp, ctr, false);
      hipGraph_t g = nullptr;
      hipError_t e = hipStreamEndCapture(s, &g);
      if (rc) {
        if (g) (void)hipGraphDestroy(g);
        return rc;
      }
      if (e != hipSuccess) return fail(BRMPPI_EDEVICE, std::string("graph capture: ") + hipGetErrorString(e));
      ctx->graph = g;
      HIPCHK(hipGraphInstantiate(&ctx->graph_exec, g, nullptr, nullptr, 0));
      ctx->graph_key = key;
    }
    HIPCHK(hipGraphLaunch(ctx->graph_exec, s));
  }
  return 0;
}

int solve_batch_locked(brmppi_ctx* ctx, const brmppi_problem* probs, uint32_t n, float* const* u_outs,
                       brmppi_stats* stats) {
  const auto t_start = Clock::now();
  if (!probs || !u_outs || n == 0 || n > BRMPPI_MAX_BATCH) return fail(BRMPPI_EINVAL, "bad batch arguments");
  std::vector<const brmppi_problem*> ps(n);
  std::vector<uint8_t> seen(ctx->ctrl.size(), 0);
  for (uint32_t i = 0; i < n; ++i) {
    int rc = validate(ctx, &probs[i]);
    if (rc) return fail(rc, "instance " + std::to_string(i) + ": " + g_err);
    if (!u_outs[i]) return fail(BRMPPI_EINVAL, "u_outs[i] is NULL");
    if (seen[probs[i].controller]) return fail(BRMPPI_EINVAL, "a controller appears twice in one batch");
    seen[probs[i].controller] = 1;
    ps[i] = &probs[i];
  }
  BatchPlanCache& pc = plan_cache(ctx);
  std::vector<uint64_t> sig;
  batch_signature(ctx, ps.data(), n, sig);
  const bool same = !pc.sig.empty() && sig == pc.sig;
  if (!same) {
    pc.sig.clear();
    pc.bp = BatchPlan{};
    plan_layout(ctx, ps.data(), n, pc.bp);
  }
  BatchPlan& bp = pc.bp;
  int rc;
  if ((rc = ensure_scratch(ctx, bp.total))) return rc;
  char* base = ctx->scratch.ptr;
  plan_descs(ctx, ps.data(), n, base, bp);
  if (!same) {
    plan_work(ctx, ps.data(), n, bp);
    pc.sig = std::move(sig);
  }
  hipStream_t s = ctx->streams[0];
  if ((rc = ctx->pin.ensure(bp.header_bytes + bp.out_floats * sizeof(float)))) return rc;
  char* pin = ctx->pin.ptr;
  stage_batch(bp, ps.data(), pin);
  const bool prof = (ctx->flags & (BRMPPI_CTX_PROFILE | BRMPPI_CTX_PROFILE_ROLLOUT)) != 0;
  if ((rc = run_batch(ctx, s, base, bp, ctx->counters, pin, !prof))) return rc;
  HIPCHK(hipStreamSynchronize(s));
  collect_timing(ctx);
  const float* pout = reinterpret_cast<const float*>(pin + bp.header_bytes);
  const double lat = std::chrono::duration<double, std::micro>(Clock::now() - t_start).count();
  int worst = BRMPPI_OK;
  for (uint32_t i = 0; i < n; ++i) {
    const float* o = pout + bp.out_pos[i];
    const int status = (int)o[3];
    std::memcpy(u_outs[i], o + 4, sizeof(float) * 3 * ps[i]->T);
    Controller& c = ctx->ctrl[ps[i]->controller];
    if (status == BRMPPI_OK) c.warm_T = ps[i]->T;
    if (stats) {
      stats[i].J_min = o[0];
      stats[i].Z = o[1];
      stats[i].ess = o[2];
      stats[i].status = status;
      stats[i].latency_us = lat;
    }
    if (status != BRMPPI_OK) worst = status;
  }
  if (worst != BRMPPI_OK) return fail(worst, "an instance had only non-finite costs");
  return BRMPPI_OK;
}

// ---------------------------------------------------------------------------
// closed loop on the device
// ---------------------------------------------------------------------------
int closed_loop_locked(brmppi_ctx* ctx, const brmppi_problem* p0, uint32_t n_up, double* x_out,
                       float* u_applied) {
  if (!p0 || n_up == 0) return fail(BRMPPI_EINVAL, "bad closed-loop arguments");
  if (p0->controller >= ctx->ctrl.size()) return fail(BRMPPI_EINVAL, "controller id out of range");
  Controller& c = ctx->ctrl[p0->controller];
  brmppi_problem p = *p0;
  if (!p.params) p.params = &c.params;
  const bool resume = (p.flags & BRMPPI_X0_RESIDENT) != 0;
  if (!resume) {
    if (!c.plant) return fail(BRMPPI_ESTATE, "controller has no path (brmppi_set_path)");
    for (int k = 0; k < 8; ++k)
      if (!std::isfinite(p.x0[k])) return fail(BRMPPI_EINVAL, "non-finite x0");
  }
  const bool plant_was_set = c.plant_set;
  if (!resume) c.plant_set = true;  // provisional (the caller's x0 is uploaded below), for validate()
  p.flags |= BRMPPI_X0_RESIDENT | BRMPPI_ADVANCE_PLANT;
  int rc = validate(ctx, &p);
  c.plant_set = plant_was_set;
  if (rc) return rc;
  LaunchShape sh = plain_shape(ctx, p);
  const ScratchLayout L = plain_layout(ctx, p);
  // The updates run in chunks of C: one descriptor upload per chunk and, when
  // the launch shape reads precomputed normals, one noise launch per chunk
  // (slot i of a chunk-sized noise region for its i-th update).  Descriptors
  // and logs go through two staging halves used in turn, so the host prepares
  // chunk j + 2 only once chunk j has completed and the device never waits
  // for the host.  Nothing here depends on n_up: a loop of any length reuses
  // the scratch and staging of a shorter one.  (Drawing the next chunk's
  // normals on a second stream while a chunk runs was measured slower: the
  // noise waves delay the rollout's, each of which is on the critical path of
  // its update.)
  const bool drawn = sh.variant == kDrawnVariant;   // the inputs are each launch's arguments
  const size_t noise_bytes = round_up(normals_bytes(ctx, p), 256);
  bool pre = variant_pre(sh.variant);
  uint32_t C = kLoopChunk;
  if (pre) {
    const size_t cap = std::min(kClosedLoopNoiseBytes, ctx->arena.size() / 2);
    C = (uint32_t)std::max<size_t>(1, std::min<size_t>(kLoopChunk, cap / noise_bytes));
  }
  const bool logs = x_out || u_applied;
  const size_t desc_bytes = round_up(sizeof(SolveDesc), 256);
  const size_t unom_bytes = p.u_nom ? sizeof(float) * 3 * p.T : 0;
  const size_t half_bytes = desc_bytes * C + round_up(sizeof(double) * kLogRecord * C, 256);
  // device: [scratch | counters (zero) | nominal | half 0 | half 1], and the normals of C updates
  // pinned: [counters | nominal | half 0 | half 1 | start state]; a half holds
  // the chunk's descriptors, then its plant states and applied inputs
  const size_t ctr_rel = 0;
  const size_t unom_rel = counter_bytes(L.n_wchunk);
  const size_t head_bytes = unom_rel + unom_bytes;
  const size_t half_rel = round_up(head_bytes, 256);
  const size_t x0_rel = half_rel + 2 * half_bytes;
  const size_t in_off = L.bytes;
  const size_t need = in_off + x0_rel;
  if ((rc = ensure_scratch(ctx, need))) return rc;
  if ((rc = ctx->pin.ensure(x0_rel + 256))) return rc;
  Normals normals(ctx);
  char* noise = nullptr;
  // the chunk's normals: of fewer updates where there is no room for all (the halves
  // keep their size), at the least of one
  if (pre) {
    const uint32_t most = C;
    while (!(noise = normals.take(need, C * noise_bytes)) && C > 1) C /= 2;
    if (!noise) {
      pre = false;
      C = most;
      sh.variant = variant_in_kernel(bucket_for(obstacle_rows(ctx, p), p.flags));
    }
  }
  const size_t lds = fused_lds(p, sh);
  char* base = ctx->scratch.ptr;
  char* pin = ctx->pin.ptr;
  hipStream_t s = ctx->streams[0];
  uint32_t* d_ctr = reinterpret_cast<uint32_t*>(base + in_off + ctr_rel);
  const float* d_unom = reinterpret_cast<const float*>(base + in_off + unom_rel);
  float* d_out = reinterpret_cast<float*>(base + L.off_out);
  auto half_dev = [&](int h) { return base + in_off + half_rel + h * half_bytes; };
  auto half_pin = [&](int h) { return pin + half_rel + h * half_bytes; };

  std::memset(pin + ctr_rel, 0, unom_rel - ctr_rel);
  if (p.u_nom) std::memcpy(pin + unom_rel, p.u_nom, unom_bytes);
  double* pin_x0 = reinterpret_cast<double*>(pin + x0_rel);
  if (!resume) {
    for (int k = 0; k < 8; ++k) pin_x0[k] = (double)p0->x0[k];
    HIPCHK(hipMemcpyAsync(c.plant, pin_x0, sizeof(double) * 8, hipMemcpyHostToDevice, s));
  } else if (x_out) {
    HIPCHK(hipMemcpyAsync(pin_x0, c.plant, sizeof(double) * 8, hipMemcpyDeviceToHost, s));
  }
  const uint32_t n_chunks = (n_up + C - 1) / C;
  // copy the logs of chunk j (complete) from its staging half to the caller
  auto take_logs = [&](uint32_t j) {
    const char* hp = half_pin((int)(j % 2));
    const uint32_t k0 = j * C, cnt = std::min(C, n_up - k0);
    const double* rec = reinterpret_cast<const double*>(hp + desc_bytes * C);
    for (uint32_t i = 0; i < cnt; ++i, rec += kLogRecord) {
      if (x_out) std::memcpy(x_out + 8 * (size_t)(k0 + i + 1), rec, sizeof(double) * 8);
      if (u_applied) std::memcpy(u_applied + 3 * (size_t)(k0 + i), rec + 8, sizeof(float) * 3);
    }
  };
  for (uint32_t j = 0; j < n_chunks; ++j) {
    const int h = (int)(j % 2);
    if (j >= 2) {
      HIPCHK(hipEventSynchronize(ctx->loop_ev[h]));
      if (logs) take_logs(j - 2);
    }
    const uint32_t k0 = j * C, cnt = std::min(C, n_up - k0);
    char* hp = half_pin(h);
    char* hd = half_dev(h);
    if (drawn) {
      for (uint32_t i = 0; i < cnt; ++i) {
        SolveArgs a;
        fill_desc(a.d, p, c, L, base, k0 + i, nullptr, ctx->drawn_ctr, d_out, true, false);
        if (logs) a.d.log = reinterpret_cast<double*>(hd + desc_bytes * C) + kLogRecord * i;
        if ((rc = enqueue_drawn(ctx, s, a, k0 + i == 0 ? p.u_nom : nullptr, lds))) return rc;
      }
    }
    for (uint32_t i = 0; i < cnt && !drawn; ++i) {
      const uint32_t k = k0 + i;
      SolveDesc* d = reinterpret_cast<SolveDesc*>(hp + desc_bytes * i);
      // only the first update reads the caller's sequence; later ones the shifted result
      fill_desc(*d, p, c, L, base, k, (k == 0 && p.u_nom) ? d_unom : nullptr, d_ctr, d_out, lds > 0, false);
      if (pre) d->noise = reinterpret_cast<float*>(noise + i * noise_bytes);
      // the update's last block writes the log (two device copies an update
      // took 2.6 us of it)
      if (logs) d->log = reinterpret_cast<double*>(hd + desc_bytes * C) + kLogRecord * i;
    }
    // the chunk's descriptors, with the first chunk the head before them
    const size_t head = j == 0 ? half_rel : 0;
    const Upload up = upload(hp - head, hd - head, head + desc_bytes * cnt);
    if (drawn) {
      // nothing to upload
    } else if (pre) {
      const SolveDesc& first = *reinterpret_cast<const SolveDesc*>(hp);
      if ((rc = enqueue_noise(ctx, s, first, cnt, noise_bytes / sizeof(float), up))) return rc;
    } else {
      HIPCHK(launch_upload(up, s));
    }
    for (uint32_t i = 0; i < cnt && !drawn; ++i)   // each with its plant step
      if ((rc = enqueue_rollout_reduce(ctx, s, reinterpret_cast<const SolveDesc*>(hd + desc_bytes * i), p, L, sh, lds)))
        return rc;
    if (logs)
      HIPCHK(hipMemcpyAsync(hp + desc_bytes * C, hd + desc_bytes * C, sizeof(double) * kLogRecord * cnt,
                            hipMemcpyDeviceToHost, s));
    HIPCHK(hipEventRecord(ctx->loop_ev[h], s));
  }
  HIPCHK(hipStreamSynchronize(s));
  normals.idle();
  collect_timing(ctx);
  if (logs) {
    for (uint32_t j = n_chunks >= 2 ? n_chunks - 2 : 0; j < n_chunks; ++j) take_logs(j);
    if (x_out) std::memcpy(x_out, pin_x0, sizeof(double) * 8);
  }
  c.plant_set = true;
  c.warm_T = p.T;
  return BRMPPI_OK;
}

// ---------------------------------------------------------------------------
// served form
// ---------------------------------------------------------------------------
// launch one batch of admitted requests on stream slot b.slot (ctx->mu held)
template <class B>
int HipServed::launch(B& b) {
  const uint32_t n = (uint32_t)b.reqs.size();
  std::vector<const brmppi_problem*> ps(n);
  for (uint32_t i = 0; i < n; ++i) ps[i] = &b.reqs[i]->prob;
  BatchPlan bp;
  plan_layout(ctx, ps.data(), n, bp);
  BatchState& st = b.state;
  st.mem = ctx->arena.alloc(bp.total);
  if (!st.mem.ptr) return fail(BRMPPI_ENOMEM, "served batch does not fit");
  char* base = st.mem.ptr;
  plan_fill(ctx, ps.data(), n, base, bp);
  hipStream_t s = ctx->streams[b.slot];
  int rc;
  if ((rc = ctx->slot_pin[b.slot].ensure(bp.header_bytes + bp.out_floats * sizeof(float)))) return rc;
  char* pin = ctx->slot_pin[b.slot].ptr;
  stage_batch(bp, ps.data(), pin);
  HIPCHK(launch_upload(upload(pin, base, bp.header_bytes), s));
  if ((rc = enqueue_batch(ctx, s, base, bp, ctx->counters + 1 + b.slot, false))) return rc;
  st.out_pos = bp.out_pos;
  st.out_floats = bp.out_floats;
  st.out_off = bp.header_bytes;
  if (!st.done_ev) HIPCHK(hipEventCreateWithFlags(&st.done_ev, hipEventDisableTiming));
  HIPCHK(hipEventRecord(st.done_ev, s));
  return 0;
}

template <class B>
int HipServed::query(B& b) {
  const hipError_t q = hipEventQuery(b.state.done_ev);
  if (q == hipSuccess) return 0;
  if (q == hipErrorNotReady) return 1;
  return -1;
}

// results of a completed batch into its requests; its memory back to the arena
template <class B>
void HipServed::retire(B& b) {
  BatchState& st = b.state;
  const float* pout = reinterpret_cast<const float*>(ctx->slot_pin[b.slot].ptr + st.out_off);
  for (size_t i = 0; i < b.reqs.size(); ++i) {
    Request* r = b.reqs[i];
    const float* o = pout + st.out_pos[i];
    r->status = (int)o[3];
    r->result.assign(o + 4, o + 4 + 3 * r->prob.T);
    r->st.J_min = o[0];
    r->st.Z = o[1];
    r->st.ess = o[2];
  }
  ctx->arena.release(st.mem);
  if (st.done_ev) (void)hipEventDestroy(st.done_ev);
  st.done_ev = nullptr;
}

// a failed batch: work of it that may already be enqueued on the slot's
// stream finishes before its memory goes back to the arena
template <class B>
void HipServed::abandon(B& b) {
  BatchState& st = b.state;
  if (st.mem.ptr) (void)hipStreamSynchronize(ctx->streams[b.slot]);
  ctx->arena.release(st.mem);
  if (st.done_ev) (void)hipEventDestroy(st.done_ev);
  st.done_ev = nullptr;
}

SlotState& HipServed::controller(uint32_t id) { return ctx->ctrl[id]; }
bool HipServed::fits(size_t bytes) { return ctx->arena.fits(bytes); }

int load_tune(brmppi_ctx* ctx) {
  if (ctx->tune_path.empty()) return 0;
  std::ifstream f(ctx->tune_path);
  if (!f) return 0;
  std::stringstream ss;
  ss << f.rdbuf();
  const std::string s = ss.str();
  // format: {"plain_<bucket>_<sclass>": [block, variant], ...} (entries of
  // other names, the batched launch's blocks of older files among them, are left alone)
  auto valid_block = [](long v) { return v >= 64 && v <= kMaxBlock && v % 64 == 0; };
  for (int bi = 0; bi < 5; ++bi) {
    for (int sc = 0; sc < 4; ++sc) {
      const std::string k = "\"plain_" + std::to_string(kBuckets[bi]) + "_" + std::to_string(sc) + "\"";
      const size_t at = s.find(k);
      if (at == std::string::npos) continue;
      const size_t br = s.find('[', at);
      if (br == std::string::npos) continue;
      char* end = nullptr;
      const long blk = std::strtol(s.c_str() + br + 1, &end, 10);
      const size_t comma = s.find(',', br);
      if (comma == std::string::npos) continue;
      const long var = std::strtol(s.c_str() + comma + 1, nullptr, 10);
      const int lanes = variant_lanes((int)var);
      if (valid_block(blk) && var >= 0 && var <= kMaxVariant && blk % lanes == 0)
        ctx->shape[bi][sc] = LaunchShape{(uint32_t)blk, (int)var};
    }
  }
  return 0;
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

const char* brmppi_last_error(void) { return g_err.c_str(); }

int brmppi_create(const brmppi_config* cfg, brmppi_ctx** out) {
  if (!cfg || !out) return fail(BRMPPI_EINVAL, "null config or output pointer");
  *out = nullptr;
  if (!cfg->arena || (reinterpret_cast<uintptr_t>(cfg->arena) % 256) != 0)
    return fail(BRMPPI_EINVAL, "arena must be a 256-byte aligned device pointer");
  if (cfg->arena_bytes < (1u << 20)) return fail(BRMPPI_EINVAL, "arena smaller than 1 MiB");
  if (cfg->n_streams < 1 || cfg->n_streams > 4) return fail(BRMPPI_EINVAL, "n_streams must be 1..4");
  for (uint32_t k = 0; k < cfg->n_streams; ++k)
    if (!cfg->streams[k]) return fail(BRMPPI_EINVAL, "stream handle is NULL");
  if (cfg->max_controllers == 0 || cfg->max_controllers > 65536)
    return fail(BRMPPI_EINVAL, "max_controllers must be 1..65536");
  hipPointerAttribute_t attr;
  if (hipPointerGetAttributes(&attr, cfg->arena) != hipSuccess || attr.type != hipMemoryTypeDevice) {
    (void)hipGetLastError();
    return fail(BRMPPI_EINVAL, "arena is not device memory");
  }
  if (cfg->device < 0 || cfg->device >= kMaxDevices) return fail(BRMPPI_EINVAL, "device ordinal out of range");
  HIPCHK(hipSetDevice(cfg->device));
  std::unique_ptr<brmppi_ctx> ctx(new brmppi_ctx());
  ctx->device = cfg->device;
  {
    // the static scratch's address on this device (looked up once per device)
    std::lock_guard<std::mutex> lk(g_static_mu);
    if (!g_static_ptr[cfg->device]) {
      void* ptr = nullptr;
      const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
      if (e != hipSuccess || !ptr)
        return fail(BRMPPI_EDEVICE, std::string("static scratch address: ") + hipGetErrorString(e));
      g_static_ptr[cfg->device] = static_cast<char*>(ptr);
    }
    ctx->static_scratch = g_static_ptr[cfg->device];
  }
  ctx->arena.init(cfg->arena, cfg->arena_bytes);
  ctx->n_streams = cfg->n_streams;
  for (uint32_t k = 0; k < cfg->n_streams; ++k) ctx->streams[k] = static_cast<hipStream_t>(cfg->streams[k]);
  ctx->srv.configure(cfg->n_streams, cfg->max_inflight);
  ctx->flags = cfg->flags;
  if (cfg->autotune_cache) ctx->tune_path = cfg->autotune_cache;
  int ncu = 0;
  HIPCHK(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, cfg->device));
  ctx->n_cu = ncu > 0 ? ncu : 256;
  ctx->ctrl.resize(cfg->max_controllers);
  const brmppi_params defaults = default_params();
  for (Controller& c : ctx->ctrl) c.params = defaults;
  // staging buffers and the closed loop's events exist for the context's life
  if (int rc = ctx->pin.ensure(kPinnedInit)) return rc;
  for (uint32_t k = 0; k < cfg->n_streams; ++k)
    if (int rc = ctx->slot_pin[k].ensure(kPinnedInit)) return rc;
  for (auto& e : ctx->loop_ev) HIPCHK(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  const size_t ctr_bytes = round_up(sizeof(BatchCounters) * 5, 256) + counter_bytes(kDrawnBlocks * kDrawnTile / kWChunk);
  ctx->counters_blk = ctx->arena.alloc(ctr_bytes);
  if (!ctx->counters_blk.ptr) return fail(BRMPPI_ENOMEM, "arena too small");
  ctx->counters = reinterpret_cast<BatchCounters*>(ctx->counters_blk.ptr);
  ctx->drawn_ctr = reinterpret_cast<uint32_t*>(ctx->counters_blk.ptr + round_up(sizeof(BatchCounters) * 5, 256));
  {
    // one staging-sized copy each way before the counters are cleared: the
    // runtime hands copies above a few KB to a DMA engine whose first use in a
    // process costs about 8 ms of host time (measured); create pays it
    // instead of the first call whose upload is that large (a closed loop's
    // descriptor chunk, a served batch)
    const size_t cb = std::min(kPinnedInit, cfg->arena_bytes);
    hipError_t e = hipMemcpyAsync(cfg->arena, ctx->pin.ptr, cb, hipMemcpyHostToDevice, ctx->streams[0]);
    if (e == hipSuccess) e = hipMemcpyAsync(ctx->pin.ptr, cfg->arena, cb, hipMemcpyDeviceToHost, ctx->streams[0]);
    if (e == hipSuccess)
      e = launch_fill_u32(reinterpret_cast<uint32_t*>(ctx->counters), 0u, ctr_bytes / 4, ctx->streams[0]);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->streams[0]);
    if (e != hipSuccess) return fail(BRMPPI_EDEVICE, std::string("context init: ") + hipGetErrorString(e));
  }
  load_tune(ctx.get());
  brmppi_ctx* raw = ctx.release();
  raw->served_dev.ctx = raw;
  raw->srv.start(raw->served_dev);
  *out = raw;
  return BRMPPI_OK;
}

int brmppi_destroy(brmppi_ctx* ctx) {
  if (!ctx) return fail(BRMPPI_EINVAL, "null context");
  // queued requests fail with ECANCELED, batches in flight drain, the request
  // thread ends
  ctx->srv.stop();
  for (uint32_t k = 0; k < ctx->n_streams; ++k) (void)hipStreamSynchronize(ctx->streams[k]);
  drop_graph(ctx);
  collect_timing(ctx);
  for (hipEvent_t e : ctx->ev_pool) (void)hipEventDestroy(e);
  delete ctx;
  return BRMPPI_OK;
}

int brmppi_get_info(brmppi_ctx* ctx, brmppi_info* out) {
  if (!ctx || !out) return fail(BRMPPI_EINVAL, "null argument");
  std::lock_guard<std::mutex> lk(ctx->mu);
  out->scratch_grows = ctx->scratch_grows;
  uint64_t pg = ctx->pin.grows;
  for (const auto& p : ctx->slot_pin) pg += p.grows;
  out->pinned_grows = pg;
  out->arena_bytes = ctx->arena.size();
  out->arena_used = ctx->arena.used();
  out->served_done = ctx->srv.done_count();
  out->served_failed = ctx->srv.failed_count();
  return BRMPPI_OK;
}

int brmppi_default_params(brmppi_params* out) {
  if (!out) return fail(BRMPPI_EINVAL, "null argument");
  *out = default_params();
  return BRMPPI_OK;
}

int brmppi_set_params(brmppi_ctx* ctx, uint32_t controller, const brmppi_params* params) {
  if (!ctx) return fail(BRMPPI_EINVAL, "null context");
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (controller >= ctx->ctrl.size()) return fail(BRMPPI_EINVAL, "controller id out of range");
  const brmppi_params P = params ? *params : default_params();
  if (int rc = validate_params(P)) return rc;
  ctx->ctrl[controller].params = P;
  return BRMPPI_OK;
}

int brmppi_set_path(brmppi_ctx* ctx, uint32_t controller, const float* path, uint32_t n, float ds) {
  if (!ctx || !path) return fail(BRMPPI_EINVAL, "null argument");
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (controller >= ctx->ctrl.size()) return fail(BRMPPI_EINVAL, "controller id out of range");
  if (n < 2 || n > BRMPPI_MAX_PATH) return fail(BRMPPI_EINVAL, "path needs 2..BRMPPI_MAX_PATH waypoints");
  if (!(ds > 0) || !std::isfinite(ds)) return fail(BRMPPI_EINVAL, "ds must be positive");
  for (size_t i = 0; i < (size_t)n * 4; ++i)
    if (!std::isfinite(path[i])) return fail(BRMPPI_EINVAL, "non-finite path value");
  Controller& c = ctx->ctrl[controller];
  if (c.busy) return fail(BRMPPI_EAGAIN, "controller has a request in flight");
  if (!c.mem.ptr) {
    c.mem = ctx->arena.alloc(sizeof(float) * 3 * BRMPPI_MAX_T + 256 + sizeof(double) * 8);
    if (!c.mem.ptr) return fail(BRMPPI_ENOMEM, "controller state does not fit in the arena");
    c.unom = reinterpret_cast<float*>(c.mem.ptr);
    c.plant = reinterpret_cast<double*>(c.mem.ptr + round_up(sizeof(float) * 3 * BRMPPI_MAX_T, 256));
  }
  if (c.path_blk.bytes < sizeof(float4) * n) {
    Block nb = ctx->arena.alloc(sizeof(float4) * n);
    if (!nb.ptr) return fail(BRMPPI_ENOMEM, "path does not fit in the arena");
    ctx->arena.release(c.path_blk);
    c.path_blk = nb;
  }
  c.path = reinterpret_cast<float4*>(c.path_blk.ptr);
  HIPCHK(hipMemcpy(c.path, path, sizeof(float4) * n, hipMemcpyHostToDevice));
  c.n_path = n;
  c.ds = ds;
  return BRMPPI_OK;
}

int brmppi_get_nominal(brmppi_ctx* ctx, uint32_t controller, float* u, uint32_t T) {
  if (!ctx || !u) return fail(BRMPPI_EINVAL, "null argument");
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (controller >= ctx->ctrl.size()) return fail(BRMPPI_EINVAL, "controller id out of range");
  Controller& c = ctx->ctrl[controller];
  if (!c.unom || c.warm_T == 0) return fail(BRMPPI_ESTATE, "no resident warm start");
  if (T != c.warm_T) return fail(BRMPPI_EINVAL, "T differs from the resident warm start");
  if (c.busy) return fail(BRMPPI_EAGAIN, "controller has a request in flight");
  HIPCHK(hipStreamSynchronize(ctx->streams[0]));
  HIPCHK(hipMemcpy(u, c.unom, sizeof(float) * 3 * T, hipMemcpyDeviceToHost));
  return BRMPPI_OK;
}

int brmppi_set_nominal(brmppi_ctx* ctx, uint32_t controller, const float* u, uint32_t T) {
  if (!ctx || !u) return fail(BRMPPI_EINVAL, "null argument");
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (controller >= ctx->ctrl.size()) return fail(BRMPPI_EINVAL, "controller id out of range");
  if (T < 1 || T > BRMPPI_MAX_T) return fail(BRMPPI_EINVAL, "T out of range");
  Controller& c = ctx->ctrl[controller];
  if (!c.unom) return fail(BRMPPI_ESTATE, "controller has no path (brmppi_set_path)");
  if (c.busy) return fail(BRMPPI_EAGAIN, "controller has a request in flight");
  for (size_t i = 0; i < (size_t)3 * T; ++i)
    if (!std::isfinite(u[i])) return fail(BRMPPI_EINVAL, "non-finite nominal value");
  HIPCHK(hipStreamSynchronize(ctx->streams[0]));
  HIPCHK(hipMemcpy(c.unom, u, sizeof(float) * 3 * T, hipMemcpyHostToDevice));
  c.warm_T = T;
  return BRMPPI_OK;
}

int brmppi_set_state(brmppi_ctx* ctx, uint32_t controller, const double x[8]) {
  if (!ctx || !x) return fail(BRMPPI_EINVAL, "null argument");
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (controller >= ctx->ctrl.size()) return fail(BRMPPI_EINVAL, "controller id out of range");
  Controller& c = ctx->ctrl[controller];
  if (!c.plant) return fail(BRMPPI_ESTATE, "controller has no path (brmppi_set_path)");
  for (int k = 0; k < 8; ++k)
    if (!std::isfinite(x[k])) return fail(BRMPPI_EINVAL, "non-finite state");
  HIPCHK(hipStreamSynchronize(ctx->streams[0]));
  HIPCHK(hipMemcpy(c.plant, x, sizeof(double) * 8, hipMemcpyHostToDevice));
  c.plant_set = true;
  return BRMPPI_OK;
}

int brmppi_get_state(brmppi_ctx* ctx, uint32_t controller, double x[8]) {
  if (!ctx || !x) return fail(BRMPPI_EINVAL, "null argument");
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (controller >= ctx->ctrl.size()) return fail(BRMPPI_EINVAL, "controller id out of range");
  Controller& c = ctx->ctrl[controller];
  if (!c.plant || !c.plant_set) return fail(BRMPPI_ESTATE, "no resident plant state");
  HIPCHK(hipStreamSynchronize(ctx->streams[0]));
  HIPCHK(hipMemcpy(x, c.plant, sizeof(double) * 8, hipMemcpyDeviceToHost));
  return BRMPPI_OK;
}

int brmppi_solve_ex(brmppi_ctx* ctx, const brmppi_problem* p, const brmppi_outputs* out, brmppi_stats* st) {
  if (!ctx) return fail(BRMPPI_EINVAL, "null context");
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (p && p->controller < ctx->ctrl.size() && ctx->ctrl[p->controller].busy)
    return fail(BRMPPI_EAGAIN, "controller has a request in flight");
  return solve_locked(ctx, p, out, st);
}

int brmppi_solve(brmppi_ctx* ctx, const brmppi_problem* p, float* u_out, brmppi_stats* st) {
  brmppi_outputs o{u_out, nullptr, nullptr};
  return brmppi_solve_ex(ctx, p, &o, st);
}

int brmppi_solve_noalloc(brmppi_ctx* ctx, const brmppi_problem* p, float* u_out, brmppi_stats* st) {
  if (!ctx) return fail(BRMPPI_EINVAL, "null context");
  if (!ctx->static_scratch) return fail(BRMPPI_ESTATE, "no static scratch on this device");
  std::lock_guard<std::mutex> dev_lk(g_static_call_mu[ctx->device]);
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (p && p->controller < ctx->ctrl.size() && ctx->ctrl[p->controller].busy)
    return fail(BRMPPI_EAGAIN, "controller has a request in flight");
  brmppi_outputs o{u_out, nullptr, nullptr};
  return solve_locked(ctx, p, &o, st, ctx->static_scratch, BRMPPI_NOALLOC_MAX_BYTES);
}

int brmppi_solve_batch(brmppi_ctx* ctx, const brmppi_problem* p, uint32_t n, float* const* u_outs,
                       brmppi_stats* st) {
  if (!ctx) return fail(BRMPPI_EINVAL, "null context");
  std::lock_guard<std::mutex> lk(ctx->mu);
  for (uint32_t i = 0; p && i < n; ++i)
    if (p[i].controller < ctx->ctrl.size() && ctx->ctrl[p[i].controller].busy)
      return fail(BRMPPI_EAGAIN, "a controller has a request in flight");
  return solve_batch_locked(ctx, p, n, u_outs, st);
}

int brmppi_closed_loop(brmppi_ctx* ctx, const brmppi_problem* p, uint32_t n_updates, double* x_out,
                       float* u_applied) {
  if (!ctx) return fail(BRMPPI_EINVAL, "null context");
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (p && p->controller < ctx->ctrl.size() && ctx->ctrl[p->controller].busy)
    return fail(BRMPPI_EAGAIN, "controller has a request in flight");
  return closed_loop_locked(ctx, p, n_updates, x_out, u_applied);
}

int brmppi_submit(brmppi_ctx* ctx, const brmppi_problem* p, uint64_t* ticket) {
  if (!ctx || !ticket) return fail(BRMPPI_EINVAL, "null argument");
  TraceRange tr("brmppi submit");
  std::lock_guard<std::mutex> lk(ctx->mu);
  // a missing warm start is allowed when an earlier queued request of the same
  // controller will leave one; the request thread re-checks at launch
  int rc = BRMPPI_OK;
  if (!p) return fail(BRMPPI_EINVAL, "null problem");
  {
    // validate everything except the warm-start length
    brmppi_problem q = *p;
    std::vector<float> dummy;
    if (!q.u_nom && q.controller < ctx->ctrl.size() && q.T >= 1 && q.T <= BRMPPI_MAX_T) {
      dummy.assign((size_t)3 * q.T, 0.0f);
      q.u_nom = dummy.data();
    }
    rc = validate(ctx, &q);
    if (rc) return rc;
  }
  const size_t fp = request_footprint(p->S, p->T);
  if (fp > ctx->arena.size()) return fail(BRMPPI_ENOMEM, "request can never fit in the arena");
  std::unique_ptr<Request> r(new Request());
  copy_problem(*r, *p, params_of(ctx, *p));
  r->footprint = fp;
  rc = ctx->srv.submit(std::move(r), ticket);
  if (rc == BRMPPI_EAGAIN) return fail(rc, "max_inflight requests queued or unpolled");
  return rc;
}

namespace {
int served_status(int rc) {
  switch (rc) {
    case BRMPPI_OK:
    case BRMPPI_PENDING:
      return rc;
    case BRMPPI_ENOTICKET:
      return fail(rc, "unknown or consumed ticket");
    case BRMPPI_ETIMEDOUT:
      return fail(rc, "deadline passed");
    case BRMPPI_EINVAL:
      return fail(rc, "u_out is NULL");
    case BRMPPI_ECANCELED:
      return fail(rc, "the context was destroyed before the request was admitted");
    case BRMPPI_ENOMEM:
      return fail(rc, "the request can never fit in the arena's free space");
    case BRMPPI_ESTATE:
      return fail(rc, "no resident warm start of the request's horizon");
    default:
      return fail(rc, "request failed or had only non-finite costs");
  }
}
}  // namespace

int brmppi_poll(brmppi_ctx* ctx, uint64_t ticket, float* u_out, brmppi_stats* st) {
  if (!ctx) return fail(BRMPPI_EINVAL, "null context");
  std::lock_guard<std::mutex> lk(ctx->mu);
  return served_status(ctx->srv.poll(ticket, u_out, st));
}

int brmppi_wait(brmppi_ctx* ctx, uint64_t ticket, float* u_out, brmppi_stats* st, uint32_t timeout_ms) {
  if (!ctx) return fail(BRMPPI_EINVAL, "null context");
  return served_status(ctx->srv.wait(ticket, u_out, st, timeout_ms));
}

int brmppi_set_launch(brmppi_ctx* ctx, uint32_t block, uint32_t variant) {
  if (!ctx) return fail(BRMPPI_EINVAL, "null context");
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (block == 0) {
    ctx->forced = LaunchShape{0, 0};
    drop_graph(ctx);
    return BRMPPI_OK;
  }
  if (block < 64 || block > (uint32_t)kMaxBlock || block % 64)
    return fail(BRMPPI_EINVAL, "block must be 64..256, a multiple of 64");
  if (variant > (uint32_t)kMaxVariant) return fail(BRMPPI_EINVAL, "variant must be 0..4");
  ctx->forced = LaunchShape{block, (int)variant};
  drop_graph(ctx);
  return BRMPPI_OK;
}

int brmppi_autotune(brmppi_ctx* ctx) {
  if (!ctx) return fail(BRMPPI_EINVAL, "null context");
  std::lock_guard<std::mutex> lk(ctx->mu);
  // synthetic problems: straight path, obstacles alternating on both sides
  const uint32_t T = 48;           // long enough that the step loop, not launch and reduction, dominates
  const uint32_t n_path = 400;
  const uint32_t S_rep[4] = {2048, 8192, 32768, 65536};   // one per S class
  std::vector<float> path(4 * n_path);
  for (uint32_t i = 0; i < n_path; ++i) {
    path[4 * i] = 0.1f * i;
    path[4 * i + 1] = 0.0f;
    path[4 * i + 2] = 0.0f;
    path[4 * i + 3] = 0.0f;
  }
  const brmppi_params P = default_params();
  hipStream_t s = ctx->streams[0];
  hipEvent_t e0, e1;
  HIPCHK(hipEventCreate(&e0));
  HIPCHK(hipEventCreate(&e1));
  std::string json = "{";
  auto add = [&](const std::string& k, const std::string& v) {
    json += std::string(json.size() > 1 ? ", " : "") + "\"" + k + "\": " + v;
  };
  int rc = BRMPPI_OK;
  for (int bi = 0; bi < 5 && rc == BRMPPI_OK; ++bi) {
    const int bucket = kBuckets[bi];
    const uint32_t K = bucket == 0 ? 3u : 5u + bucket;
    for (int sc = 0; sc < 4 && rc == BRMPPI_OK; ++sc) {
      const uint32_t S = S_rep[sc];
      const ScratchLayout L = scratch_layout(S, T, K);
      const size_t off_desc = L.bytes, off_path = off_desc + round_up(sizeof(SolveDesc), 256);
      const size_t off_unom = off_path + round_up(sizeof(float4) * n_path, 256);
      const size_t off_ctr = off_unom + round_up(sizeof(float) * 3 * T, 256);
      const size_t need = off_ctr + counter_bytes(L.n_wchunk);
      if (ensure_scratch(ctx, need) != 0) break;   // larger classes do not fit this arena
      char* base = ctx->scratch.ptr;
      SolveDesc* d_desc = reinterpret_cast<SolveDesc*>(base + off_desc);
      float4* d_path = reinterpret_cast<float4*>(base + off_path);
      float* d_unom = reinterpret_cast<float*>(base + off_unom);
      HIPCHK(hipMemcpy(d_path, path.data(), sizeof(float4) * n_path, hipMemcpyHostToDevice));
      HIPCHK(hipMemset(d_unom, 0, sizeof(float) * 3 * T));
      HIPCHK(hipMemset(base + off_ctr, 0, counter_bytes(L.n_wchunk)));   // not captured in a graph
      Resident c;
      c.path = d_path;
      c.n_path = n_path;
      c.ds = 0.1f;
      c.unom = d_unom;
      const TuneUpdate tune(bucket, S, T, P);
      SolveDesc h;
      LaunchShape best = ctx->shape[bi][sc];
      float best_ms = 1e30f;
      std::string times;             // [block, variant, ms per noise + rollout + reduce] of every candidate
      for (int variant = 0; variant <= kMaxVariant; ++variant) {
        const uint32_t lanes = (uint32_t)variant_lanes(variant);
        for (uint32_t block : {64u, 128u, 256u}) {
          const uint32_t per_tile = block / lanes;
          const uint32_t grid = (S + per_tile - 1) / per_tile;
          // time what a plain solve would run: fused epilogue where the tiles
          // are whole units, else the rollout plus k_reduce
          size_t lds = 0;
          if (fused_tile_ok(per_tile)) {
            lds = fused_lds_bytes(per_tile, T, L.n_wchunk);
            if (lds > kFusedLdsMax) lds = 0;
          }
          fill_desc(h, tune.p, c, L, base, 0, nullptr, reinterpret_cast<uint32_t*>(base + off_ctr),
                    reinterpret_cast<float*>(base + L.off_out), lds > 0, lds == 0);
          HIPCHK(hipMemcpy(d_desc, &h, sizeof(h), hipMemcpyHostToDevice));
          const uint32_t nr = L.n_wchunk * L.n_rgroup;
          SolveArgs args;
          args.d = h;
          const bool drawn = drawn_fits(ctx->n_cu, bucket, LaunchShape{block, variant}, S, T, lds);
          auto run = [&]() -> hipError_t {
            hipError_t e = hipSuccess;
            if (drawn) return launch_rollout_drawn(bucket, args, grid, lds, s);
            if (variant_pre(variant)) e = launch_noise(NoiseArgs{h.noise, 0, 0, L.S_pad, K, 0}, 1, T, Upload{}, s);
            if (e == hipSuccess)
              e = launch_rollout(bucket, variant, d_desc, grid, block, lds, s);
            if (e == hipSuccess && !lds) e = launch_reduce(d_desc, nullptr, nr, nullptr, nr, s);
            return e;
          };
          HIPCHK(run());
          HIPCHK(hipEventRecord(e0, s));
          for (int r = 0; r < 3; ++r) HIPCHK(run());
          HIPCHK(hipEventRecord(e1, s));
          HIPCHK(hipEventSynchronize(e1));
          float ms = 0.0f;
          HIPCHK(hipEventElapsedTime(&ms, e0, e1));
          ms /= 3.0f;
          char buf[64];
          std::snprintf(buf, sizeof(buf), "%s[%u, %d, %.5f]", times.empty() ? "" : ", ", block, variant, ms);
          times += buf;
          // near-ties go to a shape that reduces its own tiles (one launch per
          // update instead of two): it has to be 2 % slower to lose, so that
          // timing noise does not flip the choice from one run to the next
          const float score = lds ? ms * 0.98f : ms;
          if (score < best_ms) {
            best_ms = score;
            best = LaunchShape{block, variant};
          }
        }
      }
      ctx->shape[bi][sc] = best;
      add("plain_" + std::to_string(bucket) + "_" + std::to_string(sc),
          "[" + std::to_string(best.block) + ", " + std::to_string(best.variant) + "]");
      add("ms_plain_" + std::to_string(bucket) + "_" + std::to_string(sc), "[" + times + "]");
    }
  }
  json += "}\n";
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  drop_graph(ctx);
  if (!ctx->tune_path.empty()) {
    std::ofstream f(ctx->tune_path);
    if (f) f << json;
  }
  return rc;
}

int brmppi_profile_read(brmppi_ctx* ctx, double out[6]) {
  if (!ctx || !out) return fail(BRMPPI_EINVAL, "null argument");
  std::lock_guard<std::mutex> lk(ctx->mu);
  const int kinds[3] = {0, 1, 4};   // rollout, reduce, noise
  for (int k = 0; k < 3; ++k) {
    out[2 * k] = ctx->prof.ms[kinds[k]];
    out[2 * k + 1] = ctx->prof.n[kinds[k]];
  }
  return BRMPPI_OK;
}

int brmppi_profile_reset(brmppi_ctx* ctx) {
  if (!ctx) return fail(BRMPPI_EINVAL, "null context");
  std::lock_guard<std::mutex> lk(ctx->mu);
  ctx->prof = Profile{};
  return BRMPPI_OK;
}

int brmppi_debug_philox(brmppi_ctx* ctx, const uint32_t* ctr, const uint32_t key[2], uint32_t n, uint32_t* out) {
  if (!ctx || !ctr || !key || !out || n == 0 || n > (1u << 24)) return fail(BRMPPI_EINVAL, "bad arguments");
  std::lock_guard<std::mutex> lk(ctx->mu);
  Block b = ctx->arena.alloc(sizeof(uint32_t) * 8 * (size_t)n);
  if (!b.ptr) return fail(BRMPPI_ENOMEM, "debug buffer does not fit");
  uint32_t* d_in = reinterpret_cast<uint32_t*>(b.ptr);
  uint32_t* d_out = d_in + 4 * (size_t)n;
  hipStream_t s = ctx->streams[0];
  int rc = BRMPPI_OK;
  do {
    hipError_t e = hipMemcpyAsync(d_in, ctr, sizeof(uint32_t) * 4 * (size_t)n, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = launch_philox_dump(d_in, key[0], key[1], n, d_out, s);
    if (e == hipSuccess) e = hipMemcpyAsync(out, d_out, sizeof(uint32_t) * 4 * (size_t)n, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) rc = fail(BRMPPI_EDEVICE, hipGetErrorString(e));
  } while (0);
  ctx->arena.release(b);
  return rc;
}

int brmppi_debug_normals(brmppi_ctx* ctx, uint64_t seed, uint32_t instance, const uint32_t* s_tau, uint32_t n,
                         uint32_t K, float* out) {
  if (!ctx || !s_tau || !out || n == 0 || n > (1u << 22) || K == 0 || K > 64) return fail(BRMPPI_EINVAL, "bad arguments");
  std::lock_guard<std::mutex> lk(ctx->mu);
  Block b = ctx->arena.alloc(sizeof(uint32_t) * 2 * (size_t)n + 256 + sizeof(float) * (size_t)n * K);
  if (!b.ptr) return fail(BRMPPI_ENOMEM, "debug buffer does not fit");
  uint32_t* d_in = reinterpret_cast<uint32_t*>(b.ptr);
  float* d_out = reinterpret_cast<float*>(b.ptr + round_up(sizeof(uint32_t) * 2 * (size_t)n, 256));
  hipStream_t s = ctx->streams[0];
  int rc = BRMPPI_OK;
  do {
    hipError_t e = hipMemcpyAsync(d_in, s_tau, sizeof(uint32_t) * 2 * (size_t)n, hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
      e = launch_normals_dump((uint32_t)(seed & 0xffffffffu), (uint32_t)(seed >> 32), instance, d_in, n, K, d_out, s);
    if (e == hipSuccess) e = hipMemcpyAsync(out, d_out, sizeof(float) * (size_t)n * K, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) rc = fail(BRMPPI_EDEVICE, hipGetErrorString(e));
  } while (0);
  ctx->arena.release(b);
  return rc;
}

int brmppi_debug_box_muller(brmppi_ctx* ctx, const uint32_t* r, uint32_t n, float* out) {
  if (!ctx || !r || !out || n == 0 || n > (1u << 24)) return fail(BRMPPI_EINVAL, "bad arguments");
  std::lock_guard<std::mutex> lk(ctx->mu);
  Block b = ctx->arena.alloc(round_up(sizeof(uint32_t) * (size_t)n, 256) + sizeof(float) * 3 * (size_t)n);
  if (!b.ptr) return fail(BRMPPI_ENOMEM, "debug buffer does not fit");
  uint32_t* d_in = reinterpret_cast<uint32_t*>(b.ptr);
  float* d_out = reinterpret_cast<float*>(b.ptr + round_up(sizeof(uint32_t) * (size_t)n, 256));
  hipStream_t s = ctx->streams[0];
  int rc = BRMPPI_OK;
  do {
    hipError_t e = hipMemcpyAsync(d_in, r, sizeof(uint32_t) * (size_t)n, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = launch_box_muller_dump(d_in, n, d_out, s);
    if (e == hipSuccess) e = hipMemcpyAsync(out, d_out, sizeof(float) * 3 * (size_t)n, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) rc = fail(BRMPPI_EDEVICE, hipGetErrorString(e));
  } while (0);
  ctx->arena.release(b);
  return rc;
}

}  // extern "C"
