// C ABI of the Slow Momentum hot path: argument checking, workspace layout,
// tiling tables, per-call gradient-pointer table, counters.  All arithmetic on
// tensor elements happens in the kernels (slowmo_kernels.hip).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <vector>

#include "../../include/slowmo.h"
#include "slowmo_kernels.h"
#include "slowmo_plan.h"

using namespace slowmo;

namespace {

constexpr int kSlots = 4;            // ring of per-call tables (mixing order, de-bias table)
constexpr int kGradSlots = 16;       // gradient-pointer tables kept on the device
constexpr size_t kSectionAlign = 256;

thread_local std::string g_err = "";

size_t round_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// One slot of the mixing-table ring holds the entries of one mixing step, then its groups
// (only with more than kMixInline workers; otherwise they travel with the launch).
size_t mixtab_bytes(int32_t m) {
  return m > kMixInline ? static_cast<size_t>(m) * (sizeof(MixSend) + sizeof(uint32_t)) : 0;
}
// One slot of the de-bias ring: m * n_tensors destination pointers, then, where they do not
// travel with the launch, the m weights.
size_t ztab_bytes(int32_t m, int32_t n_tensors) {
  return static_cast<size_t>(m) * n_tensors * sizeof(void *) + static_cast<size_t>(m) * sizeof(float);
}

// Byte offsets of the sections of the caller's workspace.
struct Sections {
  size_t x0, u, h, v, xtab_t, gtab[kGradSlots], mixtab[kSlots], ztab[kSlots], slots,
      tensors, ltiles, otiles, pace, cleared, total;
};

Sections make_sections(const slowmo_config &c, int32_t n_tensors, const Layout &L, size_t n_ltiles,
                       size_t n_otiles, size_t n_btiles, size_t n_ptiles) {
  Sections s{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t at = off;
    off += round_up(std::max<size_t>(bytes, 1), kSectionAlign);
    return at;
  };
  const size_t arena = static_cast<size_t>(L.d_pad) * sizeof(float);
  const size_t n_ptr = static_cast<size_t>(c.m) * n_tensors;
  const size_t outer_copies = c.no_average ? static_cast<size_t>(c.m) : 1;
  s.x0 = take(arena * outer_copies);
  s.u = take(arena * outer_copies);
  s.h = take(arena * c.m);
  s.v = take(c.base == SLOWMO_ADAM ? arena * c.m : 0);
  s.pace = take(kPaceWords * sizeof(uint32_t));
  s.cleared = off - s.x0;   // x0, u, h, v and the pace counters start as zeros
  s.xtab_t = take(n_ptr * sizeof(void *));
  for (int i = 0; i < kGradSlots; ++i) s.gtab[i] = take(n_ptr * sizeof(void *));
  for (int i = 0; i < kSlots; ++i) s.mixtab[i] = take(mixtab_bytes(c.m));
  for (int i = 0; i < kSlots; ++i) s.ztab[i] = take(ztab_bytes(c.m, n_tensors));
  s.slots = take(n_ptr * sizeof(SlotInfo));
  s.tensors = take(static_cast<size_t>(n_tensors) * sizeof(TensorInfo));
  s.ltiles = take(n_ltiles * sizeof(TileRef));
  // ordinary tiles, then, one list after the other, big tiles, the ordinary tiles
  // they leave over (at most all of them), and the same for paced tiles
  s.otiles = take((n_otiles + (n_btiles ? n_btiles + n_otiles : 0) +
                   (n_ptiles ? n_ptiles + n_otiles : 0)) * sizeof(TileRef));
  s.total = off;
  return s;
}

int32_t env_flag(const char *name, int32_t dflt) {
  const char *s = std::getenv(name);
  if (!s || !*s) return dflt;
  return static_cast<int32_t>(std::strtol(s, nullptr, 10));
}

// SLOWMO_PACED, read at slowmo_state_bytes and slowmo_create.  Paced walks: 0 = never,
// 1 = by the rule, 2 = wherever the kernels allow.
int32_t paced_mode() { return env_flag("SLOWMO_PACED", 1); }

// All sections for a configuration and tensor list that passed check_config.
Sections make_sections(const slowmo_config &c, int32_t n_tensors, const int64_t *numel,
                       const Layout &L) {
  return make_sections(
      c, n_tensors, L, static_cast<size_t>(count_local_tiles(c.m, n_tensors, numel)),
      static_cast<size_t>(count_outer_tiles(n_tensors, numel)),
      static_cast<size_t>(count_big_tiles(n_tensors, numel)),
      static_cast<size_t>(count_paced_pieces(c.m, n_tensors, numel, paced_mode() >= 2)));
}

bool finite_pos(float v) { return std::isfinite(v) && v > 0.f; }
bool unit_interval(float v) { return std::isfinite(v) && v >= 0.f && v < 1.f; }

// Returns an empty string if cfg / tensor list are usable.
std::string check_config(const slowmo_config *c, int32_t n_tensors, const int64_t *numel) {
  if (!c) return "cfg is NULL";
  if (!numel) return "numel is NULL";
  if (n_tensors < 1) return "n_tensors must be >= 1";
  if (c->m < 1 || c->m > SLOWMO_MAX_WORKERS) return "m must be in 1..SLOWMO_MAX_WORKERS";
  if (c->tau < 1) return "tau must be >= 1";
  if (!finite_pos(c->alpha)) return "alpha must be finite and > 0";
  if (!unit_interval(c->beta)) return "beta must satisfy 0 <= beta < 1";
  if (c->base != SLOWMO_SGD_NESTEROV && c->base != SLOWMO_ADAM) return "unknown base optimizer";
  if (c->policy != SLOWMO_BUF_RESET && c->policy != SLOWMO_BUF_MAINTAIN &&
      c->policy != SLOWMO_BUF_AVERAGE)
    return "unknown buffer policy";
  if (c->grad_dtype != SLOWMO_F32 && c->grad_dtype != SLOWMO_BF16) return "unknown gradient dtype";
  if (c->no_average != 0 && c->no_average != 1) return "no_average must be 0 or 1";
  if (c->no_average && c->policy == SLOWMO_BUF_AVERAGE)
    return "no_average cannot be combined with the AVERAGE buffer policy";
  if (!(std::isfinite(c->weight_decay) && c->weight_decay >= 0.f))
    return "weight_decay must be finite and >= 0";
  if (c->base == SLOWMO_SGD_NESTEROV) {
    if (!unit_interval(c->momentum)) return "momentum must satisfy 0 <= momentum < 1";
  } else {
    if (!unit_interval(c->beta1) || !unit_interval(c->beta2))
      return "beta1 and beta2 must satisfy 0 <= . < 1";
    if (!(std::isfinite(c->eps) && c->eps >= 0.f)) return "eps must be finite and >= 0";
  }
  int64_t total = 0;
  for (int32_t j = 0; j < n_tensors; ++j) {
    if (numel[j] < 0) return "numel has a negative entry";
    if (numel[j] > (int64_t(1) << 36)) return "a tensor exceeds 2^36 elements";
    total += numel[j];
  }
  if (total * c->m > (int64_t(1) << 44)) return "m * total elements exceeds 2^44";
  if (static_cast<int64_t>(c->m) * n_tensors > (int64_t(1) << 24))
    return "m * n_tensors exceeds 2^24";
  if (count_local_tiles(c->m, n_tensors, numel) > (int64_t(1) << 31) - 16)
    return "too many tiles for one launch (m * total elements too large)";
  return "";
}

// A small host->device table that may change from call to call: a ring of
// device slots (inside the caller's workspace) with pinned staging copies,
// and one event per slot recorded after its upload, so that a staging copy is
// not rewritten while an earlier upload may still be reading it.
template <int N>
struct TableRing {
  void *d[N] = {};
  void *h[N] = {};
  hipEvent_t ev[N] = {};
  bool used[N] = {};     // the slot's device copy holds the table of its staging copy
  bool sent[N] = {};     // an upload from the slot's staging copy was enqueued (ev recorded)
  size_t len[N] = {};    // bytes of the table in each slot
  uint64_t key[N] = {};  // cheap fingerprint of the table in each slot
  int cur = -1;          // slot of the most recent upload, -1 = none

  hipError_t init(char *device_base, const size_t *offsets, size_t bytes) {
    for (int i = 0; i < N; ++i) {
      d[i] = device_base + offsets[i];
      hipError_t e = hipHostMalloc(&h[i], std::max<size_t>(bytes, 8), hipHostMallocDefault);
      if (e != hipSuccess) return e;
      e = hipEventCreateWithFlags(&ev[i], hipEventDisableTiming);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  // A few words of the table (first, last, two in between) mixed with its
  // length: distinct pointer tables differ there, so the full comparison
  // below runs for one candidate, not for every slot.
  static uint64_t fingerprint(const void *src, size_t bytes) {
    const size_t words = bytes / sizeof(uint64_t);
    uint64_t k = 0x9e3779b97f4a7c15ull ^ bytes;
    if (words == 0) return k;
    const size_t at[4] = {0, words / 3, 2 * words / 3, words - 1};
    for (size_t i : at) {
      uint64_t w;
      std::memcpy(&w, static_cast<const char *>(src) + i * sizeof(uint64_t), sizeof(w));
      k = (k ^ w) * 0xff51afd7ed558ccdull;
      k ^= k >> 32;
    }
    return k;
  }
  // Slot that already holds exactly this table (most recent first), or -1.
  // The staging copy of a slot always equals what its device copy holds once
  // the stream has reached the upload.
  int find(const void *src, size_t bytes) const {
    if (cur < 0) return -1;
    const uint64_t k = fingerprint(src, bytes);
    for (int i = 0; i < N; ++i) {
      const int slot = (cur - i + N) % N;
      if (used[slot] && key[slot] == k && len[slot] == bytes &&
          std::memcmp(h[slot], src, bytes) == 0)
        return slot;
    }
    return -1;
  }
  // The next slot's staging buffer, free to be written (waits until the
  // previous upload from it has been consumed); returns the slot or -1.
  int stage(hipError_t *err) {
    const int slot = (cur + 1) % N;
    if (sent[slot]) {
      *err = hipEventSynchronize(ev[slot]);
      if (*err != hipSuccess) return -1;
      sent[slot] = false;
    }
    used[slot] = false;
    return slot;
  }
  // Sends the first `bytes` of slot's staging buffer to `dst` (the slot's own
  // device copy when dst is NULL) and makes the slot the current one.
  hipError_t send(int slot, size_t bytes, void *dst, hipStream_t stream) {
    hipError_t e = hipMemcpyAsync(dst ? dst : d[slot], h[slot], bytes, hipMemcpyHostToDevice, stream);
    if (e != hipSuccess) return e;
    e = hipEventRecord(ev[slot], stream);
    if (e != hipSuccess) return e;
    sent[slot] = true;
    used[slot] = dst == nullptr;  // a table sent elsewhere is not found again in this slot
    len[slot] = bytes;
    key[slot] = fingerprint(h[slot], bytes);
    cur = slot;
    return hipSuccess;
  }
  // Uploads `bytes` from src into the next slot; returns the slot or -1.
  int upload(const void *src, size_t bytes, hipStream_t stream, hipError_t *err) {
    const int slot = stage(err);
    if (slot < 0) return -1;
    std::memcpy(h[slot], src, bytes);
    *err = send(slot, bytes, nullptr, stream);
    return *err == hipSuccess ? slot : -1;
  }
  void destroy() {
    for (int i = 0; i < N; ++i) {
      if (ev[i]) (void)hipEventDestroy(ev[i]);
      if (h[i]) (void)hipHostFree(h[i]);
    }
  }
};

}  // namespace

struct slowmo_ctx {
  slowmo_config cfg{};
  int32_t n_tensors = 0;
  std::vector<int64_t> numel;
  Layout layout;
  int device = 0;

  // sections of the caller's workspace (device pointers)
  float *x0 = nullptr, *u = nullptr, *h = nullptr, *v = nullptr;
  float **d_xtab_t = nullptr;  // replica pointers, tensor-major
  SlotInfo *d_slots = nullptr;
  TensorInfo *d_tensors = nullptr;
  TileRef *d_ltiles = nullptr;
  TileRef *d_otiles = nullptr;
  int32_t n_ltiles = 0, n_otiles = 0;
  // With big tiles in use, the outer step and the fused last step run twice:
  // over the big tiles (whole pieces of the tensors all of whose
  // replicas are 16-byte aligned) and over the ordinary tiles these leave
  // over.  Otherwise n_btiles = 0 and the rest list is the whole ordinary list.
  TileRef *d_btiles = nullptr, *d_rtiles = nullptr;
  int32_t n_btiles = 0, n_rtiles = 0;
  // Paced walks (gossip step fused with the local step): tiles, and the ordinary
  // tiles they leave over; paced.ntiles = 0 when the list is too short.
  PacedArgs paced{};
  TileRef *d_prtiles = nullptr;
  int32_t n_prtiles = 0;
  bool prtiles_by_group = false;  // the left-over tiles run once per connected group
  bool last_big = false, outer_big = false;  // the fused last step, the outer step take big tiles

  TableRing<kGradSlots> gtab;  // gradient-pointer tables of recent calls (m * n_tensors each)
  TableRing<kSlots> mixtab;  // update order of the current mixing step (at most m entries)
  TableRing<kSlots> ztab;  // destination pointers and weights of the current de-bias call
  std::vector<float> w;  // push-sum weights (Algorithm C.1), 1 after every exact average
  std::vector<SlotInfo> slots;      // host copies of the per-slot / per-tensor tables
  std::vector<TensorInfo> tinfo;

  int64_t t = 0;  // outer iterations done
  int32_t k = 0;  // local steps in the current outer iteration
  int64_t l = 0;  // Adam steps counted by the bias correction
  bool buffers_zero = true;  // h (and v) are to be read as zero by the next local step
  bool params_aligned = true;  // every replica pointer is 16-byte aligned
  int32_t check_pointers = 1;  // 1: caller's tensors are checked at create; 2: also per call

  void *static_table = nullptr;  // this device's static scratch (slowmo_debias_static)

  // A call that launches several kernels and fails between two of them has
  // changed device memory halfway: the context then refuses further work.
  bool broken = false;
  // Test hook (SLOWMO_TEST_FAIL_LAUNCH=n, read at create): the n-th kernel
  // launch of this context (1-based) is not issued and reports a launch
  // failure instead, so the error paths can be driven from the host.
  int64_t fail_launch_at = 0, launches = 0;

  LaunchTuning tune{};
  bool gossip_outer_nt = true;  // tune.outer_nt for an outer step after a fused gossip step
  bool after_gossip = false;    // the last inner step was one
  bool teams = true;    // short lists by teams, a wave per worker
  bool group_launches = false;  // test hook: slowmo_mix_step launches a kernel per connected group
  bool turning = true;  // sweeps over the tiles change direction (tune.backward)
  std::string err;
};

namespace {

slowmo_status fail(slowmo_ctx *ctx, slowmo_status st, const std::string &msg) {
  if (ctx) {
    ctx->err = msg;
  } else {
    g_err = msg;
  }
  return st;
}

slowmo_status fail_hip(slowmo_ctx *ctx, hipError_t e, const char *what) {
  return fail(ctx, SLOWMO_ERR_HIP,
              std::string(what) + ": " + hipGetErrorName(e) + " (" + hipGetErrorString(e) + ")");
}

// Every kernel launch of a context goes through here (see fail_launch_at).
template <typename F>
hipError_t guarded(slowmo_ctx *ctx, F &&launch) {
  if (ctx->fail_launch_at > 0 && ++ctx->launches == ctx->fail_launch_at) return hipErrorLaunchFailure;
  return launch();
}

// The launches of one sweep over the tiles are out: the next sweep goes the other way.
void swept(slowmo_ctx *ctx, bool paced = false) {
  if (ctx->turning) ctx->tune.backward = next_sweep(ctx->tune.backward, paced);
}

// Whether the gossip step goes by teams (a wave per worker), from 2 to kTeamMost workers up to
// 65 536 waves in all.  Beyond, memory is what bounds it and the walk from worker to worker
// is the better order.  Fused step, team over walk, SGD / Adam: cycle of all workers, 16 to 1024
// tiles, m = 2 0.74-0.80, 4 0.55-0.80, 8 0.36-0.70, 16 0.23-0.52, 32 0.17-0.58; 32 768 and 65 536
// waves 0.84-1.04, worst m = 2 with Adam; 131 072 waves 0.98-1.14; 262 144 1.05-1.29.  Pairs and
// groups of 4: 0.71-0.98 up to 65 536 waves, 1.1-1.4 from 131 072 on.  By itself: cycle of 8 to 32
// workers 0.24-0.93 (m = 8, 4096 tiles 1.07), pairs 0.88-1.08; 131 072 waves 1.05-1.32.  Lists with
// kept tiles (Adam with fp32 gradients, 65 536 waves) 1.02-1.25: a team streams them.
bool mix_by_team(const slowmo_ctx *ctx) {
  const int32_t m = ctx->cfg.m;
  return ctx->teams && m > 1 && m <= kTeamMost && ctx->tune.kept_mix == 0 &&
         static_cast<int64_t>(ctx->n_otiles) * m <= 65536;
}

// Whether the outer step, by itself or fused with the last local step, goes by teams (a wave per
// worker).  Team over walk: 16 to 512 tiles, 4 to 6 workers 0.80-0.96 (fused) and 0.61-0.96 (by
// itself, with the local step before it), 8 and 12 0.53-0.96, 16 to 32 0.37-0.94; 768 and 1024 tiles
// up to 16 384 waves 0.66-0.98 and 0.70-1.02, but "reset" at 1024 tiles 1.03-1.09; beyond 1024 tiles,
// or 16 384 waves, 0.8-1.29.  2 workers 1.0-1.1, 3 workers 0.93-1.06; by itself with averaged
// buffers 3 workers 0.80-1.01.
bool outer_by_team(const slowmo_ctx *ctx, bool fused) {
  const int32_t m = ctx->cfg.m, policy = ctx->cfg.policy;
  const int32_t fewest = policy == SLOWMO_BUF_AVERAGE && !fused ? 3 : 4;
  const int32_t tiles = policy == SLOWMO_BUF_RESET && fused ? 768 : 1024;
  return ctx->teams && m >= fewest && m <= kTeamMost && ctx->n_otiles <= tiles &&
         static_cast<int64_t>(ctx->n_otiles) * m <= 16384;
}

// Failure after at least one kernel of a multi-kernel call was launched.
slowmo_status fail_midway(slowmo_ctx *ctx, hipError_t e, const char *what) {
  ctx->broken = true;
  return fail(ctx, SLOWMO_ERR_HIP,
              std::string(what) + ": " + hipGetErrorName(e) + " (" + hipGetErrorString(e) +
                  ") after part of the call's kernels were launched; replicas and buffers are "
                  "partly updated and the context refuses further steps");
}

// A kernel that walks all workers per workgroup runs over the big tiles (if
// any) with `big`, then over the ordinary tiles they leave over with `rest`;
// both take (tiles, count) and return a hipError_t.  *launched counts the
// kernels of the current call issued so far: a failure after the first one is
// a failure halfway.
template <typename FB, typename FR>
slowmo_status run_tiled(slowmo_ctx *ctx, bool use_big, int *launched, const char *what, FB &&big,
                        FR &&rest) {
  for (int pass = 0; pass < 2; ++pass) {
    const bool b = pass == 0;
    if (b && !use_big) continue;
    const TileRef *tiles = b ? ctx->d_btiles : (use_big ? ctx->d_rtiles : ctx->d_otiles);
    const int32_t n = b ? ctx->n_btiles : (use_big ? ctx->n_rtiles : ctx->n_otiles);
    if (n <= 0) continue;
    const hipError_t e = guarded(ctx, [&] { return b ? big(tiles, n) : rest(tiles, n); });
    if (e != hipSuccess) return *launched ? fail_midway(ctx, e, what) : fail_hip(ctx, e, what);
    ++*launched;
  }
  swept(ctx);
  return SLOWMO_OK;
}

const char *kBrokenMsg =
    "an earlier multi-kernel call failed halfway; the context's state is undefined: destroy it";

void release(slowmo_ctx *ctx) {
  ctx->gtab.destroy();
  ctx->mixtab.destroy();
  ctx->ztab.destroy();
  delete ctx;
}

}  // namespace

extern "C" {

const char *slowmo_version(void) { return "0.1.0 gfx950"; }

const char *slowmo_last_error(const slowmo_ctx *ctx) {
  return ctx ? ctx->err.c_str() : g_err.c_str();
}

size_t slowmo_state_bytes(const slowmo_config *cfg, int32_t n_tensors, const int64_t *numel) {
  std::string bad = check_config(cfg, n_tensors, numel);
  if (!bad.empty()) {
    g_err = bad;
    return 0;
  }
  return make_sections(*cfg, n_tensors, numel, make_layout(n_tensors, numel)).total;
}

static int64_t plan_query(bool local, int32_t m, int32_t n_tensors, const int64_t *numel,
                          slowmo_plan_run *out, int64_t cap) {
  if (m < 1 || n_tensors < 1 || !numel || cap < 0 || (cap > 0 && !out)) return -1;
  for (int32_t j = 0; j < n_tensors; ++j)
    if (numel[j] < 0) return -1;
  const int64_t total =
      local ? count_local_tiles(m, n_tensors, numel) : count_outer_tiles(n_tensors, numel);
  if (cap == 0) return total;
  if (total > (int64_t(1) << 31) - 16) return -1;
  std::vector<PlanRun> runs;
  if (local) {
    plan_local(m, n_tensors, numel, runs);
  } else {
    plan_outer(n_tensors, numel, runs);
  }
  for (int64_t i = 0; i < std::min<int64_t>(cap, runs.size()); ++i) {
    out[i] = {runs[i].tile, runs[i].worker, runs[i].tensor, runs[i].n, runs[i].offset};
  }
  return total;
}

int64_t slowmo_plan_local(int32_t m, int32_t n_tensors, const int64_t *numel, slowmo_plan_run *out,
                          int64_t cap) {
  return plan_query(true, m, n_tensors, numel, out, cap);
}

int64_t slowmo_plan_outer(int32_t m, int32_t n_tensors, const int64_t *numel, slowmo_plan_run *out,
                          int64_t cap) {
  return plan_query(false, m, n_tensors, numel, out, cap);
}

slowmo_status slowmo_check_device_range(const void *ptr, size_t bytes) {
  if (!ptr) return fail(nullptr, SLOWMO_ERR_ARG, "pointer is NULL");
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(nullptr, e, "hipGetDevice");
  const char *lo = static_cast<const char *>(ptr);
  const char *ends[2] = {lo, lo + (bytes ? bytes - 1 : 0)};
  for (const char *q : ends) {
    hipPointerAttribute_t at{};
    e = hipPointerGetAttributes(&at, q);
    if (e != hipSuccess) {
      (void)hipGetLastError();  // not sticky: the next call must not see it
      return fail(nullptr, SLOWMO_ERR_ARG,
                  "the range is not memory known to the HIP runtime (ordinary host memory?)");
    }
    if (at.type == hipMemoryTypeUnregistered)
      return fail(nullptr, SLOWMO_ERR_ARG, "the range is ordinary host memory, not device-accessible");
    if (at.type == hipMemoryTypeDevice && at.device != dev)
      return fail(nullptr, SLOWMO_ERR_ARG, "the range is memory of another device");
  }
  hipDeviceptr_t base = nullptr;
  size_t size = 0;
  e = hipMemGetAddressRange(&base, &size, const_cast<void *>(ptr));
  if (e != hipSuccess) {
    (void)hipGetLastError();  // no range information for this kind of memory: both ends were known
  } else if (lo + bytes > static_cast<const char *>(base) + size) {
    return fail(nullptr, SLOWMO_ERR_ARG, "the range runs past the end of its allocation");
  }
  return SLOWMO_OK;
}

slowmo_status slowmo_create(slowmo_ctx **out, const slowmo_config *cfg, int32_t n_tensors,
                            const int64_t *numel, float *const *params, void *state,
                            size_t state_bytes, void *stream_) {
  if (!out) return fail(nullptr, SLOWMO_ERR_ARG, "out is NULL");
  *out = nullptr;
  std::string bad = check_config(cfg, n_tensors, numel);
  if (!bad.empty()) return fail(nullptr, SLOWMO_ERR_ARG, bad);
  if (!params) return fail(nullptr, SLOWMO_ERR_ARG, "params is NULL");
  if (!state) return fail(nullptr, SLOWMO_ERR_ARG, "state is NULL");
  if (reinterpret_cast<uintptr_t>(state) % kSectionAlign)
    return fail(nullptr, SLOWMO_ERR_ALIGN, "state workspace must be 256-byte aligned");

  const int32_t m = cfg->m;
  const size_t n_ptr = static_cast<size_t>(m) * n_tensors;
  struct Span {
    uintptr_t lo, hi;
  };
  std::vector<Span> spans;
  for (size_t i = 0; i < n_ptr; ++i) {
    const int64_t n = numel[i % n_tensors];
    if (n == 0) continue;
    if (!params[i]) return fail(nullptr, SLOWMO_ERR_ARG, "a parameter pointer is NULL");
    uintptr_t p = reinterpret_cast<uintptr_t>(params[i]);
    if (p % sizeof(float)) return fail(nullptr, SLOWMO_ERR_ALIGN, "a parameter pointer is not 4-byte aligned");
    spans.push_back({p, p + static_cast<uintptr_t>(n) * sizeof(float)});
  }

  slowmo_ctx *ctx = new (std::nothrow) slowmo_ctx;
  if (!ctx) return fail(nullptr, SLOWMO_ERR_NOMEM, "host allocation failed");
  ctx->cfg = *cfg;
  ctx->n_tensors = n_tensors;
  ctx->numel.assign(numel, numel + n_tensors);
  ctx->layout = make_layout(n_tensors, numel);
  ctx->tune.xcd_remap = env_flag("SLOWMO_XCD_REMAP", 1) ? 1 : 0;
  ctx->tune.xcd_run = std::max(env_flag("SLOWMO_XCD_RUN", 0), 0);
  ctx->tune.nontemporal = env_flag("SLOWMO_NT", 1) ? 1 : 0;
  // write-through stores, streaming accesses of the local and of the outer step: -1 = by
  // the rule, 0 = never, 1 = always; kept MB: -1 = by the rule
  const int32_t through = env_flag("SLOWMO_WRITE_THROUGH", -1);
  const int32_t local_nt = env_flag("SLOWMO_LOCAL_NT", -1);
  const int32_t outer_nt = env_flag("SLOWMO_OUTER_NT", -1);
  const int32_t kept_mb = env_flag("SLOWMO_KEPT", -1);
  const int64_t elements = static_cast<int64_t>(m) * ctx->layout.d;
  const int64_t grad_bytes = cfg->grad_dtype == SLOWMO_BF16 ? 2 : 4;
  const int64_t buffer_bytes = cfg->base == SLOWMO_ADAM ? 8 : 4;
  const int64_t touched_state = elements * (4 + buffer_bytes);
  const int64_t touched = touched_state + elements * grad_bytes;
  const bool past_l2 = touched > int64_t{54} << 20;
  const int64_t outer_bytes = 8 * ctx->layout.d * (cfg->no_average ? m : 1);
  const bool one_step = cfg->tau == 1 && cfg->policy == SLOWMO_BUF_RESET && !cfg->no_average;
  CacheRule caches = cache_rule({touched_state, elements * grad_bytes, grad_bytes, outer_bytes,
                                 one_step ? elements * buffer_bytes : 0, cfg->tau,
                                 cfg->base == SLOWMO_ADAM, cfg->policy == SLOWMO_BUF_AVERAGE});
  if (kept_mb >= 0) caches.kept_bytes = kept_mb * 1e6;
  const auto streams = [&](int32_t asked, bool by_rule) {
    return ctx->tune.nontemporal && (asked < 0 ? by_rule : asked != 0);
  };
  ctx->tune.local_nt = streams(local_nt, caches.streaming);
  ctx->tune.mix_nt = streams(local_nt, caches.gossip_streaming);
  ctx->tune.outer_nt = streams(outer_nt, caches.outer_streaming);
  ctx->tune.last_nt = streams(outer_nt, caches.last_streaming);
  ctx->gossip_outer_nt = streams(outer_nt, caches.gossip_outer_streaming);
  ctx->tune.write_through = through < 0 ? caches.write_through : through != 0;
  // the outer step without the average: written through 24 MB 1.10-1.12 times, 60 MB
  // 1.02-1.04, 84 MB 1.01-1.02, from 120 MB on 0.98-1.00
  ctx->tune.noavg_through = through < 0 ? elements * 12 > (int64_t{108} << 20) : through != 0;
  ctx->tune.fuse_last = env_flag("SLOWMO_FUSE_LAST", 1) ? 1 : 0;
  ctx->tune.fuse_mix = env_flag("SLOWMO_FUSE_MIX", 1) ? 1 : 0;
  // 160 KiB / 8 KiB: at most 20 single-wave workgroups per CU.  With all 32 the
  // requests of too many tiles meet in the memory and each of its pages is opened
  // more often; with 20 the local step still has twice the requests in flight that
  // it needs.  ResNet-18-shaped round, m = 8: 3.565 ms without the cap, 3.45 with 22,
  // 3.440 with 20, 3.446 with 17 wavefronts; tensors packed back to back 2.82 ->
  // 2.65 ms; Adam with bf16 gradients 0.669 -> 0.643 ms; outer step without the
  // average 4 % faster.  The de-biasing kernel (one read, one write) needs all 32:
  // 30 % slower with the cap.  Where the working set stays in the L2s there are no pages to
  // spare: 3 to 4.5 M elements, time over that before any cap, with it / without: steps
  // 0.95-1.02 / 0.92-1.00, the last one under "reset" 1.02-1.09 / 0.96-1.03.
  // SGD with kept tiles: part of its requests never reach the memory, and up to 4 GB it
  // takes 28 (300-500 MB 0.96-0.97 of the time with 20, 1 GB 0.97-1.00, 2 GB 0.98-1.00, 5 GB
  // 1.00; Adam 0.99-1.02).
  const bool more_waves = caches.kept_bytes > 0 && cfg->base == SLOWMO_SGD_NESTEROV &&
                          touched < int64_t{4} << 30;
  const auto local_cap = [&](int32_t by_rule) {
    return std::min(std::max(env_flag("SLOWMO_LOCAL_LDS", by_rule), 0), 64 * 1024);
  };
  ctx->tune.local_lds = local_cap(!past_l2 ? 0 : more_waves ? 5800 : 8192);
  ctx->tune.noavg_lds = local_cap(past_l2 ? 8192 : 0);
  // At most 16 single-wave workgroups per CU in the outer step and the fused last step,
  // for the same reason, as long as a wave walks few workers; with many its own
  // streams are what opens the pages, and fewer waves only leave requests out.  With
  // the cap over without, lists of 12 to 51 M elements and 1, 2, 4, 8, 16, 32 workers:
  // outer step 0.96-0.97, 0.96-0.97, 0.97-0.98, 0.97-0.98, 0.99-1.01, 1.00; with the
  // buffers averaged 0.97-0.98, 0.95-0.97, 0.97-0.98, 0.97-0.98, 1.00, 1.00-1.01; fused
  // last step 0.95-1.01, 0.96-1.00, 0.97-1.01, 0.99-1.01, 0.99-1.02, 1.00-1.01.
  const int32_t outer_lds = env_flag("SLOWMO_OUTER_LDS", -1);
  const auto waves_cap = [&](int32_t below) {
    return outer_lds >= 0 ? std::min(outer_lds, 64 * 1024) : m < below ? 10240 : 0;
  };
  ctx->tune.outer_lds = waves_cap(16);
  ctx->tune.last_lds = waves_cap(8);
  // big tiles: -1 = by the worker count (see kBigFusedFromWorkers), 0 = never, 1 = always
  const int32_t big = env_flag("SLOWMO_BIG_TILES", -1);
  ctx->tune.big_tiles =
      ((big < 0 ? m >= kBigFusedFromWorkers : big != 0) && ctx->tune.nontemporal) ? 1 : 0;
  ctx->tune.paced = paced_mode();
  // a list of half the L2s' 32 MB is found there in any order and has nothing to turn for
  // (18 MB 0.84-0.98 of the time, 9-15 MB 0.98-1.04)
  ctx->turning = env_flag("SLOWMO_TURN", touched > int64_t{16} << 20) != 0;
  ctx->teams = env_flag("SLOWMO_TEAM", 1) != 0;
  ctx->fail_launch_at = env_flag("SLOWMO_TEST_FAIL_LAUNCH", 0);
  ctx->group_launches = env_flag("SLOWMO_TEST_GROUP_LAUNCHES", 0) != 0;

  const int64_t n_ltiles = count_local_tiles(m, n_tensors, numel);
  const int64_t n_otiles = count_outer_tiles(n_tensors, numel);
  const Sections sec = make_sections(*cfg, n_tensors, numel, ctx->layout);
  if (state_bytes < sec.total) {
    delete ctx;
    return fail(nullptr, SLOWMO_ERR_NOMEM, "state workspace is smaller than slowmo_state_bytes()");
  }
  spans.push_back({reinterpret_cast<uintptr_t>(state), reinterpret_cast<uintptr_t>(state) + sec.total});
  std::sort(spans.begin(), spans.end(), [](const Span &a, const Span &b) { return a.lo < b.lo; });
  for (size_t i = 1; i < spans.size(); ++i) {
    if (spans[i].lo < spans[i - 1].hi) {
      delete ctx;
      return fail(nullptr, SLOWMO_ERR_ARG, "parameter tensors overlap each other or the workspace");
    }
  }

  // ---- from here on the device is needed -------------------------------------
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  hipError_t e = hipGetDevice(&ctx->device);
  if (e != hipSuccess) {
    delete ctx;
    return fail_hip(nullptr, e, "hipGetDevice");
  }
  ctx->check_pointers = env_flag("SLOWMO_CHECK_POINTERS", 1);
  if (ctx->check_pointers) {
    slowmo_status bad_ptr = slowmo_check_device_range(state, sec.total);
    for (size_t i = 0; i < n_ptr && bad_ptr == SLOWMO_OK; ++i) {
      const int64_t n = numel[i % n_tensors];
      if (n) bad_ptr = slowmo_check_device_range(params[i], static_cast<size_t>(n) * sizeof(float));
    }
    if (bad_ptr != SLOWMO_OK) {
      delete ctx;
      g_err = "parameter tensor or workspace: " + g_err;
      return bad_ptr;
    }
  }
  char *base = static_cast<char *>(state);
  ctx->x0 = reinterpret_cast<float *>(base + sec.x0);
  ctx->u = reinterpret_cast<float *>(base + sec.u);
  ctx->h = reinterpret_cast<float *>(base + sec.h);
  ctx->v = cfg->base == SLOWMO_ADAM ? reinterpret_cast<float *>(base + sec.v) : nullptr;
  ctx->d_xtab_t = reinterpret_cast<float **>(base + sec.xtab_t);
  ctx->d_slots = reinterpret_cast<SlotInfo *>(base + sec.slots);
  ctx->d_tensors = reinterpret_cast<TensorInfo *>(base + sec.tensors);
  ctx->d_ltiles = reinterpret_cast<TileRef *>(base + sec.ltiles);
  ctx->d_otiles = reinterpret_cast<TileRef *>(base + sec.otiles);
  ctx->n_ltiles = static_cast<int32_t>(n_ltiles);
  ctx->n_otiles = static_cast<int32_t>(n_otiles);
  ctx->paced.counters = reinterpret_cast<uint32_t *>(base + sec.pace);

#define CREATE_HIP(call, what)              \
  do {                                      \
    hipError_t e_ = (call);                 \
    if (e_ != hipSuccess) {                 \
      release(ctx);                         \
      return fail_hip(nullptr, e_, what);   \
    }                                       \
  } while (0)

  CREATE_HIP(ctx->gtab.init(base, sec.gtab, n_ptr * sizeof(void *)), "gradient-pointer ring");
  if (mixtab_bytes(m) > 0)
    CREATE_HIP(ctx->mixtab.init(base, sec.mixtab, mixtab_bytes(m)), "mixing-table ring");
  CREATE_HIP(ctx->ztab.init(base, sec.ztab, ztab_bytes(m, n_tensors)), "de-bias table ring");
  ctx->w.assign(m, 1.0f);
  // set-up for the entry point that may not allocate: this device's address of
  // the library's static scratch array (the create call runs with it current)
  CREATE_HIP(static_scratch(ctx->device, &ctx->static_table), "address of the static scratch array");

  int cus = 0;
  CREATE_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->device),
             "number of CUs");

  // device tables
  const Layout &L = ctx->layout;
  std::vector<SlotInfo> &slots = ctx->slots;
  std::vector<TensorInfo> &tinfo = ctx->tinfo;
  slots.resize(n_ptr);
  tinfo.resize(n_tensors);
  std::vector<float *> xtab_t(n_ptr);
  for (int32_t j = 0; j < n_tensors; ++j) tinfo[j] = {L.arena_off[j], numel[j], 0, 1.0f, cfg->weight_decay};
  for (int32_t w = 0; w < m; ++w) {
    for (int32_t j = 0; j < n_tensors; ++j) {
      const size_t slot = static_cast<size_t>(w) * n_tensors + j;
      slots[slot] = {params[slot], static_cast<int64_t>(w) * L.d_pad + L.arena_off[j], numel[j],
                     cfg->weight_decay, 1.0f};
      xtab_t[static_cast<size_t>(j) * m + w] = params[slot];
      if (numel[j] && (reinterpret_cast<uintptr_t>(params[slot]) & 15)) {
        tinfo[j].unaligned = 1;
        ctx->params_aligned = false;
      }
    }
  }
  std::vector<TileRef> bt, rt;  // big tiles and the ordinary tiles they leave over
  if (ctx->tune.big_tiles) {
    std::vector<int64_t> usable(numel, numel + n_tensors);
    for (int32_t j = 0; j < n_tensors; ++j)
      if (tinfo[j].unaligned) usable[j] = 0;
    // forced big tiles have 16 vectors, unless a test asks for another size
    const int32_t asked = env_flag("SLOWMO_TEST_BIG_VPT", kBigVpt);
    ctx->tune.big_vpt = big <= 0 ? choose_big_vpt(n_tensors, usable.data(), cus)
                                 : asked == 14 || asked == 12 ? asked : kBigVpt;
    const int64_t tile = big_tile(ctx->tune.big_vpt), per_big = tile / kOuterTile;
    for (int32_t j = 0; j < n_tensors && tile > 0; ++j) {
      const int64_t n_big = usable[j] / tile;
      for (int64_t k = 0; k < n_big; ++k) bt.push_back({j, static_cast<int32_t>(k)});
      for (int64_t k = n_big * per_big; k * kOuterTile < numel[j]; ++k)
        rt.push_back({j, static_cast<int32_t>(k)});
    }
  }
  // Kept tiles: a share of the units of every worker.  But big tiles run best while the
  // whole chip is on one worker, and lose that when some of them come from the cache and
  // others do not: the fused last step takes 2.49-2.61 instead of 2.20 ms then (m = 32, 25.6
  // M elements), 322 instead of 275 us (m = 8, 11.7 M).  Where an outer step or a fused last step
  // takes big tiles, the local step keeps whole workers, or, if one is too large, units of the
  // first.  (Where none does, units for all: rounds with averaged buffers, m = 16, 2-3 GB 0.95-0.99 of
  // the time with whole workers, m = 16 and 32, 6-12 GB 0.97-1.00.)
  static_assert(SLOWMO_BUF_RESET == 0 && SLOWMO_BUF_MAINTAIN == 1 && SLOWMO_BUF_AVERAGE == 2,
                "the policies as the kernels and the rules name them");
  const bool any_big = !bt.empty() && !cfg->no_average;
  ctx->last_big = any_big && ctx->tune.fuse_last && last_takes_big(cfg->policy, big > 0);
  ctx->outer_big = any_big && outer_takes_big(m, cfg->policy, big > 0);
  const bool big_in_use = ctx->last_big || ctx->outer_big;
  const double worker_bytes = static_cast<double>(touched_state) / m;
  const int32_t whole = kept_workers(m, caches.kept_bytes, worker_bytes);
  const auto share_of = [&](int32_t w) {
    if (!big_in_use) return kept_share(caches.kept_bytes, static_cast<double>(touched_state));
    if (whole > 0) return kept_share(w < whole ? worker_bytes : 0.0, worker_bytes);
    return kept_share(w == 0 ? caches.kept_bytes : 0.0, worker_bytes);
  };
  const auto flag_at = [&](int32_t j, int64_t element, uint64_t share) {
    return unit_kept(L.arena_off[j] / kKeptUnit + element / kKeptUnit, share) ? kTileKept : 0;
  };
  // To the kernels that walk all workers only a tile that is kept of each of them is one: the
  // outer step and the fused last step take units as such where the local step keeps them.  The
  // gossip step fused with the local step follows others of its kind and keeps units in any
  // case (rounds of 4 of them and an outer step, against streaming where big tiles are in use: m = 8
  // and 12, 0.8-2 GB 0.86-0.96, 4 GB 0.95-0.98, 12 GB 0.98-1.00; m = 16 and 32 0.94-1.01).
  const uint64_t walk_share = kept_share(caches.kept_bytes, static_cast<double>(touched_state));
  ctx->tune.kept_local = caches.kept_bytes > 0;
  const bool asked_to_keep = kept_mb >= 0;  // by SLOWMO_KEPT: in every kernel
  ctx->tune.kept_mix = walk_share == 0 ? 0 : asked_to_keep ? 2 : 1;
  ctx->tune.kept_tiles = big_in_use ? 0 : ctx->tune.kept_mix;
  ctx->tune.kept_outer = ctx->tune.kept_tiles && (asked_to_keep ||
                                            outer_keeps(m, touched, cfg->policy == SLOWMO_BUF_AVERAGE));
  // tiles in launch order: worker-major, tensors in list order, pieces ascending
  static_assert(kLocalTile == kOuterTile, "a worker's local tiles are the outer tiles");
  const auto fill = [&](TileRef *out, int32_t first_owner, uint64_t share) {
    constexpr int64_t per_unit = kKeptUnit / kOuterTile;
    for (int32_t j = 0; j < n_tensors; ++j) {
      const int64_t tiles = (numel[j] + kOuterTile - 1) / kOuterTile;
      for (int64_t k = 0; k < tiles;) {
        const int32_t flag = flag_at(j, k * kOuterTile, share);
        for (const int64_t end = std::min(k + per_unit, tiles); k < end; ++k)
          *out++ = {first_owner + j, static_cast<int32_t>(k) | flag};
      }
    }
    return out;
  };
  const std::unique_ptr<TileRef[]> lt(new (std::nothrow) TileRef[static_cast<size_t>(n_ltiles) + 1]);
  if (!lt) {
    release(ctx);
    return fail(nullptr, SLOWMO_ERR_NOMEM, "host allocation failed");
  }
  TileRef *next = lt.get();
  for (int32_t w = 0; w < m; ++w) next = fill(next, w * n_tensors, share_of(w));
  std::vector<TileRef> lists(static_cast<size_t>(n_otiles));  // the ordinary tiles and what is chosen from them
  fill(lists.data(), 0, walk_share);
  if (n_ltiles > 0)
    CREATE_HIP(hipMemcpyAsync(ctx->d_ltiles, lt.get(), static_cast<size_t>(n_ltiles) * sizeof(TileRef),
                              hipMemcpyHostToDevice, stream),
               "upload of the local-step tiles");
  // appends one more list to the upload; returns its place on the device
  auto append = [&](const std::vector<TileRef> &v) {
    TileRef *at = ctx->d_otiles + lists.size();
    lists.insert(lists.end(), v.begin(), v.end());
    return at;
  };
  if (bt.empty()) {
    ctx->d_rtiles = ctx->d_otiles;
    ctx->n_rtiles = ctx->n_otiles;
  } else {
    ctx->d_btiles = append(bt);
    ctx->d_rtiles = append(rt);
    ctx->n_btiles = static_cast<int32_t>(bt.size());
    ctx->n_rtiles = static_cast<int32_t>(rt.size());
  }
  // paced tiles
  const bool pays = ctx->tune.paced >= 2 ||
                    paced_pays(m, count_paced_pieces(m, n_tensors, numel, false), cus, touched, ctx->params_aligned);
  if (ctx->tune.paced != 0 && pays && ctx->tune.nontemporal && ctx->tune.fuse_mix &&
      count_paced_pieces(m, n_tensors, numel, ctx->tune.paced >= 2) > 0) {
    ctx->paced.members = cus / 8;
    // test hook: a limit that the workgroups reach, to run on out of step
    ctx->paced.spins = env_flag("SLOWMO_TEST_PACE_SPINS", kPaceSpins);
    std::vector<TileRef> pt, prt;
    plan_paced(m, n_tensors, numel, cus % 8 == 0 ? cus : 0, ctx->tune.paced >= 2, pt, prt);
    // The paced kernel itself keeps nothing: with plain accesses to kept units or to kept
    // workers it takes 0.99-1.01 of the time (5 to 26 M elements, 8 to 32 workers).
    for (TileRef &t : prt) t.k |= flag_at(t.owner, int64_t{t.k} * kOuterTile, walk_share);
    ctx->paced.tiles = append(pt);
    ctx->paced.ntiles = static_cast<int32_t>(pt.size());
    ctx->d_prtiles = append(prt);
    ctx->n_prtiles = static_cast<int32_t>(prt.size());
    if (const int32_t ride = env_flag("SLOWMO_PACED_REST", -1);
        ride < 0 ? rest_rides(ctx->paced.ntiles, ctx->n_prtiles, cus) : ride != 0) {
      ctx->paced.rest = ctx->d_prtiles;
      ctx->paced.nrest = ctx->n_prtiles;
      ctx->n_prtiles = 0;
    }
    // A launch per connected group walks only its replicas, but each has a tail of its
    // own.  Groups of 4 workers (m = 16 and 32, both base optimizers, one to four rows
    // of paced tiles), time over all in single waves, in one launch / one per group, by
    // the rest's share of the list: 5 % 0.93-0.97 / 0.94-1.00, 10-20 % 0.85-0.99 /
    // 0.85-0.98, 30-40 % 0.94-1.02 / 0.94-1.03, 50-65 % 0.94-1.03 / 0.92-0.98, 80 %
    // 1.01-1.05 / 0.99-1.02.  One group of all workers: no difference.
    ctx->prtiles_by_group = ctx->n_prtiles > ctx->n_otiles / 4;
  }
  if (!lists.empty())
    CREATE_HIP(hipMemcpyAsync(ctx->d_otiles, lists.data(), lists.size() * sizeof(TileRef),
                              hipMemcpyHostToDevice, stream),
               "upload of the outer-step tiles");
  CREATE_HIP(hipMemcpyAsync(ctx->d_tensors, tinfo.data(), tinfo.size() * sizeof(TensorInfo),
                            hipMemcpyHostToDevice, stream),
             "upload of the tensor table");
  CREATE_HIP(hipMemcpyAsync(ctx->d_slots, slots.data(), n_ptr * sizeof(SlotInfo),
                            hipMemcpyHostToDevice, stream),
             "upload of the slot table");
  CREATE_HIP(hipMemcpyAsync(ctx->d_xtab_t, xtab_t.data(), n_ptr * sizeof(float *),
                            hipMemcpyHostToDevice, stream),
             "upload of the replica pointers");

  // u_0 = 0, h = v = 0 (Algorithm 1, "Input"; Table C.1 caption)
  const size_t outer_copies = cfg->no_average ? static_cast<size_t>(m) : 1;
  CREATE_HIP(hipMemsetAsync(ctx->x0, 0, sec.cleared, stream), "clearing x0, u, h and v");
  // common starting point x_{0,0}: worker 0's replica, into x0 and every other replica
  {
    OuterArgs ia{};
    ia.tiles = ctx->d_otiles;
    ia.tensors = ctx->d_tensors;
    ia.xtab_t = ctx->d_xtab_t;
    ia.ntiles = ctx->n_otiles;
    ia.m = m;
    ia.x0 = ctx->x0;
    ia.d_pad = L.d_pad;
    CREATE_HIP(launch_init_broadcast(ia, static_cast<int32_t>(outer_copies), ctx->tune, stream),
               "copy of x_{0,0} into x0 and the replicas");
  }
  // the host-side tables above go out of scope: wait for their uploads
  CREATE_HIP(hipStreamSynchronize(stream), "hipStreamSynchronize");
#undef CREATE_HIP

  *out = ctx;
  return SLOWMO_OK;
}

extern "C++" {
namespace {

// Checks the arguments of a local step, uploads the gradient-pointer table if
// it changed and fills the kernel arguments.
slowmo_status prepare_local(slowmo_ctx *ctx, const void *const *grads, float lr,
                            hipStream_t stream, LocalArgs *out) {
  if (ctx->broken) return fail(ctx, SLOWMO_ERR_STATE, kBrokenMsg);
  if (!grads) return fail(ctx, SLOWMO_ERR_ARG, "grads is NULL");
  if (!finite_pos(lr)) return fail(ctx, SLOWMO_ERR_ARG, "lr must be finite and > 0");
  if (ctx->k >= ctx->cfg.tau)
    return fail(ctx, SLOWMO_ERR_STATE, "tau local steps already taken: slowmo_outer_step is due");
  const slowmo_config &c = ctx->cfg;
  const size_t n_ptr = static_cast<size_t>(c.m) * ctx->n_tensors;
  const size_t gsize = c.grad_dtype == SLOWMO_BF16 ? 2 : 4;
  // gradient-pointer table: reuse a device copy if one of the recent calls had these
  // very pointers (compared one by one; they passed the checks then)
  int slot = ctx->gtab.find(grads, n_ptr * sizeof(void *));
  if (slot < 0) {
    for (size_t i = 0, j = 0; i < n_ptr; ++i, j = j + 1 == ctx->numel.size() ? 0 : j + 1) {
      if (ctx->numel[j] == 0) continue;
      if (!grads[i]) return fail(ctx, SLOWMO_ERR_ARG, "a gradient pointer is NULL");
      if (reinterpret_cast<uintptr_t>(grads[i]) % gsize)
        return fail(ctx, SLOWMO_ERR_ALIGN, "a gradient pointer is not aligned to its element size");
    }
    hipError_t e = hipSuccess;
    if (ctx->check_pointers >= 2) {
      for (size_t i = 0; i < n_ptr; ++i) {
        const int64_t n = ctx->numel[i % ctx->n_tensors];
        if (n && slowmo_check_device_range(grads[i], static_cast<size_t>(n) * gsize) != SLOWMO_OK)
          return fail(ctx, SLOWMO_ERR_ARG, "gradient tensor: " + g_err);
      }
    }
    slot = ctx->gtab.upload(grads, n_ptr * sizeof(void *), stream, &e);
    if (slot < 0) return fail_hip(ctx, e, "upload of the gradient pointers");
  }

  LocalArgs a{};
  a.tiles = ctx->d_ltiles;
  a.slots = ctx->d_slots;
  a.ntiles = ctx->n_ltiles;
  a.gtab = static_cast<const void *const *>(ctx->gtab.d[slot]);
  a.h = ctx->h;
  a.v = ctx->v;
  // Under the reset policy the buffers written by the last step of an outer iteration are discarded
  // before they are read again: skip those stores.
  a.keep = !(c.policy == SLOWMO_BUF_RESET && ctx->k == c.tau - 1);
  a.lr = lr;
  a.wd = c.weight_decay;
  a.mu = c.momentum;
  if (c.base == SLOWMO_ADAM) {
    const double l_next = static_cast<double>(ctx->l + 1);
    a.b1 = c.beta1;
    a.b2 = c.beta2;
    a.omb1 = 1.0f - c.beta1;
    a.omb2 = 1.0f - c.beta2;
    a.eps = c.eps;
    // 1 / (1 - beta^l), l counting this step, in fp64, rounded once
    a.rc1 = static_cast<float>(1.0 / (1.0 - std::pow(static_cast<double>(c.beta1), l_next)));
    a.rc2 = static_cast<float>(1.0 / (1.0 - std::pow(static_cast<double>(c.beta2), l_next)));
  }
  *out = a;
  return SLOWMO_OK;
}

void finish_local(slowmo_ctx *ctx, bool gossip = false) {
  ctx->after_gossip = gossip;
  ctx->k += 1;
  ctx->l += 1;
  ctx->buffers_zero = false;
}

void finish_outer(slowmo_ctx *ctx) {
  ctx->k = 0;
  ctx->t += 1;
  // after the exact average every worker holds the same, unbiased point again
  if (!ctx->cfg.no_average) std::fill(ctx->w.begin(), ctx->w.end(), 1.0f);
  if (ctx->cfg.policy == SLOWMO_BUF_RESET) {  // Algorithm 1 line 2 of the next outer iteration
    ctx->buffers_zero = true;
    ctx->l = 0;
  }
}

}  // namespace
}  // extern "C++"

slowmo_status slowmo_local_step(slowmo_ctx *ctx, const void *const *grads, float lr,
                                void *stream_) {
  if (!ctx) return fail(nullptr, SLOWMO_ERR_ARG, "ctx is NULL");
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  LocalArgs a{};
  slowmo_status st = prepare_local(ctx, grads, lr, stream, &a);
  if (st != SLOWMO_OK) return st;
  const slowmo_config &c = ctx->cfg;
  hipError_t e = guarded(ctx, [&] {
    return launch_local_step(a, c.base, c.grad_dtype == SLOWMO_BF16, ctx->buffers_zero, !a.keep,
                             ctx->tune, stream);
  });
  if (e != hipSuccess) return fail_hip(ctx, e, "local-step kernel launch");
  swept(ctx);
  finish_local(ctx);
  return SLOWMO_OK;
}

extern "C++" {
namespace {

OuterArgs outer_args(const slowmo_ctx *ctx, float lr) {
  const slowmo_config &c = ctx->cfg;
  OuterArgs a{};
  a.tiles = ctx->d_otiles;
  a.tensors = ctx->d_tensors;
  a.ntiles = ctx->n_otiles;
  a.xtab_t = ctx->d_xtab_t;
  a.m = c.m;
  a.x0 = ctx->x0;
  a.u = ctx->u;
  a.lr = lr;
  a.alpha = c.alpha;
  a.beta = c.beta;
  a.m_f = static_cast<float>(c.m);
  a.d_pad = ctx->layout.d_pad;
  if (c.policy == SLOWMO_BUF_AVERAGE) {  // Algorithm 1 line 2 of the next outer iteration
    a.avg_h = ctx->h;
    a.avg_v = ctx->v;  // nullptr unless Adam
  }
  return a;
}

OuterNoAvgArgs noavg_args(const slowmo_ctx *ctx, float lr) {
  OuterNoAvgArgs na{};
  na.tiles = ctx->d_ltiles;
  na.slots = ctx->d_slots;
  na.ntiles = ctx->n_ltiles;
  na.x0 = ctx->x0;
  na.u = ctx->u;
  na.lr = lr;
  na.alpha = ctx->cfg.alpha;
  na.beta = ctx->cfg.beta;
  return na;
}

// Lines 6-8 and the copy into the replicas.  *launched: kernels of the same
// call already issued (a failure is then a failure halfway).
slowmo_status run_outer(slowmo_ctx *ctx, float lr, int *launched, hipStream_t stream) {
  const slowmo_config &c = ctx->cfg;
  LaunchTuning tune = ctx->tune;
  if (ctx->after_gossip) tune.outer_nt = ctx->gossip_outer_nt;
  if (c.no_average) {  // Section 6: lines 7-8 per worker, no line 6
    const OuterNoAvgArgs na = noavg_args(ctx, lr);
    const hipError_t e =
        guarded(ctx, [&] { return launch_outer_noavg_step(na, tune, stream); });
    if (e != hipSuccess)
      return *launched ? fail_midway(ctx, e, "outer-step kernel launch")
                       : fail_hip(ctx, e, "outer-step kernel launch");
    ++*launched;
    swept(ctx);
    return SLOWMO_OK;
  }
  OuterArgs a = outer_args(ctx, lr);
  const bool team = outer_by_team(ctx, false);
  auto with = [&](const TileRef *tiles, int32_t n) {
    a.tiles = tiles;
    a.ntiles = n;
    return a;
  };
  return run_tiled(
      ctx, ctx->outer_big, launched, "outer-step kernel launch",
      [&](const TileRef *t, int32_t n) { return launch_outer_big(with(t, n), tune, stream); },
      [&](const TileRef *t, int32_t n) {
        return team ? launch_team_outer(nullptr, with(t, n), ctx->n_tensors, 0, false, false, 0, tune, stream)
                    : launch_outer_step(with(t, n), tune, stream);
      });
}

}  // namespace
}  // extern "C++"

slowmo_status slowmo_outer_step(slowmo_ctx *ctx, float lr, void *stream_) {
  if (!ctx) return fail(nullptr, SLOWMO_ERR_ARG, "ctx is NULL");
  if (ctx->broken) return fail(ctx, SLOWMO_ERR_STATE, kBrokenMsg);
  if (!finite_pos(lr)) return fail(ctx, SLOWMO_ERR_ARG, "lr must be finite and > 0");
  if (ctx->k != ctx->cfg.tau)
    return fail(ctx, SLOWMO_ERR_STATE, "the outer step needs exactly tau local steps before it");
  int launched = 0;
  const slowmo_status st = run_outer(ctx, lr, &launched, static_cast<hipStream_t>(stream_));
  if (st != SLOWMO_OK) return st;
  finish_outer(ctx);
  return SLOWMO_OK;
}

slowmo_status slowmo_local_outer_step(slowmo_ctx *ctx, const void *const *grads, float lr,
                                      float outer_lr, void *stream_) {
  if (!ctx) return fail(nullptr, SLOWMO_ERR_ARG, "ctx is NULL");
  if (ctx->broken) return fail(ctx, SLOWMO_ERR_STATE, kBrokenMsg);
  if (!finite_pos(outer_lr)) return fail(ctx, SLOWMO_ERR_ARG, "outer_lr must be finite and > 0");
  if (ctx->k != ctx->cfg.tau - 1)
    return fail(ctx, SLOWMO_ERR_STATE,
                "the fused step is the LAST local step of an outer iteration: tau-1 local steps "
                "must have been taken");
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  LocalArgs a{};
  slowmo_status st = prepare_local(ctx, grads, lr, stream, &a);
  if (st != SLOWMO_OK) return st;
  const slowmo_config &c = ctx->cfg;
  const bool bf16 = c.grad_dtype == SLOWMO_BF16;
  if (c.no_average && ctx->tune.fuse_last) {
    const hipError_t e = guarded(ctx, [&] {
      return launch_local_noavg_step(a, noavg_args(ctx, outer_lr), c.base, bf16, ctx->buffers_zero,
                                     c.policy == SLOWMO_BUF_RESET, ctx->tune, stream);
    });
    if (e != hipSuccess) return fail_hip(ctx, e, "fused local+outer kernel launch");
    swept(ctx);
  } else if (!ctx->tune.fuse_last) {
    // same two kernels as the separate calls
    hipError_t e = guarded(ctx, [&] {
      return launch_local_step(a, c.base, bf16, ctx->buffers_zero, c.policy == SLOWMO_BUF_RESET,
                               ctx->tune, stream);
    });
    if (e != hipSuccess) return fail_hip(ctx, e, "local-step kernel launch");
    swept(ctx);
    ctx->after_gossip = false;
    int launched = 1;
    st = run_outer(ctx, outer_lr, &launched, stream);
    if (st != SLOWMO_OK) return st;
  } else {
    OuterArgs o = outer_args(ctx, outer_lr);
    auto with = [&](const TileRef *tiles, int32_t n) {
      o.tiles = tiles;
      o.ntiles = n;
      return o;
    };
    int launched = 0;
    st = run_tiled(
        ctx, ctx->last_big, &launched, "fused local+outer kernel launch",
        [&](const TileRef *t, int32_t n) {
          return launch_local_outer_big(a, with(t, n), ctx->n_tensors, c.base, bf16,
                                        ctx->buffers_zero, c.policy, ctx->tune, stream);
        },
        [&](const TileRef *t, int32_t n) {
          if (outer_by_team(ctx, true))
            return launch_team_outer(&a, with(t, n), ctx->n_tensors, c.base, bf16, ctx->buffers_zero,
                                     c.policy, ctx->tune, stream);
          return launch_local_outer_step(a, with(t, n), ctx->n_tensors, c.base, bf16,
                                         ctx->buffers_zero, c.policy, ctx->tune, stream);
        });
    if (st != SLOWMO_OK) return st;
  }
  finish_local(ctx);
  finish_outer(ctx);
  return SLOWMO_OK;
}

slowmo_status slowmo_lr_step_decay(float base_lr, float start_lr, int64_t warmup_steps,
                                   const int64_t *milestones, int32_t n_milestones, float factor,
                                   int64_t step, float *lr_out) {
  if (!lr_out || step < 0 || warmup_steps < 0 || n_milestones < 0 ||
      (n_milestones > 0 && !milestones))
    return fail(nullptr, SLOWMO_ERR_ARG, "bad arguments");
  if (!finite_pos(base_lr) || !std::isfinite(start_lr) || start_lr < 0.f ||
      !std::isfinite(factor) || factor <= 0.f || factor > 1.f)
    return fail(nullptr, SLOWMO_ERR_ARG,
                "base_lr must be finite and > 0, start_lr finite and >= 0, factor in (0, 1]");
  for (int32_t i = 0; i < n_milestones; ++i)
    if (milestones[i] < 0 || (i > 0 && milestones[i] <= milestones[i - 1]))
      return fail(nullptr, SLOWMO_ERR_ARG, "milestones must be >= 0 and ascend");
  double lr;
  if (step < warmup_steps) {  // Section 4: linear warm-up
    lr = static_cast<double>(start_lr) + (static_cast<double>(base_lr) - start_lr) *
                                             static_cast<double>(step) / static_cast<double>(warmup_steps);
  } else {                    // ... then one factor per milestone passed
    lr = base_lr;
    for (int32_t i = 0; i < n_milestones && milestones[i] <= step; ++i) lr *= static_cast<double>(factor);
  }
  *lr_out = static_cast<float>(lr);
  return SLOWMO_OK;
}

slowmo_status slowmo_lr_inverse_sqrt(float peak_lr, float init_lr, int64_t warmup_steps,
                                     int64_t step, float *lr_out) {
  if (!lr_out || step < 0 || warmup_steps < 0) return fail(nullptr, SLOWMO_ERR_ARG, "bad arguments");
  if (!finite_pos(peak_lr) || !std::isfinite(init_lr) || init_lr < 0.f)
    return fail(nullptr, SLOWMO_ERR_ARG, "peak_lr must be finite and > 0, init_lr finite and >= 0");
  double lr;
  if (step < warmup_steps) {  // Appendix A.3: linear warm-up
    lr = static_cast<double>(init_lr) + (static_cast<double>(peak_lr) - init_lr) *
                                            static_cast<double>(step) / static_cast<double>(warmup_steps);
  } else if (step == 0) {
    lr = peak_lr;
  } else {                    // ... then proportional to 1 / sqrt(step)
    lr = peak_lr * std::sqrt(static_cast<double>(warmup_steps) / static_cast<double>(step));
  }
  *lr_out = static_cast<float>(lr);
  return SLOWMO_OK;
}

slowmo_status slowmo_expgraph_in_peers(int32_t m, int64_t step, int32_t *in_peer) {
  if (m < 1 || step < 0 || !in_peer) return fail(nullptr, SLOWMO_ERR_ARG, "bad arguments");
  if (m == 1) {
    in_peer[0] = 0;
    return SLOWMO_OK;
  }
  int n_hops = 1;  // hops 2^0 .. 2^floor(log2(m-1))
  while ((int64_t(1) << n_hops) <= m - 1) ++n_hops;
  const int64_t hop = int64_t(1) << (step % n_hops);
  for (int32_t i = 0; i < m; ++i) in_peer[i] = static_cast<int32_t>(((i - hop) % m + m) % m);
  return SLOWMO_OK;
}

extern "C++" {
namespace {

// Ranges [first, last) of the mixing entries to run as separate launches: one per connected
// group of workers, consecutive groups merged when there are more than kMaxMixLaunches.
constexpr size_t kMaxMixLaunches = 32;
std::vector<std::pair<int32_t, int32_t>> mix_launch_ranges(const std::vector<int32_t> &starts,
                                                           int32_t len) {
  std::vector<std::pair<int32_t, int32_t>> out;
  const size_t per = (starts.size() + kMaxMixLaunches - 1) / kMaxMixLaunches;  // groups per launch
  for (size_t g = 0; g < starts.size(); g += per) {
    const size_t g_end = std::min(g + per, starts.size());
    out.push_back({starts[g], g_end < starts.size() ? starts[g_end] : len});
  }
  return out;
}

// The mixing order of one call, planned on the host; nothing has been launched yet when
// stage_mix returns.
struct StagedMix {
  MixInline order;                     // the order itself, or ...
  const MixSend *d_entries = nullptr;  // ... where it has been uploaded to
  const uint32_t *d_groups = nullptr;
  std::vector<int32_t> starts;         // first entry of each connected group of workers
  int32_t len = 0;                     // entries of all groups together
  bool paced = false;                  // planned for the paced kernel
  int32_t team = 0;                    // > 0: a team's order, entries of its largest group
};

// Whether the fused gossip step takes the paced tiles.  They keep the chip on one
// worker at a time, which pays when a launch over one connected group would walk
// many of them.  Measured with one tensor of 330 to 1555 paced tiles (SGD with fp32
// and Adam with bf16 gradients, time against single waves): groups of 8 or more
// workers 0.83-0.98; groups of 4 0.92-1.01 with 16 or 32 workers, 0.93-1.06 with 8;
// groups of 2 0.93-1.06.  With 4 workers 0.95-1.12.  One large group and pairs, 512 and
// 1536 tiles: 18 workers and 7 pairs 0.91-0.93, 24 and 4 pairs 0.88-0.91, 10 and 3
// pairs 0.92-0.96; random maps of 16 and 32 workers 0.86-0.98.
bool paced_mix(const slowmo_ctx *ctx, const std::vector<MixEntry> &seq) {
  if (ctx->paced.ntiles <= 0) return false;
  if (ctx->tune.paced >= 2) return true;
  const int32_t m = ctx->cfg.m;
  size_t groups = 0;
  for (const MixEntry &e : seq) groups += (e.flags & kMixGroupStart) != 0;
  return m >= kPacedFromWorkers && seq.size() >= groups * (m >= 16 ? 4 : 8);
}

// Whether the local step and the gossip step after it are one kernel.  Not where nobody moves: the
// gossip step is then nothing at all (m = 1, 3 steps: walk over local step 1.02-1.10).  Else always,
// with replicas at any element: those that are not 16-byte aligned share lines between workgroups,
// which costs less than the 8 bytes per element saved and the second launch.  Tensors packed back to
// back, rounds of 4 gossip steps, one kernel over two (SGD and Adam, exponential graph and random
// maps): 3 K and 100 K elements, m = 8 and 21 0.57-0.78; 0.5 to 2 M, m = 4 and 16 0.59-0.90; 6 M,
// m = 16 0.84-0.93; 25.6 M, m = 8 and 20 0.79-0.91; 60 M, m = 3 and 8 0.82-0.91; m = 2 to 5, 2 K to 1 M
// 0.51-0.74, 4 to 40 M 0.68-0.92.
bool fused_mix(const slowmo_ctx *ctx, const int32_t *in_peer) {
  if (!ctx->tune.fuse_mix || ctx->n_otiles == 0) return false;
  bool moves = false;
  for (int32_t i = 0; i < ctx->cfg.m; ++i) moves = moves || in_peer[i] != i;
  return moves;
}

slowmo_status stage_mix(slowmo_ctx *ctx, const int32_t *in_peer, bool with_idle, hipStream_t stream,
                        StagedMix *out, bool may_pace = false) {
  std::vector<MixEntry> seq;
  std::vector<float> share;
  plan_mix(ctx->cfg.m, in_peer, seq, share, with_idle);
  if (may_pace && paced_mix(ctx, seq)) {
    out->paced = true;
    plan_mix(ctx->cfg.m, in_peer, seq, share, with_idle, kPacedSaved);
  }
  if (seq.empty() || ctx->n_otiles == 0) return SLOWMO_OK;  // nothing to launch
  out->len = static_cast<int32_t>(seq.size());
  MixSend *entries = out->order.entry;
  uint32_t *groups = out->order.group;
  int slot = -1;
  if (ctx->cfg.m > kMixInline) {
    hipError_t e = hipSuccess;
    slot = ctx->mixtab.stage(&e);
    if (slot < 0) return fail_hip(ctx, e, "waiting for a staging buffer of the mixing entries");
    entries = static_cast<MixSend *>(ctx->mixtab.h[slot]);
    groups = reinterpret_cast<uint32_t *>(entries + seq.size());
  }
  static_assert(SLOWMO_MAX_WORKERS <= 0xffff, "worker numbers and entry counts fit 16 bits");
  for (int32_t i = 0; i < out->len; ++i) {
    const MixEntry &e = seq[i];
    entries[i] = {static_cast<uint16_t>(e.node), static_cast<uint16_t>(e.src), e.a, e.b,
                  static_cast<uint32_t>(e.flags)};
    if (e.flags & kMixGroupStart) out->starts.push_back(i);
  }
  // One group of at most four workers by itself, walked by up to 10 000 waves' worth of a team, is one
  // short launch either way, and the smaller workgroups' is (pairs, cycles of 3 and 4: team over walk
  // 1.00-1.07; beyond 0.91-1.01).  Pairs side by side: 0.84-0.99 at any length.
  const bool few = !with_idle && out->starts.size() == 1 && out->len <= 4 &&
                   static_cast<int64_t>(ctx->n_otiles) * out->len <= 10000;
  if (!out->paced && !few && mix_by_team(ctx) && (with_idle || !ctx->group_launches)) {
    // On the shortest lists of many workers a workgroup takes one connected group of them, else
    // all: 16 tiles, pairs and groups of 4 and 8, 16 workers 0.92-0.99 and 32 workers 0.70-0.78 of
    // the time; 256 tiles 1.01-1.09.
    if (ctx->cfg.m < 16 || static_cast<int64_t>(ctx->n_otiles) * ctx->cfg.m > 1024) out->starts.assign(1, 0);
    for (size_t g = 0; g < out->starts.size(); ++g) {
      const int32_t at = out->starts[g], end = g + 1 < out->starts.size() ? out->starts[g + 1] : out->len;
      out->team = std::max(out->team, end - at);
    }
    if (out->team <= kTeamMost) {
      std::vector<uint16_t> place(ctx->cfg.m, 0);
      for (size_t g = 0; g < out->starts.size(); ++g) {
        const int32_t at = out->starts[g], end = g + 1 < out->starts.size() ? out->starts[g + 1] : out->len;
        for (int32_t i = at; i < end; ++i) place[entries[i].node] = static_cast<uint16_t>(i - at);
      }
      for (int32_t i = 0; i < out->len; ++i) entries[i].src = place[entries[i].src];
    } else {
      out->team = 0;
    }
  }
  for (size_t g = 0; g < out->starts.size(); ++g) {
    const int32_t end = g + 1 < out->starts.size() ? out->starts[g + 1] : out->len;
    groups[g] = static_cast<uint32_t>(out->starts[g]) |
                static_cast<uint32_t>(end - out->starts[g]) << 16;
  }
  if (slot >= 0) {
    const size_t n_groups = out->starts.size();
    const hipError_t e = ctx->mixtab.send(
        slot, seq.size() * sizeof(MixSend) + n_groups * sizeof(uint32_t), nullptr, stream);
    if (e != hipSuccess) return fail_hip(ctx, e, "upload of the mixing entries");
    out->d_entries = static_cast<const MixSend *>(ctx->mixtab.d[slot]);
    out->d_groups = reinterpret_cast<const uint32_t *>(out->d_entries + seq.size());
  }
  return SLOWMO_OK;
}

// All entries as one range.
MixArgs mix_args(const slowmo_ctx *ctx, const StagedMix &sm) {
  MixArgs a{};
  a.tiles = ctx->d_otiles;
  a.tensors = ctx->d_tensors;
  a.xtab_t = ctx->d_xtab_t;
  a.ntiles = ctx->n_otiles;
  a.m = ctx->cfg.m;
  a.order = &sm.order;
  a.table = sm.d_entries;
  a.groups = sm.d_groups;
  a.len = sm.len;
  a.team = sm.team;
  return a;
}

// Runs a gossip kernel group after group: a workgroup then walks only its group's replicas
// per tile, and fewer memory regions visited side by side measure faster.  As one launch
// over all groups, whose blocks come in that order, or as a launch for each of them, every one
// with a start and a tail of its own.  Rounds on the exponential graph, a launch per group and
// its entries uploaded before, over one launch and the entries in its arguments: 100 K
// elements, m = 8, 8 steps 186 -> 82 us; 200 K, m = 32, 10 steps 614 -> 271 us; 1 M, m = 16, 8 steps
// 510 -> 414 us; 11.7 M, m = 8, 6 steps 2024 -> 1945 us; 25.6 M, m = 32, 12 steps 34.02 -> 33.83 ms.
// *launched: kernels of this call issued so far (a failure is then a failure halfway).
template <typename F>
slowmo_status run_groups(slowmo_ctx *ctx, const StagedMix &sm, MixArgs a, bool one_launch,
                         int *launched, const char *what, F &&launch) {
  std::vector<std::pair<int32_t, int32_t>> ranges;
  if (one_launch) {
    a.n_groups = sm.starts.size() > 1 ? static_cast<int32_t>(sm.starts.size()) : 0;
    if (sm.len > 0) ranges.assign(1, {0, sm.len});
  } else {
    ranges = mix_launch_ranges(sm.starts, sm.len);
  }
  for (const auto &r : ranges) {
    a.first = r.first;
    a.len = r.second - r.first;
    const hipError_t e = guarded(ctx, [&] { return launch(a); });
    if (e != hipSuccess) return *launched ? fail_midway(ctx, e, what) : fail_hip(ctx, e, what);
    ++*launched;
  }
  return SLOWMO_OK;
}

// `launched`: kernels of this call already issued before.
slowmo_status run_mix(slowmo_ctx *ctx, const StagedMix &sm, int launched, hipStream_t stream) {
  const slowmo_status st = run_groups(
      ctx, sm, mix_args(ctx, sm), !ctx->group_launches, &launched, "mixing kernel launch",
      [&](const MixArgs &a) {
        return a.team ? launch_team_mix(nullptr, a, ctx->layout.d_pad, ctx->n_tensors, 0, false, false,
                                        ctx->tune, stream)
                      : launch_mix_step(a, ctx->tune, stream);
      });
  if (st == SLOWMO_OK && sm.len > 0) swept(ctx);
  return st;
}

bool check_in_peer(const slowmo_ctx *ctx, const int32_t *in_peer) {
  for (int32_t i = 0; i < ctx->cfg.m; ++i)
    if (in_peer[i] < 0 || in_peer[i] >= ctx->cfg.m) return false;
  return true;
}

// the push-sum weights mix with the same P, in the same arithmetic as the replicas
void mix_weights(slowmo_ctx *ctx, const int32_t *in_peer) {
  const int32_t m = ctx->cfg.m;
  std::vector<int32_t> outdeg(m, 0);
  for (int32_t i = 0; i < m; ++i)
    if (in_peer[i] != i) ++outdeg[in_peer[i]];
  std::vector<float> w_new(m);
  for (int32_t i = 0; i < m; ++i) {
    const int32_t j = in_peer[i];
    float v = (1.0f / static_cast<float>(1 + outdeg[i])) * ctx->w[i];
    if (j != i) v = v + (1.0f / static_cast<float>(1 + outdeg[j])) * ctx->w[j];
    w_new[i] = v;
  }
  ctx->w.swap(w_new);
}

}  // namespace
}  // extern "C++"

slowmo_status slowmo_mix_step(slowmo_ctx *ctx, const int32_t *in_peer, void *stream_) {
  if (!ctx) return fail(nullptr, SLOWMO_ERR_ARG, "ctx is NULL");
  if (ctx->broken) return fail(ctx, SLOWMO_ERR_STATE, kBrokenMsg);
  if (!in_peer) return fail(ctx, SLOWMO_ERR_ARG, "in_peer is NULL");
  if (!check_in_peer(ctx, in_peer))
    return fail(ctx, SLOWMO_ERR_ARG, "in_peer entries must lie in 0..m-1");
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  StagedMix sm;
  slowmo_status st = stage_mix(ctx, in_peer, /*with_idle=*/false, stream, &sm);
  if (st == SLOWMO_OK) st = run_mix(ctx, sm, 0, stream);
  if (st != SLOWMO_OK) return st;
  mix_weights(ctx, in_peer);
  return SLOWMO_OK;
}

slowmo_status slowmo_local_mix_step(slowmo_ctx *ctx, const void *const *grads, float lr,
                                    const int32_t *in_peer, void *stream_) {
  if (!ctx) return fail(nullptr, SLOWMO_ERR_ARG, "ctx is NULL");
  if (ctx->broken) return fail(ctx, SLOWMO_ERR_STATE, kBrokenMsg);
  if (!in_peer) return fail(ctx, SLOWMO_ERR_ARG, "in_peer is NULL");
  if (!check_in_peer(ctx, in_peer))
    return fail(ctx, SLOWMO_ERR_ARG, "in_peer entries must lie in 0..m-1");
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  LocalArgs a{};
  slowmo_status st = prepare_local(ctx, grads, lr, stream, &a);
  if (st != SLOWMO_OK) return st;
  const slowmo_config &c = ctx->cfg;
  const bool bf16 = c.grad_dtype == SLOWMO_BF16;
  const bool two_kernels = !fused_mix(ctx, in_peer);
  // both tables are on their way to the device before the first kernel is launched
  StagedMix sm;
  st = stage_mix(ctx, in_peer, /*with_idle=*/!two_kernels, stream, &sm, /*may_pace=*/!two_kernels);
  if (st != SLOWMO_OK) return st;
  if (two_kernels) {
    // same kernels as the separate calls
    const hipError_t e = guarded(ctx, [&] {
      return launch_local_step(a, c.base, bf16, ctx->buffers_zero, !a.keep, ctx->tune, stream);
    });
    if (e != hipSuccess) return fail_hip(ctx, e, "local-step kernel launch");
    swept(ctx);
    st = run_mix(ctx, sm, 1, stream);
    if (st != SLOWMO_OK) return st;
  } else {
    MixArgs x = mix_args(ctx, sm);
    int launched = 0;
    bool one_launch = true;
    if (sm.paced) {
      const hipError_t e = guarded(ctx, [&] {
        return launch_local_mix_paced(a, x, ctx->layout.d_pad, ctx->n_tensors, c.base, bf16,
                                      ctx->buffers_zero, ctx->paced, stream);
      });
      if (e != hipSuccess) return fail_hip(ctx, e, "paced local+mixing kernel launch");
      ++launched;
      x.tiles = ctx->d_prtiles;
      x.ntiles = ctx->n_prtiles;
      if (!ctx->prtiles_by_group) sm.starts.assign(1, 0);
      one_launch = !ctx->prtiles_by_group;
    }
    if (x.ntiles > 0) {
      st = run_groups(ctx, sm, x, one_launch, &launched, "fused local+mixing kernel launch",
                      [&](const MixArgs &r) {
                        if (r.team)
                          return launch_team_mix(&a, r, ctx->layout.d_pad, ctx->n_tensors, c.base,
                                                 bf16, ctx->buffers_zero, ctx->tune, stream);
                        return launch_local_mix_step(a, r, ctx->layout.d_pad, ctx->n_tensors, c.base,
                                                     bf16, ctx->buffers_zero, ctx->tune, stream);
                      });
      if (st != SLOWMO_OK) return st;
    }
    swept(ctx, sm.paced);
  }
  // counters and weights move only after the last launch was accepted
  finish_local(ctx, /*gossip=*/!two_kernels);
  mix_weights(ctx, in_peer);
  return SLOWMO_OK;
}

int32_t slowmo_plan_mix(int32_t m, const int32_t *in_peer, slowmo_mix_entry *out) {
  static_assert(sizeof(slowmo_mix_entry) == sizeof(MixEntry), "public and internal entry differ");
  static_assert(SLOWMO_MIX_SAVE(5 << 6) == mix_save(5 << 6) && mix_save(5 << 6) == 5 &&
                    SLOWMO_MIX_OWN_SAVED(5 << 9) == mix_own_saved(5 << 9) &&
                    mix_own_saved(5 << 9) == 5 &&
                    SLOWMO_MIX_SOURCE_SAVED(5 << 12) == mix_src_saved(5 << 12) &&
                    mix_src_saved(5 << 12) == 5 && SLOWMO_MIX_SAVED_REGISTERS == kMixSaved &&
                    SLOWMO_MIX_GROUP_START == kMixGroupStart,
                "public and internal flags differ");
  if (m < 1 || m > SLOWMO_MAX_WORKERS || !in_peer || !out) return -1;
  for (int32_t i = 0; i < m; ++i)
    if (in_peer[i] < 0 || in_peer[i] >= m) return -1;
  std::vector<MixEntry> seq;
  std::vector<float> share;
  plan_mix(m, in_peer, seq, share);
  for (size_t i = 0; i < seq.size(); ++i)
    out[i] = {seq[i].node, seq[i].src, seq[i].a, seq[i].b, seq[i].flags & ~kMixSrcDone, 0};
  return static_cast<int32_t>(seq.size());
}

slowmo_status slowmo_get_pushsum_weights(const slowmo_ctx *ctx, float *w) {
  if (!ctx) return fail(nullptr, SLOWMO_ERR_ARG, "ctx is NULL");
  if (!w) return fail(const_cast<slowmo_ctx *>(ctx), SLOWMO_ERR_ARG, "w is NULL");
  std::memcpy(w, ctx->w.data(), ctx->w.size() * sizeof(float));
  return SLOWMO_OK;
}

extern "C++" {
namespace {

// z = x / w for every worker.  The table the kernel reads (m * n_tensors destination
// pointers, and the m weights if there are more than kMixInline or table_dev is given) is
// written straight into a pinned staging buffer of the context and sent to `table_dev`
// (NULL: the staging slot's own device copy inside the workspace, which is not sent again
// when a recent call had these very pointers).  Allocates nothing.  Rounds of gossip steps on
// random maps, de-biased after each, all of the table sent with every call before / now: 18 K
// elements, m = 7, 13 steps 282 / 173 us; 16 K in 204 tensors, m = 3, 6 steps 116 / 67 us;
// ResNet-18-shaped, m = 16, 4 steps 4179 / 4161 us.
slowmo_status debias_into(slowmo_ctx *ctx, float *const *z, void *table_dev, hipStream_t stream) {
  if (ctx->broken) return fail(ctx, SLOWMO_ERR_STATE, kBrokenMsg);
  if (!z) return fail(ctx, SLOWMO_ERR_ARG, "z is NULL");
  const int32_t m = ctx->cfg.m, nt = ctx->n_tensors;
  const size_t n_ptr = static_cast<size_t>(m) * nt;
  const bool inline_w = m <= kMixInline && !table_dev;
  int slot = inline_w ? ctx->ztab.find(z, n_ptr * sizeof(void *)) : -1;
  if (slot < 0) {  // (the pointers of a recent call passed these checks)
    for (size_t i = 0, j = 0; i < n_ptr; ++i, j = j + 1 == ctx->numel.size() ? 0 : j + 1) {
      if (ctx->numel[j] == 0) continue;
      if (!z[i]) return fail(ctx, SLOWMO_ERR_ARG, "a destination pointer is NULL");
      if (reinterpret_cast<uintptr_t>(z[i]) % sizeof(float))
        return fail(ctx, SLOWMO_ERR_ALIGN, "a destination pointer is not 4-byte aligned");
    }
  }
  if (ctx->check_pointers >= 2) {
    for (size_t i = 0; i < n_ptr; ++i) {
      const int64_t n = ctx->numel[i % nt];
      if (n && slowmo_check_device_range(z[i], static_cast<size_t>(n) * sizeof(float)) != SLOWMO_OK)
        return fail(ctx, SLOWMO_ERR_ARG, "destination tensor: " + g_err);
    }
  }
  if (ctx->n_ltiles == 0) return SLOWMO_OK;
  hipError_t e = hipSuccess;
  if (slot < 0) {
    slot = ctx->ztab.stage(&e);
    if (slot < 0) return fail_hip(ctx, e, "waiting for a staging buffer of the de-bias table");
    char *table = static_cast<char *>(ctx->ztab.h[slot]);
    std::memcpy(table, z, n_ptr * sizeof(void *));
    std::memcpy(table + n_ptr * sizeof(void *), ctx->w.data(), m * sizeof(float));
    e = ctx->ztab.send(slot, inline_w ? n_ptr * sizeof(void *) : ztab_bytes(m, nt), table_dev, stream);
    if (e != hipSuccess) return fail_hip(ctx, e, "upload of the de-bias table");
  }
  const char *dev = static_cast<const char *>(table_dev ? table_dev : ctx->ztab.d[slot]);
  DebiasArgs a{};
  a.tiles = ctx->d_ltiles;
  a.slots = ctx->d_slots;
  a.ztab = reinterpret_cast<float *const *>(dev);
  DebiasWeights weights{};
  if (inline_w) {
    std::copy(ctx->w.begin(), ctx->w.end(), weights.w);
    a.inl = &weights;
  } else {
    a.w = reinterpret_cast<const float *>(dev + n_ptr * sizeof(void *));
  }
  a.ntiles = ctx->n_ltiles;
  a.n_tensors = nt;
  e = guarded(ctx, [&] { return launch_debias(a, ctx->tune, stream); });
  if (e != hipSuccess) return fail_hip(ctx, e, "de-bias kernel launch");
  swept(ctx);
  return SLOWMO_OK;
}

}  // namespace
}  // extern "C++"

slowmo_status slowmo_debias(slowmo_ctx *ctx, float *const *z, void *stream_) {
  if (!ctx) return fail(nullptr, SLOWMO_ERR_ARG, "ctx is NULL");
  return debias_into(ctx, z, nullptr, static_cast<hipStream_t>(stream_));
}

slowmo_status slowmo_debias_static(slowmo_ctx *ctx, float *const *z, void *stream_) {
  static_assert(SLOWMO_STATIC_MAX_POINTERS == kStaticMaxPointers, "header and library disagree");
  static_assert(SLOWMO_MAX_WORKERS <= kStaticMaxWorkers, "weights must fit the static table");
  if (!ctx) return fail(nullptr, SLOWMO_ERR_ARG, "ctx is NULL");
  const size_t n_ptr = static_cast<size_t>(ctx->cfg.m) * ctx->n_tensors;
  if (n_ptr > kStaticMaxPointers)
    return fail(ctx, SLOWMO_ERR_NOMEM,
                "m * n_tensors = " + std::to_string(n_ptr) + " exceeds SLOWMO_STATIC_MAX_POINTERS = " +
                    std::to_string(kStaticMaxPointers) + ": use slowmo_debias");
  int current = -1;
  const hipError_t e = hipGetDevice(&current);
  if (e != hipSuccess) return fail_hip(ctx, e, "hipGetDevice");
  if (current != ctx->device)
    return fail(ctx, SLOWMO_ERR_STATE, "the context's device is not the current device");
  return debias_into(ctx, z, ctx->static_table, static_cast<hipStream_t>(stream_));
}

slowmo_status slowmo_set_tensor_hparams(slowmo_ctx *ctx, const float *weight_decay,
                                        const float *lr_scale, void *stream_) {
  if (!ctx) return fail(nullptr, SLOWMO_ERR_ARG, "ctx is NULL");
  const int32_t nt = ctx->n_tensors, m = ctx->cfg.m;
  for (int32_t j = 0; j < nt; ++j) {
    if (weight_decay && !(std::isfinite(weight_decay[j]) && weight_decay[j] >= 0.f))
      return fail(ctx, SLOWMO_ERR_ARG, "weight_decay entries must be finite and >= 0");
    if (lr_scale && !finite_pos(lr_scale[j]))
      return fail(ctx, SLOWMO_ERR_ARG, "lr_scale entries must be finite and > 0");
  }
  // build the new tables aside; they replace the context's only if the upload succeeds
  std::vector<SlotInfo> slots = ctx->slots;
  std::vector<TensorInfo> tinfo = ctx->tinfo;
  for (int32_t j = 0; j < nt; ++j) {
    if (lr_scale) tinfo[j].lr_scale = lr_scale[j];
    if (weight_decay) tinfo[j].wd = weight_decay[j];
    for (int32_t w = 0; w < m; ++w) {
      SlotInfo &s = slots[static_cast<size_t>(w) * nt + j];
      if (weight_decay) s.wd = weight_decay[j];
      if (lr_scale) s.lr_scale = lr_scale[j];
    }
  }
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  hipError_t e = hipMemcpyAsync(ctx->d_slots, slots.data(), slots.size() * sizeof(SlotInfo),
                                hipMemcpyHostToDevice, stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(ctx->d_tensors, tinfo.data(), tinfo.size() * sizeof(TensorInfo),
                       hipMemcpyHostToDevice, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);  // the tables above go out of scope
  if (e != hipSuccess) return fail_hip(ctx, e, "upload of the per-tensor hyper-parameters");
  ctx->slots.swap(slots);
  ctx->tinfo.swap(tinfo);
  return SLOWMO_OK;
}

extern "C++" {
namespace {

// Header of an exported state blob (256 bytes), followed by the m push-sum
// weights (padded to a multiple of 256 bytes) and the x0, u, h, v arenas
// exactly as they lie in the workspace.
struct BlobHeader {
  char magic[8];
  uint32_t version;
  int32_t m, n_tensors, base, no_average, k, buffers_zero, reserved;
  int64_t d, d_pad, t, l;
  char pad_[256 - 8 - 4 * 8 - 8 * 4];
};
static_assert(sizeof(BlobHeader) == 256, "BlobHeader layout");
constexpr uint32_t kBlobVersion = 2;
constexpr char kBlobMagic[8] = {'S', 'L', 'O', 'W', 'M', 'O', 'S', 'T'};

struct BlobParts {
  size_t arena, outer_copies, n_v, weights, total;
};
BlobParts blob_parts(const slowmo_ctx *ctx) {
  BlobParts p;
  p.arena = static_cast<size_t>(ctx->layout.d_pad) * sizeof(float);
  p.outer_copies = ctx->cfg.no_average ? ctx->cfg.m : 1;
  p.n_v = ctx->v ? ctx->cfg.m : 0;
  p.weights = round_up(static_cast<size_t>(ctx->cfg.m) * sizeof(float), 256);
  p.total = sizeof(BlobHeader) + p.weights + p.arena * (2 * p.outer_copies + ctx->cfg.m + p.n_v);
  return p;
}

}  // namespace
}  // extern "C++"

size_t slowmo_export_bytes(const slowmo_ctx *ctx) { return ctx ? blob_parts(ctx).total : 0; }

slowmo_status slowmo_export_state(slowmo_ctx *ctx, void *dst, size_t bytes, void *stream_) {
  if (!ctx) return fail(nullptr, SLOWMO_ERR_ARG, "ctx is NULL");
  if (!dst) return fail(ctx, SLOWMO_ERR_ARG, "dst is NULL");
  const BlobParts p = blob_parts(ctx);
  if (bytes < p.total) return fail(ctx, SLOWMO_ERR_NOMEM, "destination smaller than slowmo_export_bytes()");
  BlobHeader hd{};
  std::memcpy(hd.magic, kBlobMagic, 8);
  hd.version = kBlobVersion;
  hd.m = ctx->cfg.m;
  hd.n_tensors = ctx->n_tensors;
  hd.base = ctx->cfg.base;
  hd.no_average = ctx->cfg.no_average;
  hd.d = ctx->layout.d;
  hd.d_pad = ctx->layout.d_pad;
  hd.t = ctx->t;
  hd.l = ctx->l;
  hd.k = ctx->k;
  hd.buffers_zero = ctx->buffers_zero ? 1 : 0;
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  char *out = static_cast<char *>(dst);
  hipError_t e = hipMemcpyAsync(out, &hd, sizeof(hd), hipMemcpyHostToDevice, stream);
  size_t off = sizeof(hd);
  if (e == hipSuccess)
    e = hipMemcpyAsync(out + off, ctx->w.data(), ctx->w.size() * sizeof(float),
                       hipMemcpyHostToDevice, stream);
  off += p.weights;
  auto put = [&](const float *src, size_t n) {
    if (e == hipSuccess && n)
      e = hipMemcpyAsync(out + off, src, n, hipMemcpyDeviceToDevice, stream);
    off += n;
  };
  put(ctx->x0, p.arena * p.outer_copies);
  put(ctx->u, p.arena * p.outer_copies);
  put(ctx->h, p.arena * ctx->cfg.m);
  put(ctx->v, p.arena * p.n_v);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);  // the header lives on this stack frame
  if (e != hipSuccess) return fail_hip(ctx, e, "state export");
  return SLOWMO_OK;
}

slowmo_status slowmo_import_state(slowmo_ctx *ctx, const void *src, size_t bytes, void *stream_) {
  if (!ctx) return fail(nullptr, SLOWMO_ERR_ARG, "ctx is NULL");
  if (ctx->broken) return fail(ctx, SLOWMO_ERR_STATE, kBrokenMsg);
  if (!src) return fail(ctx, SLOWMO_ERR_ARG, "src is NULL");
  const BlobParts p = blob_parts(ctx);
  if (bytes < p.total) return fail(ctx, SLOWMO_ERR_ARG, "blob shorter than this context's state");
  hipStream_t stream = static_cast<hipStream_t>(stream_);
  BlobHeader hd{};
  hipError_t e = hipMemcpyAsync(&hd, src, sizeof(hd), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return fail_hip(ctx, e, "reading the blob header");
  if (std::memcmp(hd.magic, kBlobMagic, 8) != 0 || hd.version != kBlobVersion)
    return fail(ctx, SLOWMO_ERR_ARG, "not a state blob of this library version");
  if (hd.m != ctx->cfg.m || hd.n_tensors != ctx->n_tensors || hd.base != ctx->cfg.base ||
      hd.no_average != ctx->cfg.no_average || hd.d != ctx->layout.d || hd.d_pad != ctx->layout.d_pad)
    return fail(ctx, SLOWMO_ERR_ARG, "the blob was exported from a different configuration or tensor list");
  if (hd.k < 0 || hd.k > ctx->cfg.tau || hd.t < 0 || hd.l < 0 ||
      (hd.buffers_zero != 0 && hd.buffers_zero != 1))
    return fail(ctx, SLOWMO_ERR_ARG, "the blob's counters do not fit this configuration");
  const char *in = static_cast<const char *>(src);
  size_t off = sizeof(hd);
  std::vector<float> w(ctx->cfg.m);
  e = hipMemcpyAsync(w.data(), in + off, w.size() * sizeof(float), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return fail_hip(ctx, e, "reading the blob's push-sum weights");
  for (float wi : w)
    if (!finite_pos(wi)) return fail(ctx, SLOWMO_ERR_ARG, "the blob's push-sum weights are not positive");
  off += p.weights;
  // everything checkable has been checked: only now is the context touched
  bool copied = false;
  auto get = [&](float *dst, size_t n) {
    if (e == hipSuccess && n) {
      e = hipMemcpyAsync(dst, in + off, n, hipMemcpyDeviceToDevice, stream);
      copied = copied || e == hipSuccess;
    }
    off += n;
  };
  get(ctx->x0, p.arena * p.outer_copies);
  get(ctx->u, p.arena * p.outer_copies);
  get(ctx->h, p.arena * ctx->cfg.m);
  get(ctx->v, p.arena * p.n_v);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess)
    return copied ? fail_midway(ctx, e, "state import") : fail_hip(ctx, e, "state import");
  ctx->t = hd.t;
  ctx->k = hd.k;
  ctx->l = hd.l;
  ctx->buffers_zero = hd.buffers_zero != 0;
  ctx->w.swap(w);
  return SLOWMO_OK;
}

slowmo_status slowmo_destroy(slowmo_ctx *ctx) {
  if (!ctx) return SLOWMO_OK;
  release(ctx);
  return SLOWMO_OK;
}

slowmo_status slowmo_get_buffer(slowmo_ctx *ctx, int32_t which, int32_t worker, int32_t tensor,
                                float **device_ptr) {
  if (!ctx) return fail(nullptr, SLOWMO_ERR_ARG, "ctx is NULL");
  if (!device_ptr) return fail(ctx, SLOWMO_ERR_ARG, "device_ptr is NULL");
  if (tensor < 0 || tensor >= ctx->n_tensors) return fail(ctx, SLOWMO_ERR_ARG, "tensor index out of range");
  const int64_t off = ctx->layout.arena_off[tensor];
  switch (which) {
    case SLOWMO_BUF_X0:
    case SLOWMO_BUF_U: {
      int64_t woff = 0;
      if (ctx->cfg.no_average) {
        if (worker < 0 || worker >= ctx->cfg.m) return fail(ctx, SLOWMO_ERR_ARG, "worker index out of range");
        woff = static_cast<int64_t>(worker) * ctx->layout.d_pad;
      }
      *device_ptr = (which == SLOWMO_BUF_X0 ? ctx->x0 : ctx->u) + woff + off;
      return SLOWMO_OK;
    }
    case SLOWMO_BUF_H:
    case SLOWMO_BUF_V: {
      if (worker < 0 || worker >= ctx->cfg.m) return fail(ctx, SLOWMO_ERR_ARG, "worker index out of range");
      float *b = which == SLOWMO_BUF_H ? ctx->h : ctx->v;
      if (!b) return fail(ctx, SLOWMO_ERR_ARG, "this base optimizer has no v buffer");
      *device_ptr = b + static_cast<int64_t>(worker) * ctx->layout.d_pad + off;
      return SLOWMO_OK;
    }
    default: return fail(ctx, SLOWMO_ERR_ARG, "unknown buffer id");
  }
}

slowmo_status slowmo_get_counters(const slowmo_ctx *ctx, int64_t *t, int32_t *k, int64_t *l) {
  if (!ctx) return fail(nullptr, SLOWMO_ERR_ARG, "ctx is NULL");
  if (t) *t = ctx->t;
  if (k) *k = ctx->k;
  if (l) *l = ctx->l;
  return SLOWMO_OK;
}

}  // extern "C"
