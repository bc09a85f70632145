// Launch interface between the C ABI (host logic) and the gfx950 kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "slowmo_plan.h"

namespace slowmo {

struct LocalArgs {
  const TileRef *tiles;        // device, ntiles entries (owner = slot)
  const SlotInfo *slots;       // device, m * n_tensors entries
  const void *const *gtab;     // device: m * n_tensors gradient pointers of this call
  int32_t ntiles;
  float *h;                    // device: h arena, m * d_pad
  float *v;                    // device: v arena (Adam) or nullptr
  int32_t keep;                // 0: the gossip kernels do not store h and v (dead after this step)
  float lr;
  float wd;
  // SGD with Nesterov momentum
  float mu;
  // Adam: factors and reciprocal bias corrections 1 / (1 - beta^l)
  float b1, b2, omb1, omb2, rc1, rc2, eps;
};

struct OuterArgs {
  const TileRef *tiles;        // device, ntiles entries (owner = tensor)
  const TensorInfo *tensors;   // device, n_tensors entries
  float *const *xtab_t;        // device: replica pointers, tensor-major: [tensor * m + worker]
  int32_t ntiles;
  int32_t m;
  float *x0;                   // device: arena d_pad
  float *u;                    // device: arena d_pad
  float lr;                    // gamma_t (scaled per tensor in the kernel)
  float alpha;                 // slow learning rate; (alpha * gamma_t) is rounded once to fp32
  float beta;
  float m_f;                   // (float) m
  // buffer strategy "average": arenas to average over the workers (nullptr = skip)
  float *avg_h;
  float *avg_v;
  int64_t d_pad;               // worker stride of the arenas, elements
};

// Outer step without the exact average: lines 7-8 per (worker, element) with
// per-worker x0 and u arenas (m * d_pad each), over the local-step tiles.
struct OuterNoAvgArgs {
  const TileRef *tiles;        // device (owner = slot)
  const SlotInfo *slots;       // device
  int32_t ntiles;
  float *x0;                   // device: m * d_pad
  float *u;                    // device: m * d_pad
  float lr, alpha, beta;
};

// The mixing order as the kernels read it: one entry is one 16-byte scalar load.
struct MixSend {
  uint16_t node, src;
  float a, b;
  uint32_t flags;
};
static_assert(sizeof(MixSend) == 16, "MixSend layout");
// It travels with the launch, in the kernel's arguments, where it has at most kMixInline
// entries; a longer one is a table in the workspace (the entries, then the groups).  Every launch
// copies room for all of them: 64 instead of 32 take 0.1 us more on the host (rounds of 12 steps on
// 4 to 8 workers 73-78 -> 72-76 us, with the de-biased parameters after each 128-133 -> 124-130).
constexpr int32_t kMixInline = 32;
constexpr int32_t kTeamMost = 32;  // workers that a team takes
struct MixInline {
  MixSend entry[kMixInline];
  uint32_t group[kMixInline];  // connected groups of workers: first entry, number of entries << 16
};

struct MixArgs {
  const TileRef *tiles;        // device: outer-step tiles (owner = tensor)
  const TensorInfo *tensors;   // device
  float *const *xtab_t;        // device: replica pointers, tensor-major
  int32_t ntiles;
  int32_t m;
  const MixInline *order;      // host: the mixing order, or ...
  const MixSend *table;        // ... device: its entries
  const uint32_t *groups;      // ... and its groups (nullptr: one range from `first` on)
  int32_t n_groups;            // groups to run side by side in one launch (0: the entries
  int32_t first, len;          // [first, first + len))
  int32_t team;                // > 0: a team's order (see launch_team_mix), entries of its largest group
};

// Tiles of a paced walk (see kPacedTile), and what its workgroups pace each other with.
struct PacedArgs {
  const TileRef *tiles;        // device: whole kPacedTile pieces (owner = tensor)
  int32_t ntiles;
  int32_t members;             // workgroups per XCD: its number of CUs
  const TileRef *rest;         // device: ordinary tiles for the workgroups without a piece in the
  int32_t nrest;               // last row (0: they run as a launch of their own)
  int32_t spins;               // polls after which a workgroup stops waiting for the others
  uint32_t *counters;          // device: kPaceWords words, zero between launches
};

struct DebiasWeights {
  float w[kMixInline];
};
// De-biased parameters of push-sum: z^{(i)} = x^{(i)} / w_i, over the local tiles.
struct DebiasArgs {
  const TileRef *tiles;        // device (owner = slot)
  const SlotInfo *slots;       // device
  float *const *ztab;          // device: m * n_tensors destination pointers (worker-major)
  const float *w;              // device: m push-sum weights, or nullptr:
  const DebiasWeights *inl;    // host: the weights travel with the launch
  int32_t ntiles;
  int32_t n_tensors;
};

struct LaunchTuning {
  int32_t xcd_remap;    // 1: consecutive tiles go to the same XCD
  int32_t xcd_run;      // tiles an XCD takes in a row before the next XCD's run; 0 = one
                        // contiguous eighth of all tiles per XCD
  int32_t backward;     // 1: every XCD walks its contiguous eighth from the end to the start;
                        // changes with every sweep over the tiles
  int32_t nontemporal;  // 1: streaming (non-temporal) loads and stores
  int32_t fuse_last;    // 1: slowmo_local_outer_step runs one fused kernel when it can
  int32_t fuse_mix;     // 1: slowmo_local_mix_step runs one fused kernel when it can
  int32_t paced;        // the fused gossip step on paced tiles: 0 never, 1 by the rule, 2 wherever
                        // the kernel allows
  int32_t big_tiles;    // 1: whole big tiles of aligned tensors go to the big-tile kernels
  int32_t big_vpt;      // vectors per lane of a big tile: 16, 14 or 12
  int32_t local_nt;     // 1: streaming accesses in the local step and k_mix_step (0: their working set
                        // stays in the caches)
  int32_t mix_nt;       // the same for k_local_mix_step and the loads of the de-biasing
  int32_t outer_nt;     // ... for the outer step in single waves
  int32_t last_nt;      // ... for the fused last step in single waves
  int32_t kept_local;   // 1: some of the local-step tiles are kept (kTileKept)
  int32_t kept_tiles;   // 1: the fused last step reads kept outer-step tiles as such where
                        // last_keeps says so (2: on every list)
  int32_t kept_mix;     // the same for the gossip step fused with the local step (mix_keeps)
  int32_t kept_outer;   // 1: the outer step reads them as such
  int32_t write_through;  // 1: the local step writes through the L2 (sc1 stores)
  int32_t noavg_through;  // the same for the outer step without the average by itself
  int32_t local_lds;    // bytes of (unused) dynamic LDS per workgroup of the local step: caps the
                        // wavefronts per CU
  int32_t noavg_lds;    // the same for the outer step without the average
  int32_t outer_lds;    // the same for the outer step (160 KiB / outer_lds wavefronts per CU; 0 = no
                        // cap)
  int32_t last_lds;     // the same for the fused last step
};

// base: 0 SGD-Nesterov, 1 Adam.  bf16: gradient dtype.  first: the stored
// h (and v) are to be read as zero (first step after a reset / after create).
// last: h (and v) are dead after this step and are not written.
hipError_t launch_local_step(const LocalArgs &a, int base, bool bf16, bool first, bool last,
                             const LaunchTuning &tune, hipStream_t stream);
hipError_t launch_outer_step(const OuterArgs &a, const LaunchTuning &tune, hipStream_t stream);
// The last local step of an outer iteration and the outer step in one pass
// (one workgroup = 256 elements of one tensor, all workers).  policy:
// 0 reset (buffers not stored), 1 maintain (stored), 2 average (their mean
// over the workers is stored).
hipError_t launch_local_outer_step(const LocalArgs &l, const OuterArgs &o, int32_t n_tensors,
                                   int base, bool bf16, bool first, int policy,
                                   const LaunchTuning &tune, hipStream_t stream);
// The same two operations on BIG tiles (a.tiles / o.tiles list whole pieces of
// big_tile(tune.big_vpt) elements, every one full, of tensors all of whose replicas are 16-byte aligned).  Results are
// bit-identical to the ordinary tiles'.  launch_outer_big handles no buffer
// average (a.avg_h must be NULL); launch_local_outer_big handles policies 0 and 1.
hipError_t launch_outer_big(const OuterArgs &a, const LaunchTuning &tune, hipStream_t stream);
hipError_t launch_local_outer_big(const LocalArgs &l, const OuterArgs &o, int32_t n_tensors,
                                  int base, bool bf16, bool first, int policy,
                                  const LaunchTuning &tune, hipStream_t stream);
// Copies worker 0's replica into x0 (x0_copies copies, d_pad apart) and into the
// replicas of workers 1..m-1; uses a.tiles, a.tensors, a.xtab_t, a.x0, a.d_pad, a.m.
hipError_t launch_init_broadcast(const OuterArgs &a, int32_t x0_copies, const LaunchTuning &tune,
                                 hipStream_t stream);
hipError_t launch_mix_step(const MixArgs &a, const LaunchTuning &tune,
                              hipStream_t stream);
// The local step and the mixing step that follows it in one kernel; the order must
// list EVERY worker (plan_mix with idle workers).
hipError_t launch_local_mix_step(const LocalArgs &l, const MixArgs &x, int64_t d_pad,
                                 int32_t n_tensors, int base, bool bf16, bool first,
                                 const LaunchTuning &tune, hipStream_t stream);
// The same on paced tiles (whole kPacedTile pieces of any tensors); the order must come
// from plan_mix with saved_limit = kPacedSaved.
hipError_t launch_local_mix_paced(const LocalArgs &l, const MixArgs &x, int64_t d_pad,
                                  int32_t n_tensors, int base, bool bf16, bool first,
                                  const PacedArgs &p, hipStream_t stream);
// The gossip step by itself (l = nullptr) or fused with the local step, with a wave per worker on
// every tile, for short lists.  In a team's order src is the place of the source in its group
// (x.team <= kTeamMost).
hipError_t launch_team_mix(const LocalArgs *l, const MixArgs &x, int64_t d_pad, int32_t n_tensors,
                           int base, bool bf16, bool first, const LaunchTuning &tune,
                           hipStream_t stream);
// The outer step, after the last local step or by itself (l = nullptr), in the same way.
hipError_t launch_team_outer(const LocalArgs *l, const OuterArgs &o, int32_t n_tensors, int base,
                             bool bf16, bool first, int policy, const LaunchTuning &tune,
                             hipStream_t stream);
hipError_t launch_debias(const DebiasArgs &a, const LaunchTuning &tune, hipStream_t stream);

// Static device memory for the entry point that allocates nothing: room for
// the de-bias table (destination pointers, then the push-sum weights) of up to
// kStaticMaxPointers (worker, tensor) pairs.
constexpr size_t kStaticMaxPointers = 65536;
constexpr size_t kStaticMaxWorkers = 1024;
constexpr size_t kStaticScratchBytes =
    kStaticMaxPointers * sizeof(void *) + kStaticMaxWorkers * sizeof(float);
// Address of that memory on `device`.  The first call for a device must be made
// with that device current (it asks the runtime for the symbol's address
// there); later calls return the remembered address without any HIP call.
hipError_t static_scratch(int device, void **ptr);
hipError_t launch_outer_noavg_step(const OuterNoAvgArgs &a, const LaunchTuning &tune,
                                   hipStream_t stream);
// The last local step and the outer step without the average in one pass (first, last: as for
// launch_local_step).
hipError_t launch_local_noavg_step(const LocalArgs &l, const OuterNoAvgArgs &o, int base, bool bf16,
                                   bool first, bool last, const LaunchTuning &tune, hipStream_t stream);

}  // namespace slowmo
