// Host-side tiling of the tensor list into workgroup-sized units of work, and
// the device-visible descriptors the kernels read.  No HIP calls here.
//
// Measured on MI355X: the stream mix of this path (3-4 reads, 2-3 writes per
// element) runs fastest with many short-lived workgroups that each move one
// 16-byte vector per lane and retire, dispatched in memory order; looping
// (persistent) workgroups and larger tiles lose 15-20 % of bandwidth unless they
// keep each other's company (big and paced tiles below).  An ordinary tile is
// therefore small, and holds exactly one contiguous run of one tensor.
#pragma once

#include <cstdint>
#include <vector>

namespace slowmo {

// Every tensor's slice of x0 / u / h / v starts at a multiple of 64 floats
// (256 bytes) in the state arena, so the state side of a tile is 16-byte
// aligned (tiles start at multiples of 4 elements of their tensor).
constexpr int64_t kArenaAlign = 64;

// Threads per workgroup; a tile is one vec4 per lane.  Single-wavefront workgroups
// measured best for both kernels (64 > 128 > 256 > 512), and the lanes of a tile's end
// rely on them.
constexpr int32_t kLocalBlock = 64;
constexpr int32_t kLocalTile = 4 * kLocalBlock;
constexpr int32_t kOuterBlock = 64;
constexpr int32_t kOuterTile = 4 * kOuterBlock;

// Big tiles of the outer step and of the fused last step: one 1024-thread
// workgroup takes kBigVpt vectors per lane (or a few less), i.e. 256 KiB of every stream
// it walks (its 16 waves start together and move from replica to replica
// together).  Measured in one process on the same replicas against the
// single-wave tiles: the fused last step is 10-14 % faster at m = 32, 6-7 % at
// m = 16, 3-5 % at m = 8 and no faster at m = 4; the plain outer step 8 % faster
// at m = 32 and within +-4 % at m = 8.  Smaller shapes (128 or 64 KiB per stream
// and workgroup) gain half of that or nothing.  Under "maintain" the fused
// kernel stores every worker's buffers inside the walk and is 2-10 % slower in
// this shape than in single waves, so it takes big tiles only under "reset".
// Used for the whole pieces of aligned tensors from these worker counts on:
constexpr int32_t kBigBlock = 1024;
constexpr int32_t kBigVpt = 16;
// Tiles of 14 or 12 vectors per lane instead of 16, where they fill the chip's rounds
// better (choose_big_vpt).
constexpr int32_t kBigVptMin = 12;
constexpr int32_t big_tile(int32_t vpt) { return 4 * kBigBlock * vpt; }
constexpr int32_t kBigFusedFromWorkers = 8;
constexpr int32_t kBigOuterFromWorkers = 16;
// ... and only when there are enough of them to occupy the chip: one big tile
// keeps one of the 256 CUs busy.  Measured on one tensor of k big tiles (m = 8
// and 32): twice as slow as single-wave tiles at k = 64, 6-17 % slower at
// k = 128, 4-15 % faster from k = 173 on.
constexpr int32_t kBigMinTiles = 160;
static_assert(big_tile(1) % kOuterTile == 0, "a big tile is a whole number of ordinary tiles");

// Paced tiles of the fused gossip step: one 512-thread workgroup per CU, 8 vectors per
// lane, 64 KiB of a stream per tile.
constexpr int32_t kPacedBlock = 512;
constexpr int32_t kPacedVpt = 8;
constexpr int32_t kPacedTile = 4 * kPacedBlock * kPacedVpt;
constexpr int32_t kPacedFromWorkers = 8;
// Pieces a list must have: a full row and some to go with its second launch.
constexpr int32_t kPacedMinTiles = 300;
constexpr int32_t kPacedShortFromWorkers = 17;         // aligned lists of less than two rows: see paced_pays
constexpr int64_t kPacedFromBytes = 2200000000;        // bytes that a step reads, from which pacing pays,
constexpr int64_t kPacedPackedFromBytes = 1750000000;  // ... on replicas that are not 16-byte aligned
constexpr int32_t kPacedSaved = 2;      // saved values of the gossip walk (kMixSaved in single waves)
constexpr int32_t kPaceStride = 128;    // words between the counters of two XCDs
constexpr int32_t kPaceWords = 8 * kPaceStride + kPaceStride;
constexpr int32_t kPaceSpins = 300;
constexpr int32_t kRestPerWave = 6;     // left-over tiles that a wave takes during a last row
constexpr int32_t kRestMost = 1200;     // ... and that all of them take
static_assert(kPacedTile % kOuterTile == 0, "a paced tile is a whole number of ordinary tiles");

// One tile of either kernel: the k-th piece of a tensor.  For the local step
// `owner` is the slot (worker * n_tensors + tensor); for the outer step it is
// the tensor.  8 bytes, read with one scalar load.  In k
// kTileKept is set for a kept tile (a tensor has at most 2^28 pieces).
constexpr int32_t kTileKept = INT32_MIN;
struct TileRef {
  int32_t owner;
  int32_t k;
};
static_assert(sizeof(TileRef) == 8, "TileRef layout");

// How the kernels go through the caches: 8 L2s of 4 MB and one last-level cache of
// 256 MB in front of the memory.
struct CacheRule {
  bool streaming;      // non-temporal accesses (but for the kept tiles): local step, k_mix_step
  bool outer_streaming;  // the same for the outer step
  bool last_streaming;   // ... for the fused last step
  bool gossip_streaming;        // ... for the gossip step fused with the local step, de-biasing
  bool gossip_outer_streaming;  // ... for the outer step after such a gossip step
  bool write_through;  // stores leave the L2 at once
  double kept_bytes;   // of the replicas and buffers: kept in the last-level cache
};
// A step touches state_bytes of replicas and buffers and grad_bytes of gradients (grad_size
// bytes per element); x0 and u are outer_bytes, tau steps follow each other in an outer
// iteration.  idle_bytes of the state are buffers that no call of a round touches: under
// "reset" with tau = 1 all of them, but for the gossip step's.
struct Touched {
  int64_t state_bytes, grad_bytes, grad_size, outer_bytes, idle_bytes;
  int32_t tau;
  bool adam, averages;  // the base optimizer; the buffers are averaged
};
CacheRule cache_rule(const Touched &t);
// Direction of the next sweep over the tiles (1: backward) after one that went `backward`: the
// other one.  A paced walk goes forward in any case.
inline int32_t next_sweep(int32_t backward, bool paced) { return paced ? 1 : backward ^ 1; }

// Accesses of the last local step fused with the outer step without the average: streaming or plain on
// what a local step touches, on x0 and u, and whether all stores are written through, which follows the
// line of the local step.  4 workers, with against without, time of a round; tau = 1, x0 and u streaming:
// 44-52 MB that a local step touches 1.01-1.07, fp32 gradients 60-75 MB 0.94-1.00, bf16 60-75 MB
// 0.98-1.03; all streaming, from 78 MB on 0.92-1.02; tau = 3, all plain, 100-160 MB 0.96-0.99.
struct NoAvgAccess {
  bool local_nt, outer_nt, through;
};
inline NoAvgAccess noavg_access(bool local_nt, bool outer_nt, bool write_through) {
  return {local_nt, local_nt || outer_nt, write_through};
}
// Kept units: 16 384 elements of every worker.  Units are numbered along the tensors; the
// multiples of the golden ratio spread the kept ones evenly over any stretch of them, and
// so over the XCDs and the sets of the cache.
constexpr int32_t kKeptUnit = 16384;
inline bool unit_kept(int64_t unit, uint64_t share) {
  return static_cast<uint32_t>(unit) * 2654435769u < share;
}
// The share of the units, times 2^32, that is kept_bytes of state_bytes.
uint64_t kept_share(double kept_bytes, double state_bytes);
// Whether a launch over `tiles` tiles, some of them kept, reads those through plain accesses
// (in an instance of its own): the fused last step (its buffers are maintained), and the gossip
// step fused with the local step.
bool last_keeps(int64_t tiles, bool maintains);
bool mix_keeps(int64_t tiles, bool adam);
// The same for the outer step: m workers, touched_bytes as a local step touches them; the
// buffers are averaged along with the replicas.
bool outer_keeps(int32_t m, int64_t touched_bytes, bool averages);
// Where the local step keeps whole workers instead: how many of m are about kept_bytes,
// worker_bytes of replica and buffers each (0: not even the first one is).
int32_t kept_workers(int32_t m, double kept_bytes, double worker_bytes);

// Per (worker, tensor), fixed at create.
struct SlotInfo {
  float *x;        // device: the worker's replica of the tensor
  int64_t so;      // element offset of the tensor in the h / v arena (includes worker * d_pad)
  int64_t numel;   // elements in the tensor
  float wd;        // weight decay of this tensor
  float lr_scale;  // the tensor's fast learning rate is lr * lr_scale
};
static_assert(sizeof(SlotInfo) == 32, "SlotInfo layout");

// Per tensor, fixed at create (outer step).
struct TensorInfo {
  int64_t fo;         // element offset of the tensor in the x0 / u arena
  int64_t numel;
  int64_t unaligned;  // non-zero: some replica of this tensor is not 16-byte aligned
  float lr_scale;     // the tensor's fast learning rate is lr * lr_scale
  float wd;           // weight decay of this tensor
};
static_assert(sizeof(TensorInfo) == 32, "TensorInfo layout");

struct Layout {
  std::vector<int64_t> arena_off;  // per tensor, start in the per-worker arena (elements)
  int64_t d = 0;                   // total elements
  int64_t d_pad = 0;               // arena length per worker (elements, multiple of kArenaAlign)
};

struct PlanRun {  // host description of a tile (mirrors slowmo_plan_run)
  int32_t tile, worker, tensor, n;
  int64_t offset;
};

// Mixing step of gradient push (any in-neighbour map, column-stochastic weights).  The
// workers are listed in an order in which every worker comes before the worker
// it receives from, so that old values are still in memory when they are
// needed; the members of a cycle follow each other, each before its source,
// and the last one takes the first one's old value from a register.  Where an
// operand is the previous entry's source it is taken from a register too.
// kMixSaved more registers ("saved" operands) keep a sender whose later receivers or
// own turn come only after other senders have passed through the source
// register, so that it is not read (in the fused kernel: stepped) again.
constexpr int32_t kMixSaved = 4;
enum MixFlag : int32_t {
  kMixOwnFromS = 1,      // the worker's old value is the previous entry's source value
  kMixSrcFromS = 2,      // same source as the previous entry
  kMixSrcFromFirst = 4,  // the source is the worker that opened the cycle
  kMixSaveFirst = 8,     // this worker opens a cycle: keep its old value
  kMixNoSrc = 16,        // receives from nobody: x <- a * x
  kMixGroupStart = 32,   // first entry of a connected group of workers (for the launcher only)
};
// Three 3-bit fields above the flag bits, each 0 (no) or 1 + the number of a
// saved register:
//   save : before this entry's source replaces the held source value, the held
//          one is copied into that saved register;
//   own  : the worker's old value is in that saved register;
//   src  : the source value is in that saved register (and becomes the held
//          source value again).
constexpr int32_t kMixSaveShift = 6, kMixOwnSavedShift = 9, kMixSrcSavedShift = 12;
constexpr int32_t kMixFieldMask = 7;
// The source is stepped here for the last time: its own turn takes x from a
// register, so its buffers may be stored now.
constexpr int32_t kMixSrcDone = 1 << 15;
constexpr int32_t mix_save(int32_t flags) { return (flags >> kMixSaveShift) & kMixFieldMask; }
constexpr int32_t mix_own_saved(int32_t flags) { return (flags >> kMixOwnSavedShift) & kMixFieldMask; }
constexpr int32_t mix_src_saved(int32_t flags) { return (flags >> kMixSrcSavedShift) & kMixFieldMask; }
static_assert(kMixSaved <= kMixFieldMask, "register numbers must fit the fields");
struct MixEntry {
  int32_t node;    // worker updated by this entry
  int32_t src;     // worker it receives from (the worker itself with kMixNoSrc)
  float a;         // p(node, node) = 1 / (1 + outdeg(node))
  float b;         // p(node, src)  = 1 / (1 + outdeg(src))
  int32_t flags;   // MixFlag bits
  int32_t pad_;
};
static_assert(sizeof(MixEntry) == 24, "MixEntry layout");
// The update order of one mixing step for the in-neighbour map in_peer (m
// entries in 0..m-1); share[j] = 1 / (1 + outdeg(j)).  Workers that neither
// send nor receive get no entry unless with_idle is set (then: a = 1, kMixNoSrc).
// saved_limit: how many of the kMixSaved saved registers may be used.
void plan_mix(int32_t m, const int32_t *in_peer, std::vector<MixEntry> &seq,
              std::vector<float> &share, bool with_idle = false, int32_t saved_limit = kMixSaved);

Layout make_layout(int32_t n_tensors, const int64_t *numel);

// Number of tiles of each kind (no allocation).
int64_t count_local_tiles(int32_t m, int32_t n_tensors, const int64_t *numel);
int64_t count_outer_tiles(int32_t n_tensors, const int64_t *numel);
// Whole pieces of the smallest big tile over all tensors (an upper bound on the big tiles
// in use).
int64_t count_big_tiles(int32_t n_tensors, const int64_t *numel);
// Vectors per lane of the big tiles for a list (numel: its tensors, those that cannot take
// big tiles as 0) on a chip with `cus` CUs; 0: not enough of them.
int32_t choose_big_vpt(int32_t n_tensors, const int64_t *numel, int32_t cus);
// Which calls take the big tiles of a list that has some (policy: 0 reset, 1 maintain, 2
// average; asked: SLOWMO_BIG_TILES=1, wherever the kernels allow): the fused last step, and the
// outer step by itself.
bool last_takes_big(int policy, bool asked);
bool outer_takes_big(int32_t m, int policy, bool asked);
int64_t count_pieces(int32_t n_tensors, const int64_t *numel, int64_t piece);
// Whether a list of `pieces` paced tiles, of whose m workers a step reads `read_bytes`, is paced on a chip
// of `row` CUs.
bool paced_pays(int32_t m, int64_t pieces, int64_t row, int64_t read_bytes, bool aligned);
// Whole kPacedTile pieces of a list that paced walks may take: 0 when the list or the
// worker count is too small (with `forced`, only when no tensor has such a piece).
int64_t count_paced_pieces(int32_t m, int32_t n_tensors, const int64_t *numel, bool forced);
// `rest` left-over tiles ride with `paced` pieces in the same launch, on `row` CUs.
bool rest_rides(int64_t paced, int64_t rest, int64_t row);
// The pieces a paced walk takes (owner = tensor) on a chip with `row` CUs, and the
// ordinary tiles they leave over; both empty when it takes none.
void plan_paced(int32_t m, int32_t n_tensors, const int64_t *numel, int64_t row, bool forced,
                std::vector<TileRef> &paced, std::vector<TileRef> &rest);

// Tiles in launch order: worker-major, tensors in list order, offsets ascending.
void plan_local(int32_t m, int32_t n_tensors, const int64_t *numel, std::vector<PlanRun> &runs);
void plan_outer(int32_t n_tensors, const int64_t *numel, std::vector<PlanRun> &runs);

}  // namespace slowmo
