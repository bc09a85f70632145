#include "slowmo_plan.h"

#include <algorithm>
#include <utility>

namespace slowmo {

Layout make_layout(int32_t n_tensors, const int64_t *numel) {
  Layout L;
  L.arena_off.resize(n_tensors);
  int64_t off = 0;
  for (int32_t j = 0; j < n_tensors; ++j) {
    L.arena_off[j] = off;
    L.d += numel[j];
    off += (numel[j] + kArenaAlign - 1) / kArenaAlign * kArenaAlign;
  }
  L.d_pad = std::max<int64_t>(off, kArenaAlign);
  return L;
}

// The lines, from the time of one local step among others, over the time with streaming
// accesses everywhere and all sweeps in one direction; 1, 8 and 32 workers in 1 and 20 tensors each, SGD and Adam, fp32
// and bf16 gradients, 0.1 to 800 M elements.
CacheRule cache_rule(const Touched &t) {
  constexpr int64_t MiB = int64_t{1} << 20;
  const int64_t all = t.state_bytes + t.grad_bytes;
  CacheRule r{};
  // Plain accesses, gradients included, as long as all of it fits the last-level cache:
  // 30-60 MB 0.73-0.90, 60-250 MB 0.72-0.83, 256-266 MB 0.80-0.92.  Below, in the L2s,
  // streaming is as good or better (18 MB: plain 0.84-1.02, streaming 0.81-0.91), or plain
  // accesses gain only while nothing else runs (24 MB 0.76-1.07; three optimizers in turn,
  // rounds of 2 steps 0.84-1.41).  A round of one step finds nothing in the cache but what
  // the last round left there: three optimizers in turn, tau = 1, 40 MB 0.85-1.10, 70 MB
  // 0.82-1.01, 120 MB 0.96-1.13, 200 MB 0.97-1.17; tau = 2 0.79-1.00 from 40 MB on.
  const int64_t fits = (t.tau > 1 ? 240 : 72) * MiB;
  const bool plain = all > 32 * MiB && all <= fits;
  // The outer step and the fused last step, plain with x0 and u in the cache as well; time
  // of rounds of 4 steps over that with only the local step plain, 1, 4 and 16 workers: 24 MB
  // 0.82-1.09 (worst under "reset"), 40-230 MB with x0 and u 0.77-0.99; 255-290 MB
  // 0.95-1.10, 330-400 MB 1.00-1.09.  The gossip kernels, rounds by the line of the local
  // step: 24 MB 0.88-0.99, 40-120 MB 0.87-0.95, 200-245 MB 0.82-0.95.
  // With tau = 1 plain accesses in the local step alone cost where x0 and u are a small part (11
  // workers, 35-74 MB 1.05-1.24; 6 with de-biasing 1.00-1.10) and gain where they are a large one (1 to
  // 3 workers, 52-70 MB 0.84-0.99): a small part does not count, but where the outer step takes
  // the buffers as well (8 workers, 74 MB, plain over streaming outer step 1.05-1.15).
  const bool small_outer = t.tau == 1 && !t.averages && t.outer_bytes < all / 8;
  const bool with_outer = plain && (small_outer || all + t.outer_bytes <= fits);
  r.streaming = r.gossip_streaming = !plain;
  r.outer_streaming = r.last_streaming = r.gossip_outer_streaming = !with_outer;
  if (t.idle_bytes > 0) {
    // tau = 1 under "reset": calls share x, x0 and u only, and as long as what they touch at all
    // is in the L2s, plain accesses cost.  Local and outer step, plain over streaming, one optimizer
    // or three in turn, 11 workers, by what is touched: 18-31 MB 0.96-1.33, 32-33 MB 0.92-1.05,
    // 34-40 MB 0.90-1.06, 41 MB and more 0.83-0.93.  The fused step is the whole round: SGD, touching 28
    // to 47 MB, 0.89-1.10, worst with fp32 gradients from 35 MB on; Adam, 50-70 MB with the buffers,
    // 0.85-1.02.
    if (all - t.idle_bytes + t.outer_bytes <= 30 * MiB) r.streaming = r.outer_streaming = true;
    if (!t.adam || all <= 48 * MiB) r.last_streaming = true;
  }
  // SGD with averaged buffers, fused step, 8 workers, 43-50 MB 1.04-1.08 or, three in turn, 0.96-0.97.
  if (t.tau == 1 && t.averages && !t.adam && all <= 48 * MiB) r.last_streaming = true;
  // Written through: where the L2s cannot hold much of it for the next call anyway, the
  // memory takes stores better when they come at once.  With against without, plain
  // accesses: 30-50 MB 1.00-1.25; fp32 gradients 56-64 MB 0.96-1.02, 72-230 MB 0.92-0.98;
  // bf16 gradients 60-70 MB 1.04-1.06, 80-84 MB 0.99-1.03, 100-224 MB 0.96-0.99.
  // Streaming accesses on longer lists: 0.98-1.00.
  r.write_through = all > (t.grad_size == 2 ? 80 : 54) * MiB;
  // Longer lists keep a part of the replicas and buffers: a kept byte saves a read and a
  // write, a gradient's only a read.  224 MB of it, 0.6 of the state where that is less
  // (what is not kept comes from memory at the same time): 260-360 MB 0.79-0.88, 400-560
  // MB 0.80-0.90, 1 GB 0.85-0.89, 2 GB 0.90-0.92, 5 GB 0.95-0.97, 10 GB 0.98.  With 128 MB
  // 0.02 more at 1 to 2 GB; with all of the state up to 0.14 more at 300 MB.  Plain
  // accesses on such lists: 0.84-0.96 up to 500 MB, 1.03-1.10 from 2 GB on.  All of this
  // where steps follow each other; where something else has passed through the cache in
  // between, a call with kept tiles takes as long as one without.
  // With tau = 1 nothing is kept: three optimizers in turn 0.96-1.08 (tau = 2 0.89-0.98).
  if (r.streaming && r.write_through && t.tau > 1) {
    r.kept_bytes = std::min(224e6, 0.6 * static_cast<double>(t.state_bytes));
  }
  return r;
}

uint64_t kept_share(double kept_bytes, double state_bytes) {
  if (state_bytes <= 0 || kept_bytes <= 0) return 0;
  return static_cast<uint64_t>(std::min(kept_bytes / state_bytes, 1.0) * 4294967296.0);
}

// The instances for kept tiles have both walks in them and up to 46 registers more: 4 or 5 waves
// per SIMD, 4096 to 5120 on the chip.  Without them a shorter list is on its way at once, and a
// tile that is back early makes room for no other.  Rounds of 4 steps, 16 to 64 workers, kept
// tiles read as such over streamed (the local step keeps them in both).  Gossip step, SGD / Adam:
// 1500 tiles 1.32 / 1.25-1.30, 2500 1.14 / 1.01-1.08, 3000 1.05-1.10 / 0.97-1.01, 3500 0.99-1.04 /
// 0.91-0.98, 4500 0.92-0.95 / 0.86-0.95, 8000 0.88-0.95 / 0.87-0.97; in groups of 2 to 8 workers
// 2500 0.98-1.13 / 0.97-1.08, 3500 1.02-1.07 / 0.98-1.04, 4500 0.98-1.04 / 0.96-1.05, 6000
// 0.94-1.02 / 0.95-1.04 (above 1.02 with 64 workers only).  Fused last step: "maintain" 0.95-1.01 on
// 1500 to 4000 tiles, 0.95-0.98 beyond; "reset" 1.00-1.05, averaged buffers 1.01-1.07, from 4500 on
// 0.98-1.01 and 0.97-1.02.  A small share is no reason against them: at 5 and 12 GB, where 6 and 3
// % are kept, the fused last step takes 0.94-0.98 and 0.97-0.99 of its time, the gossip step
// 0.95-0.96 and 0.97-0.99: kept lines that are streamed over are not there for the next call.
bool last_keeps(int64_t tiles, bool maintains) { return maintains || tiles >= 4096; }
bool mix_keeps(int64_t tiles, bool adam) { return tiles >= (adam ? 3000 : 4096); }

// The plain outer step moves only the replicas, of which a third to a half of the kept part is, and
// has 56 registers instead of 40 then.  Its time with kept tiles over streamed, 2 to 8 workers:
// 270-500 MB 0.96-1.12, 600 MB 0.94-1.08, 800 MB 0.94-1.02, 1 GB 0.91-0.94, 5 GB 0.97; one worker
// 0.91-1.00 at all of them, 16 and 32 workers 0.97-1.03 at 270 MB, 0.87-0.97 beyond.  With averaged
// buffers 0.84-1.00 from 260 MB to 20 GB.
bool outer_keeps(int32_t m, int64_t touched_bytes, bool averages) {
  return averages || m == 1 || m >= 16 || touched_bytes > int64_t{700} << 20;
}

// To the nearest number that is not much more than the cache holds: 306 MB still are good
// (Adam, m = 8, 25.6 M elements: 866 -> 789 us, units of every worker 804).
int32_t kept_workers(int32_t m, double kept_bytes, double worker_bytes) {
  if (worker_bytes <= 0 || kept_bytes <= 0) return 0;
  return static_cast<int32_t>(std::min<double>(m, kept_bytes / worker_bytes + 0.3));
}

static int64_t tiles_of(int64_t n, int64_t tile) { return (n + tile - 1) / tile; }

int64_t count_local_tiles(int32_t m, int32_t n_tensors, const int64_t *numel) {
  int64_t per_worker = 0;
  for (int32_t j = 0; j < n_tensors; ++j) per_worker += tiles_of(numel[j], kLocalTile);
  return per_worker * m;
}

int64_t count_outer_tiles(int32_t n_tensors, const int64_t *numel) {
  int64_t t = 0;
  for (int32_t j = 0; j < n_tensors; ++j) t += tiles_of(numel[j], kOuterTile);
  return t;
}

int64_t count_pieces(int32_t n_tensors, const int64_t *numel, int64_t piece) {
  int64_t t = 0;
  for (int32_t j = 0; j < n_tensors; ++j) t += numel[j] / piece;
  return t;
}

int64_t count_big_tiles(int32_t n_tensors, const int64_t *numel) {
  return count_pieces(n_tensors, numel, big_tile(kBigVptMin));
}

// Big tiles pay in the fused last step when its buffers are dropped ("reset"); stores of every
// worker's buffers inside the walk cost them their gain (2-10 % slower than single-wave tiles
// under "maintain").  Averages of the buffers are in neither kernel: they do not fit the registers.
bool last_takes_big(int policy, bool asked) { return policy == 0 || (asked && policy == 1); }
bool outer_takes_big(int32_t m, int policy, bool asked) {
  return policy != 2 && (asked || m >= kBigOuterFromWorkers);
}

// A big tile keeps one CU busy, and all of them take about the same time, so a launch runs
// in rounds of one tile per CU.  A last round that fills a part f of the CUs is bound by what
// their loads can have in flight: it takes 0.46 of a whole one at f = 0.11-0.14, 0.59 at
// 0.33, 0.65 at 0.5, 0.70 at 0.6, 0.73 at 0.7, 0.81 at 0.8, 0.93 at 0.93 (m = 8), and up to
// 0.05 next to nothing, because the rounds are not that even.  Smaller tiles cost 1 % (14
// vectors) and 3-6 % (12) per element; 10 and 8 would cost 7-8 %.  Fused last step with 16, 14,
// 12 vectors: 25.6 M elements, m = 32 2205, 2145, 2163 us, m = 16 (first step) 930, 885, 889;
// 11.7 M, m = 8 287, 278, 276; 20.0 M, m = 16 1057, 982, 913; 16.8 M, m = 8 394, 504, 469; 76 M,
// m = 8 2608, 2646, 2750.
int32_t choose_big_vpt(int32_t n_tensors, const int64_t *numel, int32_t cus) {
  if (cus <= 0) return 0;
  int32_t best = 0;
  double best_cost = 0;
  for (const auto &[vpt, loss] : {std::pair{16, 1.0}, std::pair{14, 1.01}, std::pair{12, 1.06}}) {
    const int64_t n = count_pieces(n_tensors, numel, big_tile(vpt));
    if (n < kBigMinTiles) continue;
    const double f = static_cast<double>(n % cus) / cus;
    const double part = f <= 0.05 ? f : std::max(f, 0.42 + 0.46 * f);
    const double cost = loss * vpt * (static_cast<double>(n / cus) + part);
    if (best == 0 || cost < best_cost) best = vpt, best_cost = cost;
  }
  return best;
}

int64_t count_paced_pieces(int32_t m, int32_t n_tensors, const int64_t *numel, bool forced) {
  const int64_t n = count_pieces(n_tensors, numel, kPacedTile);
  return forced || (m >= kPacedFromWorkers && n >= kPacedMinTiles) ? n : 0;
}

// The paced kernel keeps nothing in the last-level cache, single waves keep 224 MB there, which
// tells on lists of a few GB.  Time paced over in single waves (4 steps on random maps and the
// outer step, m = 8, 12, 16, 24 and 32), by the bytes that a step reads.  SGD, fp32 gradients: 1.2 GB
// 1.02-1.10, 1.6 1.01-1.06, 1.9 1.01-1.03, 2.3 0.98-1.01, 2.6 0.95-1.00, 3.8 0.93-1.00; bf16: 1.3 GB
// 1.01-1.08, 1.9 0.97-1.03, 2.2 0.97-1.01, 3.2 0.94-1.00; Adam, fp32: 1.6 GB 1.02-1.04, 2.1
// 1.01-1.03, 2.6 0.99-1.01, 3.0 0.93-1.00, 5.1 0.92-0.99.  On tensors packed back to back single waves
// lose more: SGD, fp32 1.2 GB 1.02-1.04, 1.6 1.00-1.02, 1.9 0.98-1.00, 2.3 0.94-1.00, 3.8 0.89-0.99;
// bf16 1.3 GB 1.00-1.05, 1.6 1.00-1.01, 1.9 0.96-1.00; Adam 1.6 GB 1.00-1.03, 2.1 0.98-1.00, 5.1
// 0.89-0.98.  Aligned lists of less than two rows go by the workers instead: 300 to 511 pieces, both base
// optimizers and gradient types, maps mixed, cycles and random, m = 8 1.00-1.21, 12 1.03-1.16, 14
// 0.98-1.07, 16 0.98-1.10, 18 0.97-1.05, 20 0.97-1.04, 24 0.95-1.04, 32 0.91-1.01 (SGD, fp32, 511 pieces:
// m = 8 1066 us paced, 917 in single waves; m = 32 4180 and 4429).
bool paced_pays(int32_t m, int64_t pieces, int64_t row, int64_t read_bytes, bool aligned) {
  if (aligned && pieces < 2 * row) return m >= kPacedShortFromWorkers;
  return read_bytes >= (aligned ? kPacedFromBytes : kPacedPackedFromBytes);
}

// The CUs without a piece in the last row have its whole time for the left-over tiles, one
// per wave: a wave takes about 1.2 us per worker for one (nothing overlaps in it), a row
// about 14, and 8 waves work side by side.  A launch of their own has the whole chip instead, which
// tells from about 1500 tiles on.  Gossip step with the tiles riding over a launch of their own; m = 8,
// 16 and 32, SGD and Adam, groups of 4 to 32 workers, 2 and 4 rows; by tiles per wave: 1 of 32 CUs idle 3
// 0.95-0.99, 6 0.96-1.00, 9 1.02-1.07, 13 1.08-1.22; 2 idle 3 0.96-0.99, 6 0.97-1.01, 9 1.03-1.08; 6 idle
// 0.9 (345 tiles) 0.96-0.99, 3 (1209) 0.98-1.00, 6 (2419) 1.00-1.05, 9 (3456) 1.03-1.10; 12 idle 0.9
// (691) 0.95-0.99, 3 (2419) 0.99-1.01, 6 (4838) 0.99-1.04, 9 (6912) 1.01-1.06.
bool rest_rides(int64_t paced, int64_t rest, int64_t row) {
  if (row < 8 || paced <= 0) return false;
  const int64_t members = row / 8, busy = (paced + 7) / 8 % members;
  return busy > 0 && rest <= kRestMost && rest <= (members - busy) * 8 * 8 * kRestPerWave;
}

void plan_paced(int32_t m, int32_t n_tensors, const int64_t *numel, int64_t row, bool forced,
                std::vector<TileRef> &paced, std::vector<TileRef> &rest) {
  paced.clear();
  rest.clear();
  int64_t n = count_paced_pieces(m, n_tensors, numel, forced);
  if (n == 0 || row <= 0) return;
  constexpr int64_t per = kPacedTile / kOuterTile;
  const int64_t tiles = count_outer_tiles(n_tensors, numel);
  if (!forced) {
    // Full rows of one tile per CU, plus a last one that is at least 5/8 full: a row
    // takes the same time however full it is.  Measured on one tensor of one, two and
    // four full rows and a part of one (8, 16 and 32 workers; SGD with fp32, Adam with
    // bf16 gradients), time with the part in the paced kernel over time with it in
    // single waves, by the CUs it occupies: 48 of 256 1.05-1.21, 96 1.02-1.05, 128
    // 0.99-1.06, 144 0.96-1.00, 160 0.95-1.00, 176 0.94-0.99, 192-240 0.87-0.99.
    if (n % row < row * 5 / 8) n = n / row * row;
    // What is left over is a second launch with a tail of its own, which one row does
    // not always pay for.  Lists of one row, one cycle of 8 to 32 workers, time over
    // all in single waves: 0.86-0.99 with the rest up to 4/5 of the paced tiles,
    // 0.91-1.10 beyond (worst where the rest just opens another round of waves).  From
    // two rows on never more than 1.01.
    if (n < 2 * row && tiles - n * per > n * per * 4 / 5) return;
  }
  if (n == 0) return;
  paced.reserve(static_cast<size_t>(n));
  rest.reserve(static_cast<size_t>(tiles - n * per));
  for (int32_t j = 0; j < n_tensors; ++j) {
    const int64_t whole = std::min(numel[j] / kPacedTile, n - static_cast<int64_t>(paced.size()));
    for (int64_t k = 0; k < whole; ++k) paced.push_back({j, static_cast<int32_t>(k)});
    for (int64_t k = whole * per; k * kOuterTile < numel[j]; ++k)
      rest.push_back({j, static_cast<int32_t>(k)});
  }
}

static void cut(int32_t worker, int32_t n_tensors, const int64_t *numel, int64_t tile,
                std::vector<PlanRun> &runs) {
  for (int32_t j = 0; j < n_tensors; ++j) {
    for (int64_t off = 0; off < numel[j]; off += tile) {
      PlanRun r;
      r.tile = static_cast<int32_t>(runs.size());
      r.worker = worker;
      r.tensor = j;
      r.n = static_cast<int32_t>(std::min<int64_t>(tile, numel[j] - off));
      r.offset = off;
      runs.push_back(r);
    }
  }
}

void plan_local(int32_t m, int32_t n_tensors, const int64_t *numel, std::vector<PlanRun> &runs) {
  runs.clear();
  runs.reserve(static_cast<size_t>(count_local_tiles(m, n_tensors, numel)));
  for (int32_t w = 0; w < m; ++w) cut(w, n_tensors, numel, kLocalTile, runs);
}

void plan_outer(int32_t n_tensors, const int64_t *numel, std::vector<PlanRun> &runs) {
  runs.clear();
  runs.reserve(static_cast<size_t>(count_outer_tiles(n_tensors, numel)));
  cut(-1, n_tensors, numel, kOuterTile, runs);
}

// Mixing step for any map with at most one in-neighbour per worker.  A sender
// j splits its mass evenly over itself and its outdeg(j) receivers, so
// p(i,j) = 1 / (1 + outdeg(j)) and P is column-stochastic (Algorithm C.1).
// The replicas are mixed in place: a worker is overwritten only after every
// worker that receives from it has been served.  Seen as "i points to
// in_peer[i]", the map is a forest of trees hanging off cycles and fixed
// points.  Each tree is listed receivers-first (post-order), a sender's
// receivers that have receivers of their own before those that have none:
// then a worker is mostly followed by its source, whose old value the kernel
// already holds in a register, and receivers of one sender that follow each
// other share that register.  A cycle comes after the trees of its members,
// each member before its source.
void plan_mix(int32_t m, const int32_t *in_peer, std::vector<MixEntry> &seq,
              std::vector<float> &share, bool with_idle, int32_t saved_limit) {
  std::vector<int32_t> outdeg(m, 0);
  for (int32_t i = 0; i < m; ++i)
    if (in_peer[i] != i) ++outdeg[in_peer[i]];
  share.resize(m);
  for (int32_t j = 0; j < m; ++j) share[j] = 1.0f / static_cast<float>(1 + outdeg[j]);

  // which workers lie on a cycle: peel those nobody (left) receives from
  std::vector<int32_t> pending = outdeg, queue;
  std::vector<char> in_tree(m, 0);
  queue.reserve(m);
  for (int32_t i = 0; i < m; ++i)
    if (pending[i] == 0) queue.push_back(i);
  for (size_t q = 0; q < queue.size(); ++q) {
    const int32_t i = queue[q];
    in_tree[i] = 1;
    const int32_t j = in_peer[i];
    if (j != i && --pending[j] == 0) queue.push_back(j);
  }
  // receivers of every worker that are tree workers: first those that have
  // receivers themselves, then those that have none (CSR layout)
  std::vector<int32_t> start(m + 1, 0), recv(m);
  for (int32_t i = 0; i < m; ++i)
    if (in_peer[i] != i && in_tree[i]) ++start[in_peer[i] + 1];
  for (int32_t j = 0; j < m; ++j) start[j + 1] += start[j];
  {
    std::vector<int32_t> fill(start.begin(), start.end() - 1);
    for (int pass = 0; pass < 2; ++pass)
      for (int32_t i = 0; i < m; ++i)
        if (in_peer[i] != i && in_tree[i] && (outdeg[i] == 0) == (pass == 1))
          recv[fill[in_peer[i]]++] = i;
  }

  seq.clear();
  seq.reserve(m);
  auto emit = [&](int32_t i) {
    if (in_peer[i] != i) {
      seq.push_back({i, in_peer[i], share[i], share[in_peer[i]], 0, 0});
    } else if (outdeg[i] > 0 || with_idle) {
      seq.push_back({i, i, share[i], 0.f, kMixNoSrc, 0});
    }  // else: an idle worker keeps its value
  };
  // post-order walk of the tree below `root`; the root itself is listed only
  // if it is a tree worker (cycle members wait for their cycle)
  std::vector<std::pair<int32_t, int32_t>> stack;  // (worker, next receiver to visit)
  auto walk = [&](int32_t root) {
    stack.push_back({root, start[root]});
    while (!stack.empty()) {
      auto &top = stack.back();
      if (top.second < start[top.first + 1]) {
        const int32_t c = recv[top.second++];
        stack.push_back({c, start[c]});
      } else {
        if (in_tree[top.first]) emit(top.first);
        stack.pop_back();
      }
    }
  };
  // One group per connected set of workers: a fixed point with everything that
  // hangs off it, or a cycle with the trees of its members.  Groups share no
  // worker, so they may run as separate launches.
  std::vector<size_t> group_start;
  for (int32_t r = 0; r < m; ++r) {
    if (!(in_tree[r] && in_peer[r] == r)) continue;
    const size_t at = seq.size();
    walk(r);
    if (seq.size() > at) group_start.push_back(at);
  }
  std::vector<char> seen(m, 0);
  for (int32_t i = 0; i < m; ++i) {
    if (in_tree[i] || seen[i]) continue;
    group_start.push_back(seq.size());
    for (int32_t j = i; !seen[j]; j = in_peer[j]) {
      seen[j] = 1;
      walk(j);  // the trees of the cycle's members first
    }
    const size_t first = seq.size();
    for (int32_t j = i; seen[j] == 1; j = in_peer[j]) {
      seen[j] = 2;
      emit(j);
    }
    seq[first].flags |= kMixSaveFirst;
    seq.back().flags |= kMixSrcFromFirst;
  }
  for (size_t at : group_start) seq[at].flags |= kMixGroupStart;
  // Operands the kernel still holds when an entry needs them.  `held`: the
  // worker whose old value is in the source register (the previous entry's
  // source).  saved[k]: the worker whose old value was copied into saved
  // register k when another source took its place in the source register,
  // because it is needed again (by a later receiver, or at its own turn, which
  // is always its last use); the register is free again after that turn.
  std::vector<int32_t> last_use(m, -1);
  for (size_t idx = 0; idx < seq.size(); ++idx) {
    if (!(seq[idx].flags & kMixNoSrc)) last_use[seq[idx].src] = static_cast<int32_t>(idx);
    last_use[seq[idx].node] = static_cast<int32_t>(idx);
  }
  int32_t held = -1, saved[kMixSaved];
  for (int32_t &w : saved) w = -1;
  auto saved_in = [&](int32_t w) {
    for (int k = 0; k < kMixSaved; ++k)
      if (w >= 0 && saved[k] == w) return k;
    return -1;
  };
  std::vector<int32_t> stepped_at(m, -1);  // entry that read the worker as a source last
  for (size_t idx = 0; idx < seq.size(); ++idx) {
    MixEntry &e = seq[idx];
    if (e.flags & kMixGroupStart) {
      held = -1;
      for (int32_t &w : saved) w = -1;
    }
    const int own_saved = saved_in(e.node);
    if (e.node == held) {
      e.flags |= kMixOwnFromS;
    } else if (own_saved >= 0) {
      e.flags |= (own_saved + 1) << kMixOwnSavedShift;
    }
    if (own_saved >= 0) saved[own_saved] = -1;  // the worker's own turn is its last use
    if ((e.node == held || own_saved >= 0) && stepped_at[e.node] >= 0)
      seq[stepped_at[e.node]].flags |= kMixSrcDone;
    if (e.flags & kMixNoSrc) continue;
    const bool from_first = (e.flags & kMixSrcFromFirst) != 0;
    if (!from_first && e.src == held) {
      e.flags |= kMixSrcFromS;
      continue;
    }
    // the source register gets a new value: keep the old one if it is needed again
    if (held >= 0 && last_use[held] > static_cast<int32_t>(idx) && saved_in(held) < 0) {
      for (int k = 0; k < saved_limit; ++k) {
        if (saved[k] < 0) {
          saved[k] = held;
          e.flags |= (k + 1) << kMixSaveShift;
          break;
        }
      }
    }
    const int src_saved = from_first ? -1 : saved_in(e.src);
    if (src_saved >= 0) e.flags |= (src_saved + 1) << kMixSrcSavedShift;
    if (src_saved < 0 && !from_first) stepped_at[e.src] = static_cast<int32_t>(idx);
    held = e.src;
  }
}

}  // namespace slowmo
