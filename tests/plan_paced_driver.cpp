// Replays mixing orders planned for the paced gossip kernel (two saved values; a
// worker's buffers stored where kMixSrcDone says so, or at its own turn) in place,
// the way the kernel does, against the simultaneous update; and checks which pieces of a
// list plan_paced hands to it.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "slowmo_plan.h"

using namespace slowmo;

static void check(bool ok, const char *what, int m) {
  if (ok) return;
  std::printf("FAILED: %s (m = %d)\n", what, m);
  std::exit(1);
}

struct Stepped {
  double x, h;
};

static int replay(int m, const std::vector<int32_t> &peer, int32_t limit) {
  std::vector<MixEntry> seq;
  std::vector<float> share;
  plan_mix(m, peer.data(), seq, share, /*with_idle=*/true, limit);
  check(static_cast<int>(seq.size()) == m, "every worker has one entry", m);
  std::vector<double> x0(m), h0(m), x(m), h(m);
  std::vector<int> stores(m, 0);
  for (int i = 0; i < m; ++i) x[i] = x0[i] = 1.0 + i * i, h[i] = h0[i] = 0.5 * i;
  auto stepped = [&](int w) { return Stepped{x0[w] + 3.0 * h0[w] + 7.0, h0[w] + 1.0}; };
  int reads = 0;
  auto from_memory = [&](int w) {
    check(x[w] == x0[w] && h[w] == h0[w], "a worker is stepped from its old values", m);
    ++reads;
    return stepped(w);
  };
  auto store_buffers = [&](int w, double v) { h[w] = v, ++stores[w]; };
  double S = 0, first = 0, saved[kMixSaved + 1] = {};
  for (const MixEntry &e : seq) {
    double own;
    if (e.flags & kMixOwnFromS) {
      own = S;
    } else if (mix_own_saved(e.flags)) {
      own = saved[mix_own_saved(e.flags)];
    } else {
      const Stepped s = from_memory(e.node);
      store_buffers(e.node, s.h);
      own = s.x;
    }
    check(mix_save(e.flags) <= limit && mix_own_saved(e.flags) <= limit &&
              mix_src_saved(e.flags) <= limit, "the saved values stay within the limit", m);
    if (e.flags & kMixSaveFirst) first = own;
    double mixed = e.a * own;
    if (!(e.flags & kMixNoSrc)) {
      if (mix_save(e.flags)) saved[mix_save(e.flags)] = S;
      if (e.flags & kMixSrcFromFirst) {
        S = first;
      } else if (mix_src_saved(e.flags)) {
        S = saved[mix_src_saved(e.flags)];
      } else if (!(e.flags & kMixSrcFromS)) {
        const Stepped s = from_memory(e.src);
        if (e.flags & kMixSrcDone) store_buffers(e.src, s.h);
        S = s.x;
      }
      mixed += e.b * S;
    }
    x[e.node] = mixed;
  }
  std::vector<int> out(m, 0);
  for (int i = 0; i < m; ++i)
    if (peer[i] != i) ++out[peer[i]];
  for (int i = 0; i < m; ++i) {
    double want = (1.0f / static_cast<float>(1 + out[i])) * stepped(i).x;
    if (peer[i] != i) want += (1.0f / static_cast<float>(1 + out[peer[i]])) * stepped(peer[i]).x;
    check(x[i] == want, "the replica is the simultaneous update's", m);
    check(h[i] == h0[i] + 1.0 && stores[i] == 1, "the buffers are stepped and stored once", m);
  }
  return reads;
}

// The pieces that plan_paced gives the paced kernel; whole pieces in list order, and
// together with the rest every ordinary tile once.
static int64_t paced(int32_t m, const std::vector<int64_t> &numel, int64_t row, bool forced) {
  const int32_t nt = static_cast<int32_t>(numel.size());
  constexpr int64_t per = kPacedTile / kOuterTile;
  std::vector<TileRef> p, r;
  plan_paced(m, nt, numel.data(), row, forced, p, r);
  if (p.empty()) {
    check(r.empty(), "no paced tiles, no rest", m);
    return 0;
  }
  std::vector<int64_t> tile(nt, 0);
  size_t ip = 0, ir = 0;
  for (int32_t j = 0; j < nt; ++j) {
    for (; ip < p.size() && p[ip].owner == j; ++ip, tile[j] += per)
      check(p[ip].k * per == tile[j] && (p[ip].k + 1) * int64_t{kPacedTile} <= numel[j],
            "paced tiles are whole pieces in order", m);
    for (; ir < r.size() && r[ir].owner == j; ++ir, ++tile[j])
      check(r[ir].k == tile[j], "the rest follows them in order", m);
    check(tile[j] == (numel[j] + kOuterTile - 1) / kOuterTile, "every tile is in one list", m);
  }
  check(ip == p.size() && ir == r.size(), "no tile of another tensor", m);
  check(static_cast<int64_t>(p.size()) <= count_paced_pieces(m, nt, numel.data(), forced) &&
            static_cast<int64_t>(r.size()) <= count_outer_tiles(nt, numel.data()),
        "both lists fit the room that is kept for them", m);
  return static_cast<int64_t>(p.size());
}

static void paced_rule() {
  const int64_t T = kPacedTile, row = 256;
  check(paced(7, {400 * T}, row, false) == 0 && paced(8, {299 * T}, row, false) == 0 &&
            paced(8, {400 * T}, 0, false) == 0, "too few workers, pieces, CUs", 0);
  check(paced(8, {300 * T}, row, false) == 256, "short part of a row: single waves", 0);
  check(paced(8, {(256 + 159) * T + 5}, row, false) == 256 && paced(8, {(256 + 160) * T}, row, false) == 416 &&
            paced(8, {(512 + 159) * T}, row, false) == 512 && paced(8, {(512 + 160) * T}, row, false) == 672,
        "a part of a row from 5/8 on", 0);
  // whole pieces of several tensors, cut inside one of them
  check(paced(9, {100 * T + 1, 7, 150 * T, 0, 100 * T + 16383}, row, false) == 256, "cut inside a tensor", 0);
  // the rest against the pieces of a single row: 44 pieces and the short tensors
  const int64_t limit = 256 * 64 * 4 / 5 - 44 * 64;
  for (int64_t more : {0, 1}) {
    std::vector<int64_t> numel(static_cast<size_t>(limit + more), kOuterTile);
    numel.push_back(300 * T);
    check(paced(8, numel, row, false) == (more ? 0 : 256), "one row and a rest of 4/5", 0);
    numel.back() = 600 * T;
    check(paced(8, numel, row, false) == 512, "two rows", 0);
  }
  check(paced(1, {T - 1, T, 7, T + 5, 2 * T + 4099}, row, true) == 4 && paced(1, {T - 1, 3}, row, true) == 0,
        "forced: all whole pieces", 0);
}

// Whether a list is paced: by the bytes that a step reads, short aligned lists by the workers.
static void paying_rule() {
  const int64_t row = 256, none = 0, lots = int64_t{1} << 40;
  for (int32_t m : {8, 16, 17, 32}) {
    for (int64_t bytes : {none, lots}) {
      check(paced_pays(m, 300, row, bytes, true) == (m > 16) && paced_pays(m, 511, row, bytes, true) == (m > 16),
            "less than two rows, aligned", m);
      check(paced_pays(m, 512, row, bytes, true) == (bytes == lots), "two rows", m);
      check(paced_pays(m, 300, row, bytes, false) == (bytes == lots), "packed back to back", m);
    }
    check(!paced_pays(m, 512, row, kPacedFromBytes - 1, true) && paced_pays(m, 512, row, kPacedFromBytes, true),
          "the line of aligned lists", m);
    check(!paced_pays(m, 300, row, kPacedPackedFromBytes - 1, false) &&
              paced_pays(m, 300, row, kPacedPackedFromBytes, false), "the line of packed lists", m);
  }
}

// Left-over tiles that ride: up to 6 per wave of the CUs without a piece in the last row, and 1200.
static void riding_rule() {
  check(!rest_rides(512, 1, 256) && !rest_rides(505, 1, 256), "a full row: no CU to spare", 0);
  check(rest_rides(504, 384, 256) && !rest_rides(504, 385, 256), "one CU of each XCD", 0);
  check(rest_rides(256 + 240, 768, 256) && !rest_rides(256 + 240, 769, 256), "two CUs of each XCD", 0);
  check(rest_rides(256 + 160, 1200, 256) && !rest_rides(256 + 160, 1201, 256), "many CUs", 0);
  check(rest_rides(497, 384, 256) && !rest_rides(497, 385, 256), "by the XCD with the most pieces", 0);
  check(!rest_rides(0, 10, 256) && !rest_rides(400, 10, 0) && !rest_rides(400, 10, 7), "no pieces, few CUs", 0);
}

int main() {
  paced_rule();
  paying_rule();
  riding_rule();
  std::mt19937 rng(7);
  int reads = 0, workers = 0;
  for (int m = 1; m <= 40; ++m) {
    for (int32_t limit : {0, 1, kPacedSaved, kMixSaved}) {
      for (int hop = 0; hop < m; ++hop) {
        std::vector<int32_t> p(m);
        for (int i = 0; i < m; ++i) p[i] = (i + m - hop) % m;
        check(replay(m, p, limit) == m, "a permutation steps every worker once", m);
      }
      for (int t = 0; t < 200; ++t) {
        std::vector<int32_t> p(m);
        for (int i = 0; i < m; ++i) p[i] = static_cast<int32_t>(rng() % m);
        const int r = replay(m, p, limit);
        if (limit == kPacedSaved && m == 32) reads += r, workers += m;
      }
    }
  }
  check(reads <= 1.06 * workers, "two saved values keep the repeated steps rare", 32);
  std::printf("ok\n");
  return 0;
}
