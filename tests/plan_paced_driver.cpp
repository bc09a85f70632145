// Replays mixing orders planned for the paced gossip kernel (two saved values; a
// worker's buffers stored where kMixSrcDone says so, or at its own turn) in place,
// the way the kernel does, against the simultaneous update.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "../paper_1910_00643_amd/csrc/slowmo_plan.h"

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

int main() {
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
