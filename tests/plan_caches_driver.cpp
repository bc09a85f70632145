// The rules that say how the kernels go through the caches, and which big tiles a list gets.
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "slowmo_plan.h"

using namespace slowmo;

static void check(bool ok, const char *what, double at) {
  if (ok) return;
  std::printf("FAILED: %s (%g)\n", what, at);
  std::exit(1);
}

int main() {
  const int64_t MiB = int64_t{1} << 20;
  for (int64_t size : {int64_t{1}, 32 * MiB, 32 * MiB + 3, 48 * MiB, 54 * MiB, 72 * MiB, 72 * MiB + 3, 240 * MiB,
                       240 * MiB + 3, int64_t{1} << 40}) {
    for (int64_t grad : {2, 4}) {
      for (int32_t tau : {1, 2, 48}) {
        for (int64_t idle : {int64_t{0}, size / 3}) {
          for (bool adam : {false, true}) {
            if (idle && tau > 1) continue;
            const int64_t g = size / (8 + grad) * grad, s = size - g, fits = (tau > 1 ? 240 : 72) * MiB;
            const CacheRule r = cache_rule({s, g, grad, size / 4, idle, tau, adam, false});
            const bool in = size > 32 * MiB && size <= fits, both = in && size + size / 4 <= fits;
            // x0 and u of many workers: small, and with one step per round no reason to stream
            const CacheRule many = cache_rule({s, g, grad, size / 10, 0, tau, adam, false});
            check(many.outer_streaming == !(in && (tau == 1 || size + size / 10 <= fits)), "a small part", size);
            const CacheRule avg = cache_rule({s, g, grad, size / 10, 0, tau, adam, true});
            check(avg.outer_streaming == !(in && size + size / 10 <= fits), "averaged buffers", size);
            check(avg.last_streaming == (avg.outer_streaming || (tau == 1 && !adam && size <= 48 * MiB)),
                  "averaged buffers", size);
            const bool l2 = idle && size - idle + size / 4 <= 30 * MiB;
            check(r.streaming == (!in || l2), "plain in the caches only", size);
            check(r.outer_streaming == (!both || l2), "the outer step plain where x0 and u fit too", size);
            check(r.outer_streaming || !r.streaming, "the outer step plain only where the local step is", size);
            check(r.gossip_streaming == !in && r.gossip_outer_streaming == !both, "after gossip", size);
            check(r.last_streaming == (!both || (idle && (!adam || size <= 48 * MiB))), "fused last step", size);
            check((r.kept_bytes > 0) == (r.streaming && r.write_through && tau > 1), "kept on long lists", size);
            check(r.kept_bytes <= 0.6 * s && r.kept_bytes <= 224e6, "no more kept than fits", size);
            check(r.write_through == (size > (grad == 2 ? 80 : 54) * MiB), "written through", size);
          }
        }
      }
    }
  }
  // the kept share of any stretch of units is near the share asked for
  for (double share : {0.0, 0.004, 0.1, 0.37, 0.6, 1.0}) {
    const uint64_t of = kept_share(share * 1e9, 1e9);
    for (int64_t from : {int64_t{0}, int64_t{7777}, int64_t{1} << 33}) {
      int64_t n = 0;
      for (int64_t u = from; u < from + 1000; ++u) n += unit_kept(u, of);
      check(std::abs(n - 1000 * share) <= 8, "kept units of a stretch", share);
    }
  }
  check(kept_share(0, 1e9) == 0 && kept_share(1e9, 0) == 0, "nothing kept", 0);
  check(unit_kept(123, kept_share(5e9, 1e9)), "everything kept", 0);
  check(kept_workers(8, 224e6, 94e6) == 2 && kept_workers(32, 224e6, 204e6) == 1, "whole workers", 0);
  check(kept_workers(8, 224e6, 306e6) == 1 && kept_workers(8, 224e6, 2.5e9) == 0, "large workers", 0);
  check(kept_workers(2, 1e12, 1e6) == 2 && kept_workers(4, 0, 1e6) == 0, "limits", 0);
  // instances for kept tiles: none on lists that are on their way at once, whatever the share
  for (bool other : {false, true}) {
    check(last_keeps(4095, other) == other && last_keeps(4096, other), "fused last step", other);
    check(!mix_keeps(2999, other) && mix_keeps(3000, other) == other && mix_keeps(4096, other), "gossip", other);
    check(last_keeps(int64_t{1} << 31, other) && mix_keeps(int64_t{1} << 31, other), "small shares", other);
  }
  for (int32_t m : {1, 2, 8, 15, 16, 32}) {
    check(outer_keeps(m, 250 * MiB, true) && outer_keeps(m, 20000 * MiB, true), "averaged buffers", m);
    check(outer_keeps(m, 500 * MiB, false) == (m == 1 || m >= 16) && outer_keeps(m, 701 * MiB, false),
          "plain outer step", m);
  }
  // calls that take big tiles: never with averaged buffers, however many workers there are
  for (bool asked : {false, true}) {
    for (int32_t m : {8, 15, 16, 32}) {
      check(!outer_takes_big(m, 2, asked) && !last_takes_big(2, asked), "averaged buffers", m);
      check(outer_takes_big(m, 0, asked) == (asked || m >= 16), "outer step", m);
      check(outer_takes_big(m, 1, asked) == (asked || m >= 16), "outer step", m);
    }
    check(last_takes_big(0, asked) && last_takes_big(1, asked) == asked, "fused last step", asked);
  }
  // sweeps: the other way than the one before, and backward after a paced walk
  for (int32_t was : {0, 1}) check(next_sweep(was, false) == 1 - was && next_sweep(was, true) == 1, "sweep", was);
  // the fused last step without the average: written through where the local step is, whatever the loads
  for (bool local : {false, true}) {
    for (bool outer : {false, true}) {
      for (bool through : {false, true}) {
        const NoAvgAccess by = noavg_access(local, outer, through);
        check(by.local_nt == local && by.outer_nt == (local || outer), "streaming", local + 2 * outer);
        check(by.through == through, "written through only where asked", local + 2 * outer);
      }
    }
  }
  // big tiles: none below 160, never more than the workspace has room for
  for (int64_t n = 0; n < 4000; n += 37) {
    const std::vector<int64_t> list = {n * 20000 + 11, 65536 * (n % 90), 5};
    const int32_t v = choose_big_vpt(3, list.data(), 256);
    check(v == 0 || v == 16 || v == 14 || v == 12, "size", n);
    if (v == 0) {
      check(count_pieces(3, list.data(), big_tile(kBigVptMin)) < kBigMinTiles, "enough of the smallest", n);
    } else {
      const int64_t tiles = count_pieces(3, list.data(), big_tile(v));
      check(tiles >= kBigMinTiles && tiles <= count_big_tiles(3, list.data()), "number of tiles", n);
    }
  }
  const int64_t full = 256 * int64_t{65536};
  check(choose_big_vpt(1, &full, 256) == 16, "one full round", 0);
  check(choose_big_vpt(1, &full, 0) == 0, "no CUs", 0);
  std::puts("ok");
  return 0;
}
