// Pass::pair_at on the CPU: 64 lanes, their permute, and a choice of which lane is heard where several name the same one.
// Prints "ok" if every sign of every unit finds its (operator, record) pair, whichever lane is heard.
#include <algorithm>
#include <cstdio>
#include <random>
#include <vector>

#include "fbx_lists.h"

// The rooms of lists of layer 1 and of later layers: apart from each other, from the staged text while that is read, and all of
// the text's section for later layers where no text is staged.
static bool rooms() {
  for (uint32_t all : {0u, 10u, 400u})
    for (uint32_t text = 0; text <= all; ++text)
      for (uint32_t cap : {0u, 5u, 100u, 1000u}) {
        const fbx::ListRoom r = fbx::list_room(true, all, text, cap);
        if (r.behind ? r.first != all - text || r.first <= cap || r.later != text : r.first != cap || r.later != all) return false;
        const fbx::ListRoom p = fbx::list_room(false, all, 0, cap);
        if (p.behind || p.first != cap || p.later != all) return false;
      }
  return true;
}

int main() {
  if (!rooms()) { std::printf("rooms\n"); return 1; }
  std::mt19937 rng(7);
  for (int round = 0; round < 3000; ++round) {
    const uint32_t pairs = 1 + rng() % 400, mostly = rng() % 4;
    std::vector<uint32_t> start(pairs + 1, 0);
    std::vector<uint32_t> owner;
    for (uint32_t p = 0; p < pairs; ++p) {
      const uint32_t n = mostly == 0 ? rng() % 4 : mostly == 1 ? (rng() % 40 == 0) : mostly == 2 ? 1 : (rng() % 90 == 0 ? rng() % 300 : 0);
      start[p + 1] = start[p] + n;
      owner.insert(owner.end(), n, p);
    }
    for (uint32_t q0 = 0; q0 < owner.size(); q0 += 64) {
      // (the first pair looked at: any that starts at or before the unit)
      uint32_t lo = owner[q0];
      lo -= std::min<uint32_t>(lo, rng() % 100);
      for (int heard = 0; heard < 3; ++heard) {  // the lowest lane, the highest, any
        uint32_t pair[64] = {0};
        for (uint32_t w = lo;; w += 64) {
          uint32_t s[65], in = 0;
          for (uint32_t l = 0; l < 64; ++l) {
            uint32_t from = ~0u;
            if (w + l < pairs) from = start[w + l] > q0 ? start[w + l] - q0 : 0u;
            in += from < 64;
            s[l] = std::min(from, 63u);
          }
          s[64] = 63;
          std::vector<std::vector<uint32_t>> got(64);
          for (uint32_t l = 0; l < 64; ++l) {
            const fbx::PairSend to = fbx::pair_send(s[l], s[l + 1], w + l + 1, w + in);
            if (to.lane > 63) return 1;
            got[to.lane].push_back(to.number);
          }
          for (uint32_t l = 0; l < 64; ++l)
            if (!got[l].empty())
              pair[l] = std::max(pair[l], heard == 0 ? got[l].front() : heard == 1 ? got[l].back() : got[l][rng() % got[l].size()]);
          if (in < 64) break;
        }
        for (uint32_t l = 0, best = 0; l < 64 && q0 + l < owner.size(); ++l) {
          best = std::max(best, pair[l]);
          if (best != owner[q0 + l] + 1) { std::printf("round %d unit %u lane %u heard %d: %u, not %u\n", round, q0, l, heard, best, owner[q0 + l] + 1); return 1; }
        }
      }
    }
  }
  std::printf("ok\n");
  return 0;
}
