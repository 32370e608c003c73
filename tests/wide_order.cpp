// Walks walk_tiles (csrc/tva_wide_order.h) with steps that keep a wave's queue of transfers, and checks for every piece of up
// to `kMostTiles` tiles that what a step reads has landed for every wave of the workgroup before the barrier in front of it, that a
// place of the ring is filled again only when everybody is done with it, and that all waves meet as often.
#include <cstdio>
#include <map>
#include <vector>

#include "tva_wide_order.h"

namespace {
constexpr int kMostTiles = 100, kMostMasked = 6;  // (at most one ragged tile and four of the tree; one more)

struct Wave {
  std::vector<int> queue;                 // tiles in the order asked for; -1: a spare one
  size_t landed = 0;                      // of the queue's front
  std::vector<size_t> landed_at;          // by barrier
  std::vector<std::pair<int, int>> asked, read;  // (tile, barriers so far)
  int wrong = 0;                          // waits for fewer than none
  int meets() const { return (int)landed_at.size(); }
};

template <int AHEAD>
Wave walk(int n, int n_full, bool only_moves) {
  Wave w;
  auto ask = [&](int i) { w.queue.push_back(i); w.asked.push_back({i, w.meets()}); };
  auto spare = [&]() { w.queue.push_back(-1); };
  auto wait = [&](int left, auto most) {
    if (left < 0) ++w.wrong;
    const size_t may = (size_t)(left < decltype(most)::value ? left : decltype(most)::value);
    if (w.queue.size() > may && w.queue.size() - may > w.landed) w.landed = w.queue.size() - may;
  };
  auto meet = [&]() { w.landed_at.push_back(w.landed); };
  auto reads = [&](int tile) { if (tile < n) w.read.push_back({tile, w.meets()}); };
  auto first = [&]() { reads(0); };
  auto step = [&](int i) { reads(i + 1); reads(i); };
  auto run = [&](int) {};
  auto run_step = [&](int i, int u) {
    step(i + u);
    if (i + u + AHEAD < n_full) ask(i + u + AHEAD);
    else spare();
  };
  for (int i = 0; i < n && i < AHEAD; ++i) ask(i);
  jk::tva::walk_tiles<AHEAD>(n, n_full, only_moves, ask, spare, wait, meet, first, step, run, run_step);
  return w;
}

template <int AHEAD>
int check() {
  int bad = 0, pieces = 0;
  for (int n_full = 0; n_full <= kMostTiles; ++n_full)
    for (int masked = 0; masked <= kMostMasked; ++masked) {
      const int n = n_full + masked;
      if (n == 0) continue;
      ++pieces;
      const Wave works = walk<AHEAD>(n, n_full, false), moves = walk<AHEAD>(n, n_full, true);
      const char* what = nullptr;
      int which = 0;
      if (works.wrong || moves.wrong) what = "a wait for fewer than no tiles";
      if (works.meets() != moves.meets()) what = "barriers";
      std::map<int, int> last_read;  // tile: barriers in front of its last read
      for (const auto& r : works.read) last_read[r.first] = r.second;
      for (const Wave* w : {&works, &moves}) {
        std::map<int, int> place;  // tile: where in the queue
        for (size_t k = 0; k < w->queue.size(); ++k)
          if (w->queue[k] >= 0 && !place.emplace(w->queue[k], (int)k).second) what = "asked for twice", which = w->queue[k];
        for (const auto& r : works.read)
          if (!what && (!place.count(r.first) || (int)w->landed_at[r.second - 1] <= place[r.first])) what = "read before it was waited for", which = r.first;
        for (const auto& a : w->asked)
          if (!what && a.first > AHEAD && last_read[a.first - AHEAD - 1] >= a.second) what = "asked for into a place in use", which = a.first;
        if (!what && (int)place.size() != n) what = "tiles not asked for";
      }
      for (int i = 0; i < n; ++i)
        if (!what && !last_read.count(i)) what = "not read", which = i;
      if (what) {
        ++bad;
        std::printf("ahead %d, %d tiles without masks, %d with: %s (tile %d)\n", AHEAD, n_full, masked, what, which);
      }
    }
  std::printf("ahead %d: %d pieces, %d wrong\n", AHEAD, pieces, bad);
  return bad;
}
}  // namespace

int main() { return check<jk::tva::wide_ahead(128)>() + check<jk::tva::wide_ahead(64)>() == 0 ? 0 : 1; }
