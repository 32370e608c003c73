// Walks the two loops of csrc/tva_wide_order.h with steps that check them.
// "tiles": walk_tiles with a wave's queue of transfers.  For every piece of up to `kMostTiles` tiles: what a step reads has
// landed for every wave of the workgroup before the barrier in front of it, a place of the ring is filled again only when
// everybody is done with it, and all waves meet as often.
// "pieces": merge_pieces with a thread per workgroup, one of which runs at a time, another at every access to memory, chosen
// by a seed.  However long each is held up, and however soon the second of two stops waiting: one has all pieces in the
// end, once each, made of results that were whole when they were read; the words are zero again.
#include <condition_variable>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <random>
#include <set>
#include <thread>
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

// One thread at a time: a thread that is about to touch memory hands the turn to one that the seed chooses, now and then
// always the same one for a while (the others are held up)
class Turns {
 public:
  Turns(int n, unsigned seed) : rng_(seed), alive_(n) {
    for (int i = 0; i < n; ++i) alive_[i] = i;
    turn_ = pick();
  }
  void wait(int me) {
    std::unique_lock<std::mutex> l(m_);
    cv_.wait(l, [&] { return turn_ == me; });
  }
  void pass(int me) {
    {
      std::lock_guard<std::mutex> l(m_);
      turn_ = pick();
      if (turn_ == me) return;
    }
    cv_.notify_all();
    wait(me);
  }
  void end(int me) {
    std::lock_guard<std::mutex> l(m_);
    for (size_t k = 0; k < alive_.size(); ++k)
      if (alive_[k] == me) alive_.erase(alive_.begin() + k);
    turn_ = alive_.empty() ? -1 : pick();
    cv_.notify_all();
  }

 private:
  int pick() {
    if (rng_() % 8 == 0) favourite_ = (int)(rng_() % 64);
    const int n = (int)alive_.size();
    return alive_[favourite_ >= 0 && rng_() % 4 ? favourite_ % n : (int)(rng_() % n)];
  }
  std::mt19937 rng_;
  std::vector<int> alive_;
  int turn_ = -1, favourite_ = -1;
  std::mutex m_;
  std::condition_variable cv_;
};

struct Slot {
  std::multiset<int> results;
  bool whole = true;
};

int merge(int pieces, unsigned limit, unsigned seed, int* took_over) {
  std::vector<unsigned> word(pieces, 0u);
  std::vector<Slot> slot(pieces);
  std::vector<std::multiset<int>> has_all;
  int bad = 0;
  Turns turns(pieces, seed);
  std::vector<std::thread> threads;
  for (int me = 0; me < pieces; ++me)
    threads.emplace_back([&, me] {
      turns.wait(me);
      std::multiset<int> mine{me};
      bool first = false;
      auto arrive = [&](int m) {
        turns.pass(me);
        first = word[m]++ == 0u;
        for (unsigned polls = 0; !first && polls <= limit; ++polls) {
          turns.pass(me);
          const int at = jk::tva::others_results(word[m], false);
          if (at >= 0) return at;
        }
        return -1;
      };
      auto leave = [&](int m) {
        slot[me].whole = false;
        turns.pass(me);
        slot[me].results = mine;
        slot[me].whole = true;
        turns.pass(me);
        const unsigned w = word[m];
        word[m] |= jk::tva::left_results(first, me);
        const int at = jk::tva::others_results(w, first);
        if (first && at >= 0) ++*took_over;
        return at;
      };
      auto add = [&](int m, int at) {
        word[m] = 0u;
        for (int half = 0; half < 2; ++half) {
          turns.pass(me);
          if (!slot[at].whole) ++bad;
        }
        mine.insert(slot[at].results.begin(), slot[at].results.end());
      };
      if (jk::tva::merge_pieces(me, pieces, arrive, leave, add)) has_all.push_back(mine);
      turns.end(me);
    });
  for (auto& t : threads) t.join();
  std::multiset<int> all;
  for (int i = 0; i < pieces; ++i) all.insert(i);
  if (has_all.size() != 1 || has_all[0] != all) ++bad;
  for (unsigned w : word) bad += w != 0u;
  if (bad) std::printf("%d pieces, %u polls, seed %u: wrong\n", pieces, limit, seed);
  return bad;
}

int check_pieces() {
  int bad = 0, took_over = 0;
  for (int pieces = 1; pieces <= 9; ++pieces)
    for (unsigned limit : {0u, 1u, 3u, 1000u})
      for (unsigned seed = 0; seed < 150; ++seed) bad += merge(pieces, limit, seed, &took_over);
  for (int a : {0, 1, jk::tva::kMeetingPieces - 1})
    for (int b : {0, 1, jk::tva::kMeetingPieces - 1}) {
      const unsigned w = 2u | jk::tva::left_results(true, a) | jk::tva::left_results(false, b);
      bad += jk::tva::others_results(w, false) != a || jk::tva::others_results(w, true) != b;
    }
  std::printf("merges: %d wrong; %d times the first to come went on\n", bad, took_over);
  return bad + (took_over == 0);
}
}  // namespace

int main(int argc, char** argv) {
  if (argc > 1 && std::strcmp(argv[1], "pieces") == 0) return check_pieces() == 0 ? 0 : 1;
  return check<jk::tva::wide_ahead(128)>() + check<jk::tva::wide_ahead(64)>() == 0 ? 0 : 1;
}
