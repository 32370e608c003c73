// The protocols by which the workgroups of a call meet, over one header, in turn: the merge of tva_bf16.hip (a group word whose call
// number stays), the pairs of tva_wide.hip (tva_wide_order.h), the counted parts of tva_f32.hip and the counters of the greedy
// launch, with the words of csrc/jk_words.h.  A thread per workgroup, one of which runs at a time, another at every access to
// memory, chosen by a seed; waits that expire at once, soon, or practically never.  Of every call: whoever merges finds all
// results of this call in memory, and everything is merged; behind it the words that are counted in from zero are zero.
#include <condition_variable>
#include <cstdio>
#include <functional>
#include <mutex>
#include <random>
#include <set>
#include <thread>
#include <vector>

#include "jk_words.h"
#include "tva_wide_order.h"

namespace {
using namespace jk;

std::vector<unsigned> header(kMaxFusedGroups * kLineWords, 0u);
int bad = 0, gave_up = 0, left_over = 0;

// Runs the workgroups, one at a time; each passes the turn in front of an access to memory
class Turns {
 public:
  Turns(std::mt19937& rng, const std::vector<std::function<void(Turns&, int)>>& work) : rng_(rng) {
    for (int i = 0; i < (int)work.size(); ++i) alive_.push_back(i);
    turn_ = pick();
    std::vector<std::thread> threads;
    for (int i = 0; i < (int)work.size(); ++i)
      threads.emplace_back([&, i] {
        wait(i);
        work[i](*this, i);
        std::lock_guard<std::mutex> l(m_);
        for (size_t k = 0; k < alive_.size(); ++k)
          if (alive_[k] == i) alive_.erase(alive_.begin() + k);
        turn_ = alive_.empty() ? -1 : pick();
        cv_.notify_all();
      });
    for (auto& t : threads) t.join();
  }
  void pass(int me) {
    {
      std::lock_guard<std::mutex> l(m_);
      turn_ = pick();
      if (turn_ == me) return;
      cv_.notify_all();
    }
    wait(me);
  }

 private:
  void wait(int me) {
    std::unique_lock<std::mutex> l(m_);
    cv_.wait(l, [&] { return turn_ == me; });
  }
  int pick() {  // (now and then the same one for a while: the others are held up)
    if (rng_() % 8 == 0) favourite_ = (int)(rng_() % 64);
    const int n = (int)alive_.size();
    return alive_[favourite_ >= 0 && rng_() % 4 ? favourite_ % n : (int)(rng_() % n)];
  }
  std::mt19937& rng_;
  std::vector<int> alive_;
  int turn_ = -1, favourite_ = -1;
  std::mutex m_;
  std::condition_variable cv_;
};
typedef std::vector<std::function<void(Turns&, int)>> Work;

void expect(bool ok, const char* what) {
  if (!ok) {
    ++bad;
    std::printf("%s\n", what);
  }
}

// tva_bf16.hip: a group's workgroups each merge a slice once all partials are there
void grouped(std::mt19937& rng, int group, int splits, unsigned limit) {
  std::vector<bool> stored(splits, false);
  std::vector<int> merged(splits, 0);
  unsigned* word = &header[group_word(group)];
  auto merge = [&](int slice) {
    if (slice >= splits) return;  // (a mark left by a call of more splits: no rows)
    for (int s = 0; s < splits; ++s) expect(stored[s], "grouped: merged before all results were there");
    ++merged[slice];
  };
  Work work(splits, [&](Turns& t, int me) {
    t.pass(me);
    stored[me] = true;
    t.pass(me);
    const unsigned S = (unsigned)splits, old = *word;
    *word += 1u;
    const unsigned epoch = old >> 16;
    int mode = 1;
    unsigned lo = 0u, hi = 0u;
    if ((old & kSyncCountMask) == S - 1) {
      const unsigned gone = (old >> 8) & 0xffu;
      t.pass(me);
      *word += kSyncEpochOne - S - gone * kSyncGaveUpOne;
      if (gone) {
        mode = 2;
        t.pass(me);
        lo = word[1]; word[1] = 0u;
        t.pass(me);
        hi = word[2]; word[2] = 0u;
        ++left_over;
      }
    } else {
      for (unsigned polls = 0;;) {
        t.pass(me);
        unsigned v = *word;
        if ((v >> 16) != epoch || (v & kSyncCountMask) == S) break;
        if (++polls > limit) {
          t.pass(me);
          word[1 + (me >> 5)] |= 1u << (me & 31);
          t.pass(me);
          v = *word;
          *word += kSyncGaveUpOne;
          if (!((v >> 16) != epoch || (v & kSyncCountMask) == S)) mode = 0;
          ++gave_up;
          break;
        }
      }
    }
    if (mode == 0) return;
    unsigned long long left = ((unsigned long long)hi << 32 | lo) & ~(1ull << me);
    t.pass(me);
    merge(me);
    for (int j = 0; j < 64; ++j)
      if (mode == 2 && (left >> j & 1ull)) merge(j);
  });
  Turns(rng, work);
  for (int s = 0; s < splits; ++s) expect(merged[s] > 0, "grouped: a slice is not merged");
}

// tva_wide.hip: pieces at places base, base + 1, ...
void paired(std::mt19937& rng, int base, int pieces, unsigned limit) {
  std::vector<std::multiset<int>> slot(pieces);
  int complete = 0;
  std::multiset<int> all;
  for (int i = 0; i < pieces; ++i) all.insert(i);
  Work work(pieces, [&](Turns& t, int me) {
    std::multiset<int> mine{me};
    bool first = false;
    auto word = [&](int m) -> unsigned& { return header[wide_word(base + m)]; };
    auto arrive = [&](int m) {
      t.pass(me);
      first = word(m)++ == 0u;
      for (unsigned polls = 0; !first && polls <= limit; ++polls) {
        t.pass(me);
        const int at = tva::others_results(word(m), false);
        if (at >= 0) return at;
      }
      return -1;
    };
    auto leave = [&](int m) {
      t.pass(me);
      slot[me] = mine;
      t.pass(me);
      const unsigned w = word(m);
      word(m) |= tva::left_results(first, me);
      return tva::others_results(w, first);
    };
    auto add = [&](int m, int at) {
      word(m) = 0u;
      t.pass(me);
      mine.insert(slot[at].begin(), slot[at].end());
    };
    if (tva::merge_pieces(me, pieces, arrive, leave, add)) complete += mine == all;
  });
  Turns(rng, work);
  expect(complete == 1, "paired: not one workgroup with everything");
}

// Parts counted from zero: true for the last of them, which clears the word
bool last_of(Turns& t, int me, unsigned& word, int parts) {
  t.pass(me);
  const bool last = word++ == (unsigned)parts - 1u;
  if (last) {
    t.pass(me);
    word = 0u;
  }
  return last;
}

// tva_f32.hip
void counted(std::mt19937& rng, int tile, int parts) {
  std::vector<bool> stored(parts, false);
  int merged = 0;
  Work work(parts, [&](Turns& t, int me) {
    t.pass(me);
    stored[me] = true;
    if (!last_of(t, me, header[f32_word((unsigned)tile)], parts)) return;
    for (int s = 0; s < parts; ++s) expect(stored[s], "counted: merged before all results were there");
    ++merged;
  });
  Turns(rng, work);
  expect(merged == 1, "counted: not merged once");
}

// accept.hip: the parts of a row, then the rows of the tree
void greedy(std::mt19937& rng, int trees, int rows, int parts) {
  std::vector<int> walked(trees, 0);
  Work work(trees * rows * parts, [&](Turns& t, int me) {
    const int row = me / parts, b = row / rows;
    if (parts > 1 && !last_of(t, me, *greedy_word(header.data(), trees + row), parts)) return;
    if (rows > 1 && !last_of(t, me, *greedy_word(header.data(), b), rows)) return;
    ++walked[b];
  });
  Turns(rng, work);
  for (int w : walked) expect(w == 1, "greedy: a tree is not walked once");
}

void call(std::mt19937& rng) {
  const unsigned limits[] = {0u, 1u, 4u, 100000u};
  const unsigned limit = limits[rng() % 4];
  // (mostly the same few groups, places and tiles, so that calls meet in their lines)
  auto index = [&](int most) { return rng() % 4 ? (int)(rng() % 4) : (int)(rng() % most); };
  switch (rng() % 4) {
    case 0: grouped(rng, index(kMaxFusedGroups), 2 + (int)(rng() % (rng() % 4 ? 15 : 39)), limit); break;
    case 1: paired(rng, index(kMaxCounted - 12), 2 + (int)(rng() % 8), limit); break;
    case 2: counted(rng, rng() % 2 ? index(kMaxCounted) : (int)(rng() % 4) + kMaxFusedGroups * (int)(rng() % kCountingWords), 2 + (int)(rng() % 15)); break;
    default: greedy(rng, 1 + (int)(rng() % 2), 1 + (int)(rng() % 4), 1 + (int)(rng() % 3));
  }
  for (int i = 0; i < (int)header.size(); ++i)
    if (i % kLineWords >= kFirstCounting) expect(header[i] == 0u, "a counting word is not zero behind a call");
}

// Within its range every word is another one, inside the header and of the words that are its owner's
template <class F>
void owns(const char* who, int n, int lo, F word) {
  std::set<long long> seen;
  for (int i = 0; i < n; ++i) {
    const long long w = (long long)word(i);
    if (!seen.insert(w).second || w < 0 || w >= (long long)header.size() || w % kLineWords < lo) {
      expect(false, who);
      return;
    }
  }
}
}  // namespace

int main() {
  owns("wide_word", kMaxCounted, kFirstCounting, [](int i) { return wide_word(i); });
  owns("f32_word", kMaxCounted, kFirstCounting, [](int i) { return f32_word((unsigned)i); });
  owns("greedy_word", kGreedyWords, kFirstCounting, [](int i) { return greedy_word(header.data(), i) - header.data(); });
  for (int g = 0; g < kMaxFusedGroups; ++g) expect(group_word(g) == (unsigned long)g * kLineWords, "group_word");
  for (unsigned seed = 0; seed < 40 && bad == 0; ++seed) {
    std::mt19937 rng(seed);
    for (unsigned& w : header) w = 0u;
    for (int n = 0; n < 60 && bad == 0; ++n) call(rng);
    if (bad) std::printf("seed %u\n", seed);
  }
  std::printf("%d wrong; %d expired waits, %d times the last to come merged for others\n", bad, gave_up, left_over);
  return bad == 0 && gave_up > 0 && left_over > 0 ? 0 : 1;
}
