// Two loops of tva_wide.hip, apart from what their steps do: the kernel walks them with its own steps, and a host test with
// steps that check the order (nothing that a run on the card could show: a transfer that was not waited for has usually
// arrived, and a workgroup hardly ever stops waiting for another).  The first is the order in which a wave asks for the tiles
// of its piece, waits for them and reads them, the second the merge of the pieces.  Not installed.
#pragma once

namespace jk {
namespace tva {

// Tiles asked for in front of the one in use: a ring of 64 KB for each of K and V, of tiles of 32 bf16 rows, less one
constexpr int wide_ahead(int head_dim) { return 64 * 1024 / (32 * 2 * head_dim) - 1; }

template <int N>
struct Const {
  static constexpr int value = N;
};

// A wave's transfers complete in the order in which they were issued, so a wait is a number of tiles that may still be on their
// way, and holds for a tile only if that many were asked for behind it.  The steps:
//   ask(i)            ask for tile i
//   spare()           ask for a tile that nobody needs (to where nobody reads)
//   wait(left, most)  until no more than min(left, most) tiles are on their way (most: a constant's type)
//   meet()            the workgroup's barrier
//   first()           reads K of tile 0
//   step(i)           one tile, wherever it lies: reads K of tile i + 1, where there is one, and V of tile i
//   run(i)            in front of four such steps without masks
//   run_step(i, u)    step i + u of them; asks for tile i + u + AHEAD, or, where that is not a tile without masks, for a spare one
// n tiles, the first n_full of them without masks, of which min(n, AHEAD) have been asked for.  The ring has a place more than
// AHEAD: while tile i is in use nobody reads tile i - 1 any more, and its place takes tile i + AHEAD.
template <int AHEAD, class Ask, class Spare, class Wait, class Meet, class First, class Step, class Run, class RunStep>
__attribute__((always_inline)) constexpr void walk_tiles(int n, int n_full, bool only_moves, Ask& ask, Spare& spare, Wait& wait,
                                                         Meet& meet, First& first, Step& step, Run& run, RunStep& run_step) {
  auto least = [](int a, int b) { return a < b ? a : b; };
  auto most = [](int a, int b) { return a > b ? a : b; };
  int asked = least(n, AHEAD);  // tiles asked for, in order
  // Tile i is there, for the whole workgroup; everybody is also done with tile i - 2, whose place is therefore free
  auto landed = [&](int i) __attribute__((always_inline)) {
    wait(asked - 1 - i, Const<AHEAD - 2>());
    meet();
  };
  wait(asked - 1, Const<AHEAD - 1>());
  meet();
  first();
  if (only_moves) {  // a wave of padding rows
    for (int i = 0; i + 1 < n; ++i) {
      landed(i + 1);
      for (; asked < least(n, i + AHEAD + 1); ++asked) ask(asked);
    }
    if (n_full >= 5 && ((n_full - 1) & ~3) + 1 == n) meet();  // (the others' last step of four met for a tile that does not exist)
    return;
  }
  int i = 0;
  auto one = [&]() __attribute__((always_inline)) {
    if (i + 1 < n) landed(i + 1);
    for (; asked < least(n, i + AHEAD + 1); ++asked) ask(asked);
    step(i);
    ++i;
  };
  one();
  // Runs of four tiles without masks, from tile 1 on.  Their waits are constants: a step leaves AHEAD - 2 tiles on their way, so
  // that many have to be asked for behind the tile it needs (K of the next).  That is so where tile t was asked for in step
  // t - AHEAD, one tile a step.  Two kinds of tiles are not:
  //   - the first ones of a piece with fewer tiles than the ring takes: spare ones up to the ring's size follow them;
  //   - the first tile with a mask, asked for between two runs, behind the AHEAD mod 4 = 3 spare ones of the run in front that
  //     have had its turn and the next two's.  Its K is read by the last run only if that ends right in front of it: then
  //     two spare ones follow.
  // (A spare tile is 8 or 16 KB out of a cache.)
  static_assert(AHEAD % 4 == 3, "the number of spare ones above");
  if (n_full >= 5)
    for (int k = asked; k < AHEAD + 1; ++k) spare();
  for (; i + 4 <= n_full; i += 4) {
    for (asked = most(asked, n_full); asked < least(n, i + AHEAD); ++asked) ask(asked);
    if (i + 4 == n_full && n_full < n) {
      spare();
      spare();
    }
    run(i);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      wait(AHEAD - 2, Const<AHEAD - 2>());
      meet();
      run_step(i, u);
    }
  }
  wait(0, Const<0>());  // (what is still on its way: spare ones, tiles with masks)
  asked = most(asked, least(n_full, i + AHEAD));
  while (i < n) one();
}

// Merge of the pieces of a row tile, two and two: 0 with 1, 2 with 3, then those with each other, and so on.  Of the two
// workgroups that meet the first to come leaves its results in memory and is done; the second, which still has its own in
// registers, adds them: half the traffic of leaving all results for another kernel, and nobody waits for a workgroup that has
// not come yet (so any number of them may still be to start).  The second does wait for the first one's stores, but not
// for ever: then it leaves its results as well, and of the two the one whose word about that is the later finds the other's
// and adds them.  So everything is added whoever is held up, and for however long.
//
// A workgroup leaves its results at the place of its own piece (`split`), wherever it has got to: those that it left before it
// went on after all are read by nobody.  The meeting of two groups of pieces has a word at the place of the right one's
// first piece: arrivals, and for each of the two that its results are in memory, and the piece where.  Zero again behind it.
constexpr unsigned kFirstLeft = 0x10u, kSecondLeft = 0x20u;
constexpr int kMeetingPieces = 1 << 12;  // (a sequence's pieces: at most the batch's places, 64 sequences times 64 splits)
constexpr unsigned left_results(bool first, int piece) { return first ? kFirstLeft | (unsigned)piece << 8 : kSecondLeft | (unsigned)piece << 20; }
constexpr int others_results(unsigned word, bool first) {  // where the other one's are, or -1
  if (!(word & (first ? kSecondLeft : kFirstLeft))) return -1;
  return (int)(word >> (first ? 20 : 8)) & (kMeetingPieces - 1);
}

// The steps:
//   arrive(m)    at meeting m: where the other one's results are, if this is the second to come and they are there in time,
//                or -1
//   leave(m)     leaves the own results, says so, and returns where the other one's are if those were left before, or -1
//   add(m, at)   adds the results at place `at` to the own, and clears the meeting's word (both have said their last)
// True for the workgroup that has all pieces in the end.
template <class Arrive, class Leave, class Add>
__attribute__((always_inline)) constexpr bool merge_pieces(int split, int pieces, Arrive& arrive, Leave& leave, Add& add) {
  int lo = split;  // this workgroup holds pieces lo ... lo + held - 1
  for (int held = 1; held < pieces; held *= 2) {
    const bool right = (lo & held) != 0;
    if (!right && lo + held >= pieces) continue;  // (nobody there)
    const int m = right ? lo : lo + held;
    int at = arrive(m);
    if (at < 0) {
      at = leave(m);
      if (at < 0) return false;
    }
    // (of the other group, whatever a workspace that was never initialised says)
    const int first = right ? lo - held : m, last = (right || m + held < pieces ? first + held : pieces) - 1;
    add(m, at < first ? first : (at > last ? last : at));
    lo &= ~held;
  }
  return true;
}

}  // namespace tva
}  // namespace jk
