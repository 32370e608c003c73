// Who owns which word of a workspace's header: the words through which the workgroups of one call meet.  Plain C++, so that a
// host test can walk the protocols over one header.  Not installed.
//
// The header is kMaxFusedGroups lines of sixteen words behind the error word's 256 bytes, all zero before a workspace's first
// use; calls of every kind take turns on it, one at a time.  Of a line
//   word 0       the merge in tva_bf16.hip, a word per group (unit, row tile).  NOT zero between calls: it keeps the call number
//   words 1, 2   that merge's slices whose workgroup has given up waiting; a stray mark may stay
//   words 3 - 15 words that every call leaves at zero, and may therefore count in from zero: the pairs of tva_wide.hip, the parts
//                of tva_f32.hip, and (4 - 15) the rows and trees of the greedy launch (accept.hip)
#pragma once

namespace jk {

constexpr int kMaxFusedGroups = 508, kLineWords = 16;
constexpr int kFirstCounting = 3, kCountingWords = kLineWords - kFirstCounting;  // of a line
constexpr int kMaxCounted = kMaxFusedGroups * kCountingWords;
constexpr int kGreedyWords = kMaxFusedGroups * 12;

// Group word of tva_bf16.hip: bits 0-7 arrivals of this call, bits 8-15 workgroups that gave up waiting, bits
// 16-31 call number (epoch).  The last arriver adds 2^16 - S - (give-ups << 8): count and
// give-ups return to zero and the epoch moves on, which is what the waiting workgroups look for.
constexpr unsigned kSyncCountMask = 0xffu, kSyncGaveUpOne = 0x100u, kSyncEpochOne = 0x10000u;
constexpr unsigned long group_word(int group) { return (unsigned long)group * kLineWords; }

// Meeting of two pieces' workgroups of tva_wide.hip, at the place of the right one's first piece
constexpr int wide_word(int place) { return place / kCountingWords * kLineWords + kFirstCounting + place % kCountingWords; }

// Parts of a row tile of tva_f32.hip, counted from zero; the last to come clears it.  Neighbours 64 bytes apart (an atomic takes 11
// ns of the memory channel that has its word)
constexpr unsigned f32_word(unsigned tile) {
  constexpr unsigned lines = kMaxFusedGroups;
  return tile % lines * kLineWords + kFirstCounting + tile / lines;
}

// Counters of the greedy launch: number i's line and word in it, neighbours 256 bytes apart.  (With the words of four trees in
// one channel, four trees of 61 rows in two parts each spent 5 us on them.)
constexpr unsigned* greedy_word(unsigned* words, int i) {
  const int line = i % kMaxFusedGroups, blocks = kMaxFusedGroups / 4;
  return words + ((line % blocks) * 4 + line / blocks) * kLineWords + 4 + i / kMaxFusedGroups;
}

}  // namespace jk
