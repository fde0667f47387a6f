// Piece sizes of the d_c 128 decode's balanced schedule: the arithmetic of
// tok_schedule (split_slice.h), as constexpr functions so that the host can run
// it too.  G pieces at most, B < G sequences, N tokens in all.
#pragma once

#include "host_plan.h"

namespace egmla {

constexpr int kTokCandidates = 64;               // piece sizes tried, one per lane of a wave
constexpr int kTokEvenLane = kTokCandidates - 1;  // the one that cuts into G / 2 pieces

// Multiples of 16, none beyond the split kernel's token list: lane i < 63 tries
// lo + step * i, from N / G, below which there are always more than G pieces,
// to N / (G - B), which always fits (the plan keeps that end within the list).
// The last lane tries a tenth above an even cut into G / 2 pieces; where it
// makes at most that many, one work-group per compute unit starts, loads and
// merges half as often.  It is about twice the others, so it is the one that
// can reach the list's end (from 0.95 M tokens at 16 heads): it stops there.
struct TokSizes {
  int lo, step, even;
};
constexpr TokSizes tok_sizes(int N, int G, int B) {
  const int half = G / 2;
  const int lo0 = (N / G + 15) & ~15, hi0 = (N / (G - B) + 16) & ~15;
  const int lo = lo0 > kTokPieceMin ? lo0 : kTokPieceMin, hi = hi0 > lo ? hi0 : lo;
  const int step = ((hi - lo) / (kTokCandidates - 2) + 16) & ~15;
  const int even0 = (N / half + N / (10 * half) + 15) & ~15;
  const int even = even0 > kTokPieceMin ? even0 : kTokPieceMin;
  return {lo, step, even < kMaxSliceSplitTokens ? even : kMaxSliceSplitTokens};
}
constexpr int tok_candidate(const TokSizes& s, int lane) {
  const int c = lane == kTokEvenLane ? s.even : s.lo + s.step * lane;
  return c < kMaxSliceSplitTokens ? c : kMaxSliceSplitTokens;
}
// Pieces that lane's candidate may make to be taken.
constexpr int tok_candidate_limit(int G, int lane) { return lane == kTokEvenLane ? G / 2 : G; }
// The candidate taken, of those that keep to their limit (a bit each).
constexpr int tok_choice(uint64_t fits) {
  if (fits >> kTokEvenLane) return kTokEvenLane;
  return fits ? __builtin_ctzll(fits) : kTokEvenLane - 1;
}
// Pieces of a sequence of L tokens: ceil(L / c), exact for lengths below 2^24 (rc = 1 / c).
constexpr int tok_piece_count(int L, int c, float rc) {
  const int x = L + c - 1;
  const int q = static_cast<int>(static_cast<float>(x) * rc);
  const int r = x - q * c;
  return q + (r >= c ? 1 : 0) - (r < 0 ? 1 : 0);
}
// Tokens of each of its k > 0 pieces (the last may have fewer): at most c, so
// that the k - 1 first pieces stay below L.
constexpr int tok_piece_tokens(int L, int k) { return ((L + k - 1) / k + 15) & ~15; }

}  // namespace egmla
