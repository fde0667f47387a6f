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
// Pieces of a sequence of L > 0 tokens beyond its first, ceil(L / c) - 1, from
// tok_key(L) and rc = 1 / c.  (L - 1/2) / c is at least 1 / (2 c) away from any
// whole number, more than the two roundings move it for L below 2^22, so three
// instructions do.  (The search of tok_schedule runs this for every sequence and
// candidate; with an integer quotient and its corrections the launch that holds
// it took 1.2 us more for 384 sequences.)
constexpr float tok_key(int L) { return L > 0 ? static_cast<float>(L) - 0.5f : 0.f; }
constexpr int tok_more_pieces(float key, float rc) { return static_cast<int>(key * rc); }
constexpr int tok_piece_count(int L, float rc) { return L > 0 ? 1 + tok_more_pieces(tok_key(L), rc) : 0; }
// Tokens of each of its k > 0 pieces (the last may have fewer): at most c, so
// that the k - 1 first pieces stay below L.
constexpr int tok_piece_tokens(int L, int k) { return ((L + k - 1) / k + 15) & ~15; }

}  // namespace egmla
