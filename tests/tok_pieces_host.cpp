// Host run of the decode plan (host_plan.cpp) and of the d_c 128 decode's
// balanced schedule (tok_pieces.h, step by step as tok_schedule takes it on the
// device).
//
//   plan H B CAP [DV]     prints the plan: balanced (0 or 1), pieces, split, workspace bytes
//   cut H B CAP           reads B lengths from stdin; prints "sequence first tokens" per piece
//   sweep H               every batch with a balanced schedule, lengths to the capacity, equal and
//                         mixed; prints "balanced plans, cuts, longest piece" and fails on a piece
//                         beyond the token list, too many pieces or tokens not covered once
//   quotients             tok_piece_count against integer division; fails on a difference
//   server H DH DV DC DR DTYPE B CAP
//                         batches up to B that one workspace, sized for B, holds and that plans
//                         with the most rows fit: "batches fitting of them, all fitting"
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "host_plan.h"
#include "tok_pieces.h"

using namespace egmla;

namespace {

eg_mla_dims layer(int heads) {
  eg_mla_dims d = {};
  d.num_heads = heads;
  d.head_dim = d.v_head_dim = d.latent_dim = d.gate_dim = 128;
  d.rope_dim = 64;
  d.vocab_size = 1000;
  d.page_size = 1;
  d.dtype = EG_MLA_BF16;
  return d;
}

struct Piece {
  int seq, first, tokens;
};

std::vector<Piece> cut(const std::vector<int>& len, int G) {
  const int B = static_cast<int>(len.size());
  int N = 0;
  for (int L : len) N += L;
  const TokSizes sizes = tok_sizes(N, G, B);
  uint64_t fits = 0;
  for (int lane = 0; lane < kTokCandidates; ++lane) {
    const int c = tok_candidate(sizes, lane);
    const float rc = 1.f / static_cast<float>(c);
    int k = 0;
    for (int L : len) k += tok_piece_count(L, rc);
    if (k <= tok_candidate_limit(G, lane)) fits |= uint64_t{1} << lane;
  }
  const int c = tok_candidate(sizes, tok_choice(fits));
  const float rc = 1.f / static_cast<float>(c);
  std::vector<Piece> out;
  for (int b = 0; b < B; ++b) {
    const int k = tok_piece_count(len[b], rc);
    if (k <= 0) continue;
    const int size = tok_piece_tokens(len[b], k);
    for (int i = 0; i < k; ++i) out.push_back({b, i * size, std::min(size, len[b] - i * size)});
  }
  return out;
}

// The longest piece, or -1 (with a message) if the cut is wrong.
int check(const std::vector<int>& len, int G, int heads) {
  const std::vector<Piece> p = cut(len, G);
  std::vector<int> at(len.size(), 0);
  int longest = 0;
  bool ok = static_cast<int>(p.size()) <= G;
  for (const Piece& x : p) {
    ok = ok && x.tokens > 0 && x.tokens <= kMaxSliceSplitTokens && x.first == at[x.seq];
    at[x.seq] += x.tokens;
    longest = std::max(longest, x.tokens);
  }
  ok = ok && at == len;
  if (!ok)
    std::printf("bad cut: H %d B %zu longest length %d: %zu pieces of at most %d, longest %d of %d tokens\n", heads,
                len.size(), *std::max_element(len.begin(), len.end()), p.size(), G, longest, kMaxSliceSplitTokens);
  return ok ? longest : -1;
}

bool plan_of(int heads, int B, int cap, DecodePlan* p, int v_dim = 128) {
  eg_mla_dims d = layer(heads);
  d.v_head_dim = v_dim;
  return make_decode_plan(d, B, cap, nullptr, p) == EG_MLA_OK;
}

int sweep(int heads) {
  long plans = 0, cuts = 0;
  int longest = 0;
  unsigned rng = 12345;
  auto next = [&](int n) { return static_cast<int>((rng = rng * 1664525u + 1013904223u) >> 8) % n; };
  for (int B = 33; B <= kTokMaxBatch; ++B)
    // capacities a step of about 3 % apart, and beyond the last that takes the schedule
    for (int cap = 1024; cap <= 64 * 1024; cap += 1 + cap / 32) {
      DecodePlan p;
      if (!plan_of(heads, B, cap, &p)) return 2;
      if (!p.tok_balanced) continue;
      ++plans;
      std::vector<std::vector<int>> mixes;
      for (int L : {cap, cap - cap / 7, cap / 2 + 1}) mixes.push_back(std::vector<int>(B, L));  // equal
      for (int lo : {0, cap / 2, cap - cap / 8}) {                                               // mixed
        std::vector<int> v(B);
        for (int& L : v) L = lo + next(cap - lo + 1);
        v[0] = cap;
        mixes.push_back(v);
      }
      std::vector<int> few(B, 0);  // some full, the others empty or short
      for (int b = 0; b < B; ++b) few[b] = b % 3 == 0 ? cap : b % 3 == 1 ? 0 : 1 + next(64);
      mixes.push_back(few);
      for (const auto& v : mixes) {
        ++cuts;
        const int got = check(v, p.pieces, heads);
        if (got < 0) return 1;
        longest = std::max(longest, got);
      }
    }
  std::printf("%ld %ld %d\n", plans, cuts, longest);
  return 0;
}

// tok_piece_count against the integer quotient: every multiple of the step of 16 up to the list, lengths around
// every multiple of it and the largest.
int quotients() {
  for (int c = 16; c <= kMaxSliceSplitTokens; c += 16) {
    const float rc = 1.f / static_cast<float>(c);
    for (int64_t m = 0; m <= (1 << 22); m += c)
      for (int d = -1; d <= 1; ++d) {
        const int64_t L = m + d;
        if (L < 0 || L >= (1 << 22)) continue;
        if (tok_piece_count(static_cast<int>(L), rc) != (L + c - 1) / c) return 1;
      }
  }
  std::printf("0\n");
  return 0;
}

int server(char** v) {
  eg_mla_dims d = layer(std::atoi(v[0]));
  d.head_dim = std::atoi(v[1]);
  d.v_head_dim = std::atoi(v[2]);
  d.latent_dim = d.gate_dim = std::atoi(v[3]);
  d.rope_dim = std::atoi(v[4]);
  d.dtype = std::atoi(v[5]);
  const int B = std::atoi(v[6]), cap = std::atoi(v[7]);
  const size_t bytes = decode_workspace_bytes(d, B, cap, nullptr);
  int old_fit = 0, both = 0, now = 0;
  for (int b = 1; b <= B; ++b) {
    DecodePlan p;
    if (make_decode_plan(d, b, cap, nullptr, &p, PlanRows::kMost) != EG_MLA_OK) return 2;
    const bool most = p.bytes <= bytes, fit = fit_decode_plan(d, b, cap, nullptr, bytes, &p) == EG_MLA_OK;
    if (fit && p.bytes > bytes) return 2;
    old_fit += most;
    both += most && fit;
    now += fit;
  }
  std::printf("%d %d %d\n", old_fit, both, now);
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  if (argc == 2 && !std::strcmp(argv[1], "quotients")) return quotients();
  if (argc == 10 && !std::strcmp(argv[1], "server")) return server(argv + 2);
  if (argc == 3 && !std::strcmp(argv[1], "sweep")) return sweep(std::atoi(argv[2]));
  if (argc != 5 && argc != 6) return 2;
  const int heads = std::atoi(argv[2]), B = std::atoi(argv[3]), cap = std::atoi(argv[4]);
  DecodePlan p;
  if (!plan_of(heads, B, cap, &p, argc == 6 ? std::atoi(argv[5]) : 128)) return 2;
  if (!std::strcmp(argv[1], "plan")) {
    std::printf("%d %d %d %zu\n", p.tok_balanced ? 1 : 0, p.pieces, p.split_tokens, p.bytes);
    return 0;
  }
  if (std::strcmp(argv[1], "cut") || !p.tok_balanced) return 2;
  std::vector<int> len(B);
  for (int& L : len)
    if (std::scanf("%d", &L) != 1) return 2;
  for (const Piece& x : cut(len, p.pieces)) std::printf("%d %d %d\n", x.seq, x.first, x.tokens);
  return 0;
}
