// Which form of the decode attention a batch takes.  Host code only.
#pragma once

#include <algorithm>

namespace mtmc {
namespace bf16 {

// How many sequences of a prompt share a workgroup of the decode attention (1: the plain form, a workgroup per sequence and
// kv head), for B sequences in runs of `share` samples per prompt that advance together.
//
// The plain form takes a round of workgroups per 256 (sequence, kv head) pairs at 128 dims (a CU holds one by its registers),
// per 512 at 64 dims; the shared form reads a prompt's pages once for n sequences, but each one's own pages with the
// columns of the others idle.  Up to 256 pairs the plain form is one round and the shared form would leave CUs idle.  Beyond,
// the shorter of two measured times: with p pairs of pages read by the 8 wavefronts of a workgroup,
//   128 dims: plain 5 + 2 p / 8 us a round, shared 6 + 3 p / 8;
//    64 dims: plain 4.2 + 1.3 p / 8 (2.5 more for each further round), shared 4.4 + p / 8,
// p = shared + own pairs in the plain form and shared + n own in the other, own = the mean over the generation.  Over 2636
// cases (20 to 128 rows, 2 to 16 samples per prompt, 4 to 16 kv heads, 16 to 2048 + 33 to 1025 tokens) the choice takes 0.79 of
// the plain form's time and is slower than it by more than 3 % in 43, by more than 10 % in 10 (at most 33 %: a short prompt and
// a long generation at the edge of a round); the fewest sequences that make one round, whatever the lengths, 0.80, 327 and
// 200 (at most 120 %: 35 rows of 8 kv heads and 64 dims, 7 samples, 16 + 512 tokens, 11.0 us against 5.0).
// By the call's sizes alone, and the padded length where prompts differ: calls of one shape take one form.
inline int attention_sequences(int head_dim, int n_q_heads, int n_kv_heads, int B, int share, int prompt_len, int max_new) {
  const int pairs = B * n_kv_heads, most = std::min(16 * n_kv_heads / n_q_heads, 8);  // 16 columns; 8 wavefronts append
  if (share < 2 || B % share != 0 || pairs <= 256) return 1;
  const double shared = prompt_len / 32, own = std::max(1.0, (prompt_len % 32 + 0.5 * max_new) / 32.0);
  auto rounds = [](int workgroups, int per) { return (workgroups + per - 1) / per; };
  auto time = [&](int n) {
    const double p = (shared + n * own) / 8.0;
    if (head_dim == 128) return n == 1 ? rounds(pairs, 256) * (5.0 + 2.0 * p) : rounds(pairs / n, 256) * (6.0 + 3.0 * p);
    return n == 1 ? rounds(pairs, 512) * (6.7 + 1.3 * p) - 2.5 : rounds(pairs / n, 256) * (4.4 + p);
  };
  int best = 1;
  for (int n = 2; n <= most; ++n)
    if (share % n == 0 && time(n) < time(best)) best = n;
  return best;
}

}  // namespace bf16
}  // namespace mtmc
