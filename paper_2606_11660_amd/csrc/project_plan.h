// Host-side plan of the projection: which kernel a call takes, and the rounds
// of a call whose workspace or grid does not hold all of its chunks.  Plain C++
// with no device code, so the rules can be checked on the CPU.
#pragma once

#include <algorithm>
#include <cmath>
#include <stddef.h>
#include <stdint.h>

#include "kernels.h"

namespace attr {

// The split kernel's rate over the general one's, and the lead that a quarter as
// long a chain gives it, in token-elements per element of the widest module.
struct FewRule {
  double rate, lead;
};
inline FewRule few_rule(bool bf16, int nk, bool tok) {
  if (tok) return nk == 1 ? FewRule{0.75, bf16 ? 28000.0 : 40000.0} : nk == 2 ? FewRule{0.79, 4000} : FewRule{0.60, 1000};
  if (!bf16) return {0.94, 12000};
  return nk == 1 ? FewRule{0.84, 26000} : nk == 2 ? FewRule{0.95, 6000} : FewRule{0.91, 4000};
}

// Which kernel a call takes.  The general kernel reads a once per group and runs a
// little faster where there are items enough; the split one has a chain a quarter
// as long and wastes at most 63 tokens of a chunk.  A chunk costs either kernel
// its tokens and some more (64 of 256, 16 of 64: a 60-token example takes the
// general kernel 40% of a 256-token chunk's time).  The rule sees the widths of
// the modules but not which of them share their input rows: the two kernels add in
// different orders, and modules that share rows give the same bits as separate
// copies.  So the line lies between the two.  General / split in us, bf16, k = 16:
// 2 1B-shaped layers of 8 x 2048 tokens 503 / 541 shared and 529 / 543 separate,
// of 6 x 2048 440 / 394 and 383 / 402 (general from here on), of 4 x 2048 312 /
// 285 and 259 / 270, of 2 x 2048 280 / 157; 12 GPT-2-shaped layers of 16 x 512 376
// / 377, of 8 x 512 215 / 198, of 200 x 60 943 / 546, one of 389 tokens 86 / 46.
// k = 64: 2 1B-shaped layers of 2 x 2048 404 / 328, of 4 x 2048 449 / 486.
// Lengths are on the device and not known here: three quarters of a slot's tokens
// are counted where they are given.  Next to the line the split kernel is far
// ahead where they are even over T / 8 .. T (k = 32, 2 1B-shaped layers, 8 x 2048:
// 323 / 249) and behind where nearly all are T (497 / 577).  fp32 at k = 32 and 64
// is bound by the matrix cores and always takes the split kernel, which computes
// no tile without tokens (16 ragged GPT-2-shaped examples of up to 512 tokens: 682
// / 609 at k = 32, 1224 / 926 at k = 64; 16384 tokens: 1916 / 1752 and 3552 /
// 2796).
// Per-token calls (tok) have a rule of their own: both kernels also write k^2
// values per token and module, which hides a part of the general one's chain.
// bf16, k = 16: 12 GPT-2-shaped layers of 16 x 512 tokens 507 / 542, of 8 x 512
// 296 / 296, one of 512 tokens 73 / 51; 2 1B-shaped layers of 4 x 2048 289 / 299
// (general from here on), of 2 x 2048 186 / 151.  k = 32: 4 GPT-2-shaped layers of
// 8 x 512 150 / 175 (general), of 4 x 512 90 / 88.  fp32, k = 16: 12 layers of 16
// x 512 896 / 940, of 8 x 512 510 / 459 (general), of 4 x 512 272 / 238.  k = 64,
// bf16: 2 layers of 4 x 512 111 / 139 (general), of 2 x 512 78 / 63.  fp32 at k =
// 32 and 64 up to 6% behind at single sizes (4 layers of 8 x 512, k = 32: 233 /
// 249), up to 70% ahead at others.
// slot_cost, longest: sum and maximum over the modules of d_in + d_out.
inline ProjFewPlan plan_project_few(bool bf16, int nk, bool tok, int64_t slot_cost, int64_t longest,
                                    int64_t n_slots, int64_t n_ex, int64_t T, bool ragged) {
  ProjFewPlan P{};
  if (T > ((int64_t)1 << 24)) return P;  // (refused; the workspace query takes any length)
  if (bf16 || nk == 1) {
    const double valid = ragged ? 0.75 * (double)T : (double)T;
    // tokens that an example in chunks of c costs, extra ones per chunk
    auto cost = [&](double c, double extra) {
      return valid + extra * (ragged && (double)T > c ? valid / c + 0.5 : std::ceil((double)T / c));
    };
    const FewRule r = few_rule(bf16, nk, tok);
    const double behind = cost(64, 16) / r.rate - cost(project_chunk_tokens(nk, tok), 64);
    if (!((double)slot_cost * (double)n_ex * behind < r.lead * (double)longest)) return P;
  }
  // One token tile per workgroup where even then few workgroups exist and the
  // modules are wide: the longest module's chain is shorter, R and S are read four
  // times as often (one 149-token example of 2 1B-shaped layers: 40 -> 29 us; of 128
  // tokens over 12 GPT-2-shaped layers: 28 -> 32 us).  A summed call pays for the
  // partials of more chunks, k x k each, and in bf16 for a reduce where 64 tokens
  // hold an example, while the chain of the matrix products grows with k only in
  // fp32: so from k = 32 in bf16 and at k = 64 in fp32 the longest module has to be
  // worth them.  16 / 64 tokens, bf16, k = 64: one GPT-2-shaped layer of 300 tokens 90
  // / 50 us (the general kernel 72), of 512 134 / 62 (83), 2 1B-shaped layers of 300
  // tokens 132 / 90, of 16 tokens 42 / 49, a module of 8192 x 28672 and 128 tokens
  // 156 / 202; k = 32: one GPT-2-shaped layer of 512 tokens 46 / 32, 2 1B-shaped layers of
  // 149 44 / 54; fp32, k = 64: one GPT-2-shaped layer of 149 tokens 73 / 90, of 512
  // 153 / 110.
  // (in double: the workspace query takes any count)
  const double blocks = (double)n_slots * (double)((T + 15) / 16) * (double)n_ex;
  const double more = (double)((T + 15) / 16 - (T + 63) / 64) + (bf16 && T <= 64 ? 6 : 0);
  const double worth = bf16 ? (nk == 1 ? 0 : nk == 2 ? 580 : 1800) : (nk == 4 ? 320 : 0);
  const bool one = tok || T <= 16 || (double)longest >= worth * more;
  P.ct = one && blocks * 24 <= (double)(slot_cost / n_slots) ? 16 : 64;
  P.n_chunks = (int)((T + P.ct - 1) / P.ct);
  return P;
}

// A launch has fewer than 2^32 threads: fewer than 2^24 workgroups of 256.
constexpr int64_t kProjectMaxBlocks = ((int64_t)1 << 24) - 1;

// The query asks for the partials of all chunks up to kProjectRoundBytes, beyond
// that for as many chunks as those bytes hold: a round of 256 MiB is at least
// 16384 workgroups.
constexpr size_t kProjectRoundBytes = (size_t)256 << 20;
inline size_t project_few_query(const ProjFewPlan& P, size_t part_bytes) {
  if (!part_bytes) return 0;  // (a count past 64 bits: the call is refused)
  const size_t fit = std::max<size_t>(1, kProjectRoundBytes / part_bytes);
  return part_bytes * std::min<size_t>(fit, (size_t)P.n_chunks);
}

// Chunks per round of the split kernel: as many as one launch takes (items:
// slots times examples) and the partials have room for (room bytes; part_bytes a
// chunk of all items; 0: no partials).  The least workspace that a call accepts
// holds the general kernel's partials, one chunk of 256 tokens at least, so it
// holds one of these.
inline int project_few_round(const ProjFewPlan& P, int64_t items, size_t room, size_t part_bytes) {
  const int64_t fit = part_bytes ? (int64_t)(room / part_bytes) : P.n_chunks;
  return (int)std::min<int64_t>({fit, kProjectMaxBlocks / items, P.n_chunks});
}

}  // namespace attr
