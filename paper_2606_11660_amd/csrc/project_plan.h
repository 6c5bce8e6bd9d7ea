// Host-side plan of the projection: which kernel a call takes, and the rounds
// of a call whose workspace or grid does not hold all of its chunks.  Plain C++
// with no device code, so the rules can be checked on the CPU.
#pragma once

#include <algorithm>
#include <stddef.h>
#include <stdint.h>

#include "kernels.h"

namespace attr {

// Rates of the two kernels in elements of token rows (a and g widths times
// tokens) per us and CU, and the latency of the longest item's K-groups that
// the split saves, in us per group; from 12-layer GPT-2-shaped and 2- to
// 6-layer 1B-shaped calls of 16 to 16384 tokens, even and ragged.
struct FewRates {
  double general, few, group;
};
inline FewRates few_rates(bool bf16, int nk) {
  if (bf16) return nk == 1 ? FewRates{14000, 12800, 0.3} : nk == 2 ? FewRates{12000, 11250, 0.15} : FewRates{10500, 8000, 0.08};
  return FewRates{7000, 6700, 0.3};
}

// The general kernel reads a once per group and runs a little faster where
// there are items enough; the split one has a chain a quarter as long and
// wastes at most 63 tokens of a chunk.  Both times are modelled and the lower
// one is taken.  fp32 at k = 32 and 64 is bound by the matrix cores and always
// takes the split kernel, which computes no tile without tokens (16 ragged
// GPT-2-shaped examples of up to 512 tokens: 682 -> 609 us at k = 32, 1224 ->
// 926 at k = 64; 16384 tokens: 1916 -> 1752 and 3552 -> 2796).  bf16, k = 16,
// 12 GPT-2-shaped layers, general / split: one example of 16 tokens 46 / 16
// us, 389 tokens 86 / 46, 1024 tokens 99 / 75, 8 x 512 tokens 228 / 209, 16 x
// 512 397 / 392, 32 x 512 743 / 759; 2 1B-shaped layers: 149 tokens 229 / 29,
// 4 x 1343 297 / 187, 8 x 2048 506 / 538.
inline ProjFewPlan plan_project_few(bool bf16, int nk, int64_t group_cost, int64_t slot_cost, int64_t longest,
                             int64_t n_slots, int64_t n_ex, int64_t T, bool ragged) {
  ProjFewPlan P{};
  constexpr int64_t kCus = 256;
  const int64_t ct = kProjectChunk;
  if (T > ((int64_t)1 << 24)) return P;  // (refused; the workspace query takes any length)
  if (bf16 || nk == 1) {
    // tokens an example costs; of ragged ones about 0.56 T are valid (lengths
    // even over T / 8 .. T), with half a chunk lost at the end.  At k = 16 a
    // chunk's tokens are spread over the waves and only the loads cost.
    const double valid = ragged ? 0.56 * (double)T : (double)T;
    auto cost_tokens = [&](int64_t c) {
      if (nk == 1) return valid + 32.0;
      return ragged && T > c ? valid + 0.5 * (double)c : (double)((T + c - 1) / c * c);
    };
    const FewRates r = few_rates(bf16, nk);
    const double tg = (double)group_cost * cost_tokens(ct) * (double)n_ex / (double)kCus / r.general;
    const double tf = (double)slot_cost * cost_tokens(64) * (double)n_ex / (double)kCus / r.few;
    const double groups = (double)longest * (bf16 ? 2 : 4) / 128.0;
    if (!(tf < tg + r.group * groups)) return P;
  }
  // One token tile per workgroup where even then few workgroups exist and the
  // modules are wide: R and S are read four times as often (one 149-token
  // example of 2 1B-shaped layers: 40 -> 29 us; of 128 tokens over 12
  // GPT-2-shaped layers: 28 -> 32 us).
  // (in double: the workspace query takes any count)
  const double blocks = (double)n_slots * (double)((T + 15) / 16) * (double)n_ex;
  P.ct = blocks * 24 <= (double)(slot_cost / n_slots) ? 16 : 64;
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
