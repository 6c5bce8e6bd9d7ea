// CPU check of the projection planner's arithmetic (host-only header), over
// widths, module counts, example counts and lengths: the least workspace that a
// call accepts (the general kernel's partials) holds at least one chunk of the
// few-item plan's partials, so its rounds advance and cover every chunk, and the
// queried size takes them in as few rounds as launches of fewer than 2^32 threads
// allow.  Prints "ok" or the first violation and
// exits non-zero.
#include <cstdio>

#include "project_plan.h"

int main() {
  long long checked = 0;
  for (bool bf16 : {true, false})
    for (int nk : {1, 2, 4})
      for (long long d : {64ll, 768ll, 4096ll, 65536ll})
        for (long long mods : {1ll, 3ll, 4ll, 48ll, 64ll, 112ll, 4096ll})
          for (long long n : {1ll, 2ll, 7ll, 64ll, 1000ll, 65536ll, 1ll << 22, 1ll << 24})
            for (long long T : {1ll, 16ll, 63ll, 64ll, 65ll, 255ll, 256ll, 257ll, 2048ll, 100000ll, 1ll << 24})
              for (bool ragged : {false, true}) {
                const long long ct = attr::project_chunk_tokens(nk, false), chunks = (T + ct - 1) / ct;
                if ((double)mods * chunks * n > (double)(1 << 24)) continue;  // the call is refused
                if (mods * n == 1 << 24) continue;  // one launch cannot take even one chunk: refused
                const attr::ProjFewPlan P =
                    attr::plan_project_few(bf16, nk, false, 2 * d * mods, 2 * d, mods, n, T, ragged);
                const bool always = !bf16 && nk > 1;  // fp32 at k = 32 and 64: no general kernel
                if (always && (!P.ct || !attr::plan_project_few(bf16, nk, true, 2 * d * mods, 2 * d, mods, n, T, ragged).ct)) {
                  std::printf("violation: fp32 nk=%d d=%lld mods=%lld n=%lld T=%lld: no split plan\n", nk, d, mods, n, T);
                  return 1;
                }
                if (!P.ct) continue;
                const size_t kk = (size_t)256 * nk * nk, part = mods * n * kk * 4;
                bool ok = (P.ct == 16 || P.ct == 64) && (long long)P.n_chunks * P.ct >= T &&
                          (long long)(P.n_chunks - 1) * P.ct < T;
                const int least = attr::project_few_round(P, mods * n, part * (size_t)chunks, part);
                const int most = attr::project_few_round(P, mods * n, part * (size_t)P.n_chunks, part);
                const int tok = attr::project_few_round(P, mods * n, 0, 0);  // per-token calls: no partials
                ok = ok && least >= 1 && least <= most && most == tok;
                const size_t query = attr::project_few_query(P, part);
                ok = ok && query >= part && (query <= attr::kProjectRoundBytes || query == part) &&
                     (query == part * P.n_chunks || query + part > attr::kProjectRoundBytes);
                // fewer than 2^32 threads in x, and no smaller than it has to be
                ok = ok && mods * n * most * 256 < 1ll << 32;
                ok = ok && (most == P.n_chunks || mods * n * (most + 1) * 256 >= 1ll << 32);
                if (!ok) {
                  std::printf("violation: bf16=%d nk=%d d=%lld mods=%lld n=%lld T=%lld ragged=%d -> ct=%d chunks=%d round=%d\n",
                              bf16, nk, d, mods, n, T, ragged, P.ct, P.n_chunks, least);
                  return 1;
                }
                ++checked;
              }
  std::printf("ok %lld plans\n", checked);
  return 0;
}
