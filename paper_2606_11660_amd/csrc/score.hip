// Query x gradient-store scoring with exact streaming top-k (section
// "Attribution Pipelines": every gradient store supports exact top-k lookup
// of the most influential items).
//
// Score tiles are 64 queries x 128 store rows, a matrix-core GEMM over D
// (fp16 16x16x32 or fp32 16x16x4 MFMA, fp32 accumulate).  Store rows stream
// with line-coalesced loads and pass through a per-wave LDS tile into MFMA
// fragments (as in the projection); query fragments come from L2.
//
// Three plans, chosen on the host from the problem shape:
//  * streaming (large stores, fewer than 128 fp16 queries): see
//    score_stream_kernel.  Rows are visited in increasing index order, so a
//    strict ">" keeps the lower index on ties.  The Q x N score matrix never
//    reaches memory.
//  * GEMM (128 or more fp16 queries): the 256 x 256 GEMM core scores chunks
//    of rows into the workspace and an exact selection kernel reads them.
//  * split-K (small stores, too few tiles to fill 256 CUs): workgroups own
//    (tile, D-slice) pairs and write fp32 partial scores; one workgroup per
//    query sums the slices in slice order and selects by a threshold from
//    its threads' best rows and a sort.
// Where rows are partitioned, the sorted lists are merged per query in (score
// desc, index asc) order by a threshold and a sort (k up to 8: by rounds of
// arg-max), which also merges a previous result when a store is scored chunk by
// chunk.
#include <type_traits>

#include "common.h"
#include "gemm.h"
#include "kernels.h"

namespace attr {
namespace {

constexpr int SQB = 64;       // queries per workgroup
constexpr int STN = 128;      // store rows per tile (4 waves x 32 rows)
constexpr int SPD = 3;        // 128-byte K-groups of store loads in flight (up to 12: no faster)

template <bool F16>
struct STag;
template <>
struct STag<true> {
  using tag = F16Tag;
  static constexpr int bytes = 2;
};
template <>
struct STag<false> {
  using tag = F32Tag;
  static constexpr int bytes = 4;
};

// acc[qt][rt] (+)= Q[16 qt + i, groups) . G[32 wave + 16 rt + j, groups) for
// the K-groups [g_begin, g_end).  Lane layout of acc: query 16 qt + 4 (lane
// / 16) + r (register r), row 16 rt + lane % 16.
// QT: 16-query tiles of the block (1, 2 or 4): a block of few queries issues no
// products and no loads for the others (10 queries x 11335 rows x 6528 in fp16
// 64 -> 51 us a call, 15 x 6161 x 3840 in fp32, where the products count, 64 ->
// 40 us).
template <bool F16, int QT>
__device__ inline void score_tile(__amdgpu_buffer_rsrc_t rq, int64_t ldq,
                                  __amdgpu_buffer_rsrc_t rg, int64_t ldg, int g_begin,
                                  int g_end, int lane, i32x4* __restrict__ xp,
                                  f32x4 (&acc)[QT][2]) {
  using Tag = typename STag<F16>::tag;
  constexpr int EB = STag<F16>::bytes;
  constexpr int E = 16 / EB;
  constexpr int KS = 4 * E;
  const int lrow = lane >> 3, lch = lane & 7;
  const uint32_t g_base = (uint32_t)((int64_t)lrow * ldg * EB + lch * 16);
  const uint32_t g_half = (uint32_t)(8 * ldg * EB);
  const uint32_t g_tile = (uint32_t)(16 * ldg * EB);
  const int wslot = lrow * 8 + (lch ^ lrow);
  const int ri = lane & 15, rgrp = lane >> 4;
  const int rslot0 = ri * 8 + (rgrp ^ (ri & 7));
  const int rslot1 = ri * 8 + ((4 + rgrp) ^ (ri & 7));
  const uint32_t q_base = (uint32_t)(((int64_t)ri * ldq + E * rgrp) * EB);
  const uint32_t q_tile = (uint32_t)(16 * ldq * EB);

  i32x4 gbuf[SPD][2][2], qcur[2][QT], qnxt[2][QT];
  auto issue_g = [&](int grp, i32x4 (&gb)[2][2]) {
    const uint32_t off = g_base + (uint32_t)grp * 128u;
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) {
      gb[rt][0] = load16_stream(rg, off + rt * g_tile);
      gb[rt][1] = load16_stream(rg, off + rt * g_tile + g_half);
    }
  };
  auto issue_q = [&](int grp, i32x4 (&qf)[2][QT]) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int qt = 0; qt < QT; ++qt)
        qf[s][qt] = load16_cached(rq, q_base + qt * q_tile + (uint32_t)((2 * grp + s) * KS * EB));
  };
#pragma unroll
  for (int u = 0; u < SPD - 1; ++u)
    if (g_begin + u < g_end) issue_g(g_begin + u, gbuf[u]);
  issue_q(g_begin, qcur);

  for (int g0 = g_begin; g0 < g_end; g0 += SPD) {
#pragma unroll
    for (int u = 0; u < SPD; ++u) {
      const int grp = g0 + u;
      if (grp + SPD - 1 < g_end) issue_g(grp + SPD - 1, gbuf[(u + SPD - 1) % SPD]);
      if (grp < g_end) {
        if (grp + 1 < g_end) issue_q(grp + 1, qnxt);
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
          xp[rt * 128 + wslot] = gbuf[u][rt][0];
          xp[rt * 128 + 64 + wslot] = gbuf[u][rt][1];
        }
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
          const i32x4 f0 = xp[rt * 128 + rslot0];
          const i32x4 f1 = xp[rt * 128 + rslot1];
#pragma unroll
          for (int qt = 0; qt < QT; ++qt) {
            acc[qt][rt] = mma16(Tag{}, qcur[0][qt], f0, acc[qt][rt]);
            acc[qt][rt] = mma16(Tag{}, qcur[1][qt], f1, acc[qt][rt]);
          }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int qt = 0; qt < QT; ++qt) qcur[s][qt] = qnxt[s][qt];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// streaming plan (large stores)
// ---------------------------------------------------------------------------
// A workgroup owns 64 queries (16 per wave) and a contiguous partition of
// store rows, walked in tiles of 64 TR rows (TR = 1 or 2).  The tile
// sequence is cut into 128-byte K-groups ("stages"): for every stage the
// tile's store rows and the 64 query rows go straight from memory into a
// shared LDS ring by
// direct-to-LDS buffer loads (1 KB, line-coalesced instructions that land in
// the XOR-swizzled fragment layout), RING - 1 stages ahead.  No vector load
// feeds a register inside the loop, so the only waits are explicit: every
// stage costs each wave exactly LPW = 2 (TR + 1) load instructions, the wait
// for stage st is vmcnt <= LPW * (stages issued after st), then one barrier
// (all waves' loads landed; all waves finished the previous stage, whose
// slot is then refilled).
//
// Each wave computes its 16 queries (every fourth of the block) x the tile,
// so after a tile it holds every score of its own queries and needs no
// exchange.  Top-k selection is software-pipelined behind the stream: when
// a tile ends its scores move to a pending copy and are compared with the
// 16 running thresholds (k-th best so far, kept in registers); during the
// next tile's stages the wave walks its queries in order, a few per stage,
// and inserts the passing rows of each, in row order.  Each query's sorted
// list is held in registers (entry p in lane p % 64 of register p / 64,
// padded with (-inf, -1)); an insertion uses all 64 lanes at once (the
// position is the number of entries >= s: existing entries have lower row
// indices, so ties keep them first; the tail moves one lane up through a
// wave-wide DPP shift).  Register arrays need compile-time indices, so the
// query being served is always list 0 and the wave's list array rotates by
// one after each query (16 moves of one or two registers pairs): the
// selection code is one short loop body, not a per-query unrolled copy,
// and it stays in the instruction cache.
//
// Optionally each query starts from a floor: a lower bound on its k-th best
// score over the whole store.  Rows below the floor cannot be in the
// answer, so they never enter a list; without it every partition list fills
// with k rows and then takes ~k ln(rows / k) more insertions, which at 64
// queries and k = 100 cost more than the stream itself.  The bound is the
// k-th largest of the maxima of the first 16384 rows' 64-row segments (k
// distinct rows score at least that much), found by this kernel run with
// k = 1 over one-tile partitions and a per-query sort of the 256 maxima.
// A list then may end with fewer than k rows above the floor; the merge
// takes the global top k, all of which are at or above it.
// Partitions are mapped so that the query blocks sharing a partition run on
// the same XCD at the same time and share its L2.
constexpr int SR = 64;  // store rows per tile
constexpr int SQ = 64;  // queries per workgroup

template <int N>
__device__ inline void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// vmcnt <= n for a run-time n that is a multiple of L (n <= 6 L)
template <int L>
__device__ inline void wait_vmcnt_m(int n) {
  switch (n / L) {
    case 6: wait_vmcnt<6 * L>(); break;
    case 5: wait_vmcnt<5 * L>(); break;
    case 4: wait_vmcnt<4 * L>(); break;
    case 3: wait_vmcnt<3 * L>(); break;
    case 2: wait_vmcnt<2 * L>(); break;
    case 1: wait_vmcnt<L>(); break;
    default: wait_vmcnt<0>(); break;
  }
}

__device__ inline float sel4(const f32x4& a, int r) {
  float v = a[0];
  v = r == 1 ? a[1] : v;
  v = r == 2 ? a[2] : v;
  v = r == 3 ? a[3] : v;
  return v;
}

// lane l takes lane l - 1's value, lane 0 takes `fill` (DPP wave_shr:1)
__device__ inline int wave_shr1(int v, int fill) {
  return __builtin_amdgcn_update_dpp(fill, v, 0x138, 0xf, 0xf, false);
}

// Largest float below x (-inf for x = -inf or NaN): a strict ">" against it
// admits every score >= x.
__device__ inline float float_below(float x) {
  if (!(x > -__builtin_inff())) return -__builtin_inff();
  if (x == 0.f) return -__builtin_bit_cast(float, 1);  // -denorm_min
  const int b = __builtin_bit_cast(int, x);
  return __builtin_bit_cast(float, x > 0.f ? b - 1 : b + 1);  // +inf -> FLT_MAX
}

// Register-resident sorted list of one query: entry p in lane p % 64 of
// slot p / 64; positions >= k are don't-care.
template <int NS>
struct RegList {
  float s[NS];
  int i[NS];
  // kth entry's score
  __device__ inline float kth(int k) const {
    float t = s[0];
#pragma unroll
    for (int j = 1; j < NS; ++j) t = (k - 1) / 64 == j ? s[j] : t;
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, t), (k - 1) & 63));
  }
  // insert (v, idx): idx exceeds every row present, v > kth(k)
  __device__ inline void insert(float v, int idx, int k, int lane) {
    int pos = 0;
#pragma unroll
    for (int j = 0; j < NS; ++j)
      pos += __builtin_popcountll(__builtin_amdgcn_ballot_w64(64 * j + lane < k && s[j] >= v));
    float us[NS];
    int ui[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const int cs = j ? __builtin_amdgcn_readlane(__builtin_bit_cast(int, s[j - 1]), 63) : 0;
      const int ci = j ? __builtin_amdgcn_readlane(i[j - 1], 63) : 0;
      us[j] = __builtin_bit_cast(float, wave_shr1(__builtin_bit_cast(int, s[j]), cs));
      ui[j] = wave_shr1(i[j], ci);
    }
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const int p = 64 * j + lane;
      s[j] = p < pos ? s[j] : (p == pos ? v : us[j]);
      i[j] = p < pos ? i[j] : (p == pos ? idx : ui[j]);
    }
  }
};

// At least two waves per SIMD (two workgroups per CU): the compiler keeps
// every configuration within 256 VGPRs (64 queries with two-register lists
// and 128-row tiles would otherwise take 268 and run one workgroup per CU).
template <bool F16, int KMAX, int RING, int GPS, int QPW, int TR>
__global__ __launch_bounds__(256, 2) void score_stream_kernel(
    const char* __restrict__ Q, int64_t n_q, int64_t ldq, const char* __restrict__ G,
    int64_t n_g, int64_t ldg, int n_grp, int k, int64_t rows_per_part, int n_parts, int n_qb,
    const float* __restrict__ bound, float* __restrict__ part_s, int64_t* __restrict__ part_i,
    int64_t index_base) {
  // GPS 128-byte K-groups per stage: a stage row is RB bytes (CPR chunks),
  // RPI rows per 1 KB load; tiles of SRT = 64 TR store rows; LPW loads per
  // wave and stage (16 TR store rows and 16 query rows)
  constexpr int SRT = SR * TR;
  constexpr int RB = 128 * GPS, CPR = 8 * GPS, RPI = 8 / GPS, LPW = 2 * GPS * (TR + 1);
  static_assert(RING >= 3 && RING - 2 <= 6, "wait_vmcnt_m range");
  static_assert(TR == 1 || TR == 2, "candidate bits: 4 TR row tiles x 4 queries");
  using Tag = typename STag<F16>::tag;
  constexpr int EB = STag<F16>::bytes;
  constexpr int NS = (KMAX + 63) / 64;
  __shared__ i32x4 ring[RING][(SRT + SQ) * CPR];  // store rows, then query rows

  const uint32_t b = blockIdx.x;
  const int xcd = (int)(b & 7u);
  const uint32_t jb = b >> 3;
  const int qb = (int)(jb % (uint32_t)n_qb);
  const int p = (int)(jb / (uint32_t)n_qb) * 8 + xcd;
  if (p >= n_parts) return;  // uniform
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;

  const int64_t q0 = (int64_t)qb * SQ;
  int64_t nq_blk = n_q - q0;
  nq_blk = nq_blk > SQ ? SQ : nq_blk;
  // wave w holds block queries w, w + 4, ..., w + 60 (slot j = query 4 j + w), so
  // that a partial block spreads its selection work over all four waves
  int nq_w = (int)((nq_blk - wave + 3) / 4);
  nq_w = nq_w < 0 ? 0 : (nq_w > QPW ? QPW : nq_w);  // the host sizes QPW to the block
  // a store read by a single query block is not kept in L2
  const bool g_nt = n_qb == 1;

  const int64_t r_begin = (int64_t)p * rows_per_part;
  int64_t r_end = r_begin + rows_per_part;
  r_end = r_end > n_g ? n_g : r_end;
  const int64_t nrows = r_end > r_begin ? r_end - r_begin : 0;
  const int n_tiles = (int)((nrows + SRT - 1) / SRT);
  const int n_stg = n_grp / GPS;  // stages per tile (n_grp is a multiple of GPS)
  const int total = n_tiles * n_stg;
  const int spg = (QPW + n_stg - 1) / n_stg;  // selection steps per stage

  // the wave's QPW sorted lists, in registers; the list of the query being
  // selected is always lists[0]: the array rotates by one after every step
  RegList<NS> lists[QPW];
#pragma unroll
  for (int ql = 0; ql < QPW; ++ql)
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      lists[ql].s[j] = -__builtin_inff();
      lists[ql].i[j] = -1;
    }
  auto rotate = [&]() {
    const RegList<NS> t = lists[0];
#pragma unroll
    for (int ql = 0; ql + 1 < QPW; ++ql) lists[ql] = lists[ql + 1];
    lists[QPW - 1] = t;
  };

  const i32x4 dq = make_desc(Q + q0 * ldq * EB, (uint32_t)(nq_blk * ldq * EB));
  // load lane -> row lr of the instruction's RPI rows, LDS slot lane % CPR of
  // that row, which holds chunk (lane % CPR) ^ (row % 8)
  const int lr = lane / CPR;
  const int ri = lane & 15, rgrp = lane >> 4;
  const uint32_t ring_base = (uint32_t)(uintptr_t)&ring[0][0];
  constexpr uint32_t SLOT_BYTES = (SRT + SQ) * RB;
  // per-lane byte offsets of this wave's 16 TR store rows / 16 query rows in
  // groups of RPI rows (stage 0); query slot j is block query 4 j + wave
  uint32_t goff[2 * GPS * TR], qoff[2 * GPS];
#pragma unroll
  for (int h = 0; h < 2 * GPS * TR; ++h) {
    const int lc = (lane % CPR) ^ ((RPI * h + lr) & 7);  // LDS rows 16 TR wave + RPI h + lr
    goff[h] = (uint32_t)((int64_t)(16 * TR * wave + RPI * h + lr) * ldg * EB + lc * 16);
  }
#pragma unroll
  for (int h = 0; h < 2 * GPS; ++h) {
    const int lc = (lane % CPR) ^ ((RPI * h + lr) & 7);  // LDS rows SRT + 16 wave + RPI h + lr
    qoff[h] = (uint32_t)((int64_t)(4 * (RPI * h + lr) + wave) * ldq * EB + lc * 16);
  }
  const uint32_t lds_g = ring_base + (uint32_t)(16 * TR * wave) * RB;
  const uint32_t lds_q = ring_base + (uint32_t)(SRT + 16 * wave) * RB;

  // issue cursor: next stage to load is (it_tile, it_g) into slot islot
  int it_tile = 0, it_g = 0, issued = 0, islot = 0;
  i32x4 dt{0, 0, 0, 0};
  auto tile_desc = [&](int tile) {
    const int64_t row0 = r_begin + (int64_t)tile * SRT;
    int64_t nr = r_end - row0;
    nr = nr > SRT ? SRT : nr;
    dt = make_desc(G + row0 * ldg * EB, (uint32_t)(nr * ldg * EB));
  };
  auto issue_next = [&]() {
    const uint32_t sb = (uint32_t)islot * SLOT_BYTES;
    const uint32_t go = (uint32_t)it_g * RB;
    if (g_nt) {
#pragma unroll
      for (int h = 0; h < 2 * GPS * TR; ++h) lds_dma16_nt(dt, goff[h] + go, lds_g + sb + 1024u * h);
    } else {
#pragma unroll
      for (int h = 0; h < 2 * GPS * TR; ++h) lds_dma16(dt, goff[h] + go, lds_g + sb + 1024u * h);
    }
#pragma unroll
    for (int h = 0; h < 2 * GPS; ++h) lds_dma16(dq, qoff[h] + go, lds_q + sb + 1024u * h);
    ++issued;
    islot = islot == RING - 1 ? 0 : islot + 1;
    if (++it_g == n_stg) {
      it_g = 0;
      ++it_tile;
      if (it_tile < n_tiles) tile_desc(it_tile);
    }
  };

  if (total > 0) tile_desc(0);
#pragma unroll
  for (int u = 0; u < RING - 1; ++u)
    if (issued < total) issue_next();

  // floor4: per query, the largest float below a lower bound on its k-th
  // best score over the whole store (rows below it cannot be in the answer),
  // else -inf; running thresholds thr4 start there.  Lane l of thr4[r] and
  // floor4[r] holds slot 4 (l / 16) + r.
  f32x4 floor4 = f32x4{-__builtin_inff(), -__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
  if (bound) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int ql = 4 * rgrp + r;
      if (ql < nq_w) floor4[r] = float_below(bound[q0 + 4 * ql + wave]);
    }
  }
  f32x4 thr4 = floor4;
  // pending tile: scores (pend[rt][r] in lane l: query 4 (l / 16) + r, row
  // 16 rt + l % 16), candidate bits cm (bit 4 rt + r) and its first row
  f32x4 pend[4 * TR];
  uint32_t cm = 0;
  bool pend_any = false;
  int pend_rbase = 0;

  auto process_query = [&](int ql, RegList<NS>& L) {
    const int r = ql & 3, grp = ql >> 2;
    uint64_t m[4 * TR];
    bool has = false;
#pragma unroll
    for (int rt = 0; rt < 4 * TR; ++rt) {
      m[rt] = __builtin_amdgcn_ballot_w64(rgrp == grp && ((cm >> (4 * rt + r)) & 1u));
      has |= m[rt] != 0;
    }
    if (!has) return;
    float thr = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, sel4(thr4, r)), 16 * grp));
    const float flo = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, sel4(floor4, r)), 16 * grp));
#pragma unroll
    for (int rt = 0; rt < 4 * TR; ++rt) {
      const float v = sel4(pend[rt], r);
      uint64_t mm = m[rt];
      while (mm) {
        const int src = __builtin_ctzll(mm);
        mm &= mm - 1;
        const float cv = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), src));
        if (cv > thr) {
          L.insert(cv, pend_rbase + 16 * rt + (src & 15), k, lane);
          thr = fmaxf(L.kth(k), flo);
        }
      }
    }
    const bool mine = rgrp == grp;
    thr4[0] = mine && r == 0 ? thr : thr4[0];
    thr4[1] = mine && r == 1 ? thr : thr4[1];
    thr4[2] = mine && r == 2 ? thr : thr4[2];
    thr4[3] = mine && r == 3 ? thr : thr4[3];
  };

  int st = 0, cslot = 0;
  for (int tile = 0; tile < n_tiles; ++tile) {
    f32x4 acc[4 * TR];
#pragma unroll
    for (int rt = 0; rt < 4 * TR; ++rt) acc[rt] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int g = 0; g < n_stg; ++g, ++st) {
      // stage st landed: at most (loads issued after it) of this wave's
      // loads are still outstanding
      const int after = total - 1 - st;
      if (after >= RING - 2) {
        wait_vmcnt<LPW * (RING - 2)>();
      } else {
        wait_vmcnt_m<LPW>(LPW * after);
      }
      // this wave's LDS reads of the previous stage are complete before
      // anyone refills that slot
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      if (issued < total) issue_next();
      const i32x4* sl = ring[cslot];
      cslot = cslot == RING - 1 ? 0 : cslot + 1;
#pragma unroll
      for (int s2 = 0; s2 < 2 * GPS; ++s2) {
        const int qrow = SRT + 16 * wave + ri;
        const i32x4 qf = sl[qrow * CPR + ((4 * s2 + rgrp) ^ (qrow & 7))];
#pragma unroll
        for (int rt = 0; rt < 4 * TR; ++rt) {
          const int grow = 16 * rt + ri;
          const i32x4 gf = sl[grow * CPR + ((4 * s2 + rgrp) ^ (grow & 7))];
          acc[rt] = mma16(Tag{}, qf, gf, acc[rt]);
        }
      }
      // previous tile's selection, spread over this tile's stages
      // steps [g c, (g + 1) c) of the QPW, in order, c = ceil(QPW / n_stg)
      if (pend_any)
        for (int ql = g * spg; ql < QPW && ql < (g + 1) * spg; ++ql) {
          if (ql < nq_w) process_query(ql, lists[0]);
          rotate();
        }
    }
    // hand this tile over to the selection
    const int rbase = tile * SRT;
    const int nvalid = (int)(nrows - rbase > SRT ? SRT : nrows - rbase);
    cm = 0;
#pragma unroll
    for (int rt = 0; rt < 4 * TR; ++rt) {
      pend[rt] = acc[rt];
#pragma unroll
      for (int r = 0; r < 4; ++r)
        cm |= (4 * rgrp + r < nq_w && 16 * rt + ri < nvalid && acc[rt][r] > thr4[r]) ? 1u << (4 * rt + r) : 0u;
    }
    pend_any = __builtin_amdgcn_ballot_w64(cm != 0) != 0;
    pend_rbase = rbase;
  }
  if (pend_any)
    for (int ql = 0; ql < QPW; ++ql) {
      if (ql < nq_w) process_query(ql, lists[0]);
      rotate();
    }
#pragma unroll
  for (int ql = 0; ql < QPW; ++ql) {
    if (ql >= nq_w) continue;
    const int64_t q = q0 + 4 * ql + wave;
    float* ds = part_s + (q * n_parts + p) * (int64_t)k;
    int64_t* di = part_i + (q * n_parts + p) * (int64_t)k;
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const int pos = 64 * j + lane;
      if (pos < k) {
        const int idx = lists[ql].i[j];
        ds[pos] = lists[ql].s[j];
        di[pos] = idx >= 0 ? index_base + r_begin + idx : -1;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// GEMM plan (many queries: the scan is bound by the matrix cores)
// ---------------------------------------------------------------------------
// The store is taken in chunks of rows.  For each chunk the 256 x 256 block
// GEMM core computes the fp32 score matrix S[q][r] into the workspace (sized
// to stay in the MALL), then one workgroup per query selects that chunk's
// top k exactly:
//  * a strided sample of RS_SMP scores is sorted; the sample at a rank
//    chosen so that ~2k + 256 scores are expected above it is a threshold tau;
//  * one pass collects the scores >= tau into LDS (counting them all); if
//    there are at least k of them the top k are all among them (the k-th
//    best is >= tau), and if at most RS_CAP a bitonic sort orders them by
//    (score desc, index asc) and the first k are the chunk's list;
//  * otherwise tau moves by bisection over the sample ranks (more passes);
//    if no rank works (a chunk of massive ties or one ordered against the
//    sample), k arg-max passes over the chunk give the same list exactly.
// Chunks of at most 4096 rows are sorted whole.  NaN and -inf scores are
// never selected; lists are padded with (-inf, -1).  Chunk lists are merged
// by the common merge kernel.
constexpr int RS_CAP = 2048;  // candidates sorted per (query, chunk)
constexpr int RS_SMP = 1024;  // threshold samples
constexpr int RS_SEG = 64;    // chunk rows per score segment (one maximum each)
constexpr int64_t RS_MAXCHUNK = 262144;  // rows of the largest chunk (its segment tables sit in LDS)
constexpr int RS_MAXSEG = (int)(RS_MAXCHUNK / RS_SEG);  // segments of the largest chunk

// v of another lane of the same row of 16 (DPP control C, full masks)
template <int C>
__device__ inline float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), C, 0xf, 0xf, false));
}

// Epilogue of a score tile.  A wave's columns are 64-row segments of the
// chunk (accumulator column blocks 4 g .. 4 g + 3 form segment g); the 16
// lanes that share a query row reduce each segment's maximum, which is
// stored for the selection.  With a bound from earlier chunks (running k-th
// best score of the query), a segment whose maximum is below it cannot
// contribute and is not written.  bound(row) gives the bound of the tile's
// query row.
template <typename Core, typename Bound>
__device__ inline void score_tile_store(const Core& core, int64_t q0, int64_t nq, int64_t c0,
                                        int64_t nr, float* __restrict__ S, int64_t lds,
                                        float* __restrict__ segmax, int64_t n_seg, Bound bound) {
  constexpr int NJ = Core::NJ, NG = NJ / 4;
  const int lane = threadIdx.x & 63;
  const int64_t seg0 = c0 / RS_SEG + Core::col_base() / RS_SEG;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = Core::row_of(i, r);
      float m[NG];
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        float v = -__builtin_inff();
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
          if (Core::col_of(4 * g + jj) < nr) v = fmaxf(v, core.acc[i][4 * g + jj][r]);
        // rotations within each row of 16 lanes (DPP row_ror 8, 4, 2, 1)
        v = fmaxf(v, dpp_f<0x128>(v));
        v = fmaxf(v, dpp_f<0x124>(v));
        v = fmaxf(v, dpp_f<0x122>(v));
        v = fmaxf(v, dpp_f<0x121>(v));
        m[g] = v;
      }
      if (row < nq) {
        const float b = bound(row);
        if ((lane & 15) == 0) {
#pragma unroll
          for (int g = 0; g < NG; ++g) segmax[(q0 + row) * n_seg + seg0 + g] = m[g];
        }
        float* dst = S + (q0 + row) * lds + c0;
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int col = Core::col_of(j);
          if (col < nr && !(m[j >> 2] < b)) dst[col] = core.acc[i][j][r];
        }
      }
    }
}

// Scores of one chunk of store rows: items are (query tile, row tile) pairs.
// XCD x (workgroup b goes to XCD b % 8) takes a contiguous range of items,
// query tile fastest: the query tiles of one row tile read the same store
// rows through the same L2.  NT (a single query tile): every store row is
// read once, with the non-temporal cache policy.
template <typename Tag, bool NT>
__global__ __launch_bounds__(256) void score_gemm_kernel(
    const _Float16* __restrict__ Q, int64_t n_q, int64_t ldq, const _Float16* __restrict__ G,
    int64_t nc, int64_t ldg, int n_qt, int n_items, int per_xcd, int n_st,
    float* __restrict__ S, int64_t lds, float* __restrict__ segmax, int64_t n_seg,
    const float* __restrict__ thr, int use_bound) {
  __shared__ GemmSmem sm;
  const int item = (int)(blockIdx.x & 7u) * per_xcd + (int)(blockIdx.x >> 3);
  if (item >= n_items) return;  // uniform
  const int qt = item % n_qt, rt = item / n_qt;
  const int64_t q0 = (int64_t)qt * GT, c0 = (int64_t)rt * GT;
  int64_t nq = n_q - q0, nr = nc - c0;
  nq = nq > GT ? GT : nq;
  nr = nr > GT ? GT : nr;
  const i32x4 dq = make_desc(Q + q0 * ldq, (uint32_t)(nq * ldq * 2));
  const i32x4 dg = make_desc(G + c0 * ldg, (uint32_t)(nr * ldg * 2));
  // the tile's query bounds, staged in LDS (the main loop's barriers publish them)
  __shared__ float tb[GT];
  tb[threadIdx.x] = use_bound && q0 + threadIdx.x < n_q ? thr[q0 + threadIdx.x] : -__builtin_inff();
  GemmCore<Tag, NT> core;
  core.zero();
  core.run(sm, dq, ldq, dg, ldg, n_st);
  score_tile_store(core, q0, nq, c0, nr, S, lds, segmax, n_seg, [&](int row) { return tb[row]; });
}

// The same with 128-query x 256-row tiles on the three-slot ring
// (GemmCoreR): for query counts whose last 256-query tile would be at most
// half used.
template <typename Tag, bool NT>
__global__ __launch_bounds__(256) void score_gemm_r_kernel(
    const _Float16* __restrict__ Q, int64_t n_q, int64_t ldq, const _Float16* __restrict__ G,
    int64_t nc, int64_t ldg, int n_qt, int n_items, int per_xcd, int n_st,
    float* __restrict__ S, int64_t lds, float* __restrict__ segmax, int64_t n_seg,
    const float* __restrict__ thr, int use_bound) {
  __shared__ GemmSmemR sm;
  const int item = (int)(blockIdx.x & 7u) * per_xcd + (int)(blockIdx.x >> 3);
  if (item >= n_items) return;  // uniform
  const int qt = item % n_qt, rt = item / n_qt;
  const int64_t q0 = (int64_t)qt * GRQ, c0 = (int64_t)rt * GRR;
  int64_t nq = n_q - q0, nr = nc - c0;
  nq = nq > GRQ ? GRQ : nq;
  nr = nr > GRR ? GRR : nr;
  // this wave's 64 store rows
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  int64_t nw = nr - 64 * wave;
  nw = nw < 0 ? 0 : (nw > 64 ? 64 : nw);
  const i32x4 dq = make_desc(Q + q0 * ldq, (uint32_t)(nq * ldq * 2));
  const i32x4 dg = make_desc(G + (c0 + 64 * wave) * ldg, (uint32_t)(nw * ldg * 2));
  // the tile's query bounds, staged in LDS (the ring's barriers publish them)
  __shared__ float tb[GRQ];
  if (threadIdx.x < GRQ)
    tb[threadIdx.x] = use_bound && q0 + threadIdx.x < n_q ? thr[q0 + threadIdx.x] : -__builtin_inff();
  GemmCoreR<Tag, NT> core;
  core.zero();
  core.run(sm, dq, ldq, dg, ldg, n_st);
  score_tile_store(core, q0, nq, c0, nr, S, lds, segmax, n_seg, [&](int row) { return tb[row]; });
}

// Order-preserving key of a float (larger float, larger key).  Selectable
// scores are those above -inf and not NaN: keys in (fkey(-inf), fkey(+inf)].
__device__ inline uint32_t fkey(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ inline float fkey_inv(uint32_t key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}
__device__ inline bool selectable(uint32_t key) { return key > 0x007fffffu && key <= 0xff800000u; }
// (score desc, index asc) as one descending 64-bit key; 0 is padding
__device__ inline uint64_t rs_key(uint32_t key, int64_t j) {
  return ((uint64_t)key << 32) | (uint64_t)(0xffffffffu - (uint32_t)j);
}

// A threshold at or below the k-th largest of the block's keys (key(v), v < V, per
// thread; 0 = none; below 2^bits) that at least k keys reach: exactly that key, or,
// with slack, the first threshold found that at most k + slack keys reach.  reach:
// how many do.  0 (and reach 0) when fewer than k keys are there.  Two bits a step
// from the top, counted by ballots: 16 steps of one barrier each for 32 bits, where
// a bitonic sort of 1024 keys takes 55 (k-th of the 256 prefix maxima of a query:
// 21 -> 5 us).  cnt: 48 counters in LDS.
template <int V, typename F>
__device__ inline uint32_t block_kth(F&& key, int k, int slack, int* cnt, int& reach, int bits = 32) {
  const int t = threadIdx.x;
  __syncthreads();  // the counters' last readers are done
  if (t < 48) cnt[t] = 0;
  __syncthreads();
  uint32_t T = 0u;
  reach = 0;
  const int steps = (bits + 1) / 2;
  for (int it = 0; it < steps; ++it) {
    const int sh = 2 * (steps - 1 - it);
    int n[3] = {0, 0, 0};
#pragma unroll
    for (int v = 0; v < V; ++v)
#pragma unroll
      for (uint32_t b = 1; b <= 3; ++b)
        n[b - 1] += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key(v) >= (T | (b << sh))));
    if ((t & 63) == 0) {
#pragma unroll
      for (int b = 0; b < 3; ++b)
        if (n[b]) atomicAdd(&cnt[3 * it + b], n[b]);
    }
    __syncthreads();
    int have = 0;
#pragma unroll
    for (int b = 2; b >= 0; --b)
      if (have == 0 && cnt[3 * it + b] >= k) {
        have = cnt[3 * it + b];
        T |= (uint32_t)(b + 1) << sh;
      }
    reach = have ? have : reach;
    if (slack && have && have <= k + slack) break;  // uniform
  }
  return T;
}

// The block's sum of per-wave counts (n: uniform over the wave).
__device__ inline int block_total(int n, int* cnt) {
  __syncthreads();
  if (threadIdx.x == 0) cnt[0] = 0;
  __syncthreads();
  if ((threadIdx.x & 63) == 0 && n) atomicAdd(cnt, n);
  __syncthreads();
  return cnt[0];
}

// Descending bitonic sort of n (a power of two) keys in LDS, 256 threads.
template <typename T>
__device__ inline void bitonic_desc(T* a, int n) {
  for (int size = 2; size <= n; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      __syncthreads();
      for (int t = threadIdx.x; t < n / 2; t += 256) {
        const int i = 2 * t - (t & (stride - 1));
        const int j = i + stride;
        const T x = a[i], y = a[j];
        const bool down = (i & size) == 0;
        if (down ? (x < y) : (x > y)) {
          a[i] = y;
          a[j] = x;
        }
      }
    }
  __syncthreads();
}

__device__ inline uint64_t block_max_u64(uint64_t v, uint64_t* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, off, kWave);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), off, kWave);
    const uint64_t o = ((uint64_t)hi << 32) | lo;
    v = o > v ? o : v;
  }
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  uint64_t m = red[0];
#pragma unroll
  for (int w = 1; w < 4; ++w) m = red[w] > m ? red[w] : m;
  return m;
}

__global__ __launch_bounds__(256) void score_rselect_kernel(
    const float* __restrict__ S, int64_t lds, const float* __restrict__ segmax, int64_t n_seg,
    float* __restrict__ thr, int64_t nc, int k, int part, int n_parts, int64_t index_base,
    float* __restrict__ part_s, int64_t* __restrict__ part_i) {
  __shared__ uint64_t cand[RS_CAP];
  __shared__ uint32_t smp[RS_SMP];  // samples, sorted
  __shared__ int kcnt[48];
  __shared__ uint16_t segs[RS_MAXSEG];
  __shared__ uint64_t red_u[4];
  __shared__ int n_cand, n_pass;
  const int64_t q = blockIdx.x;
  const int t = threadIdx.x;
  const float* s = S + q * lds;
  const float* sm = segmax + q * n_seg;
  const int n_sc = (int)((nc + RS_SEG - 1) / RS_SEG);
  float* ds = part_s + (q * n_parts + part) * (int64_t)k;
  int64_t* di = part_i + (q * n_parts + part) * (int64_t)k;

  // Bound from this call's earlier chunks, all of lower index: the running
  // maximum of their k-th scores has k entries at or above it that precede
  // every row of this chunk, so only scores strictly above it can still
  // enter the top k.  Segments whose maximum is below it were not written.
  const float bnd = part > 0 ? thr[q] : -__builtin_inff();
  const uint32_t bkey = fkey(bnd);
  const bool has_b = part > 0 && selectable(bkey);
  const uint32_t floor_key = has_b ? bkey + 1u : 0x00800000u;
  const float floor_f = fkey_inv(floor_key);  // NaN when the bound is +inf: nothing passes

  // collect every selectable score >= tau (up to RS_CAP of them), reading
  // only the segments whose maximum reaches tau; returns how many there are
  auto take = [&](float v, int64_t j, uint32_t tau) {
    const uint32_t key = fkey(v);
    if (selectable(key) && key >= tau) {
      const int p = atomicAdd(&n_cand, 1);
      if (p < RS_CAP) cand[p] = rs_key(key, j);
    }
  };
  auto collect = [&](uint32_t tau) -> int {
    const float tau_f = fkey_inv(tau);  // the float whose key is tau
    __syncthreads();
    if (t == 0) {
      n_cand = 0;
      n_pass = 0;
    }
    __syncthreads();
    for (int g = t; g < n_sc; g += 256)
      if (sm[g] >= tau_f) segs[atomicAdd(&n_pass, 1)] = (uint16_t)g;
    __syncthreads();
    const int np = n_pass;
    // 16 threads per segment (16 bytes each), SB segments per group in flight
    constexpr int SB = 4;
    const int grp = t >> 4, l16 = t & 15;
    const f32x4* s4 = reinterpret_cast<const f32x4*>(s);  // rows are 1 KB aligned
    for (int e0 = 0; e0 < np; e0 += 16 * SB) {
      f32x4 v[SB];
      int64_t j0[SB];
#pragma unroll
      for (int u = 0; u < SB; ++u) {
        const int e = e0 + 16 * u + grp;
        j0[u] = e < np ? (int64_t)segs[e] * RS_SEG + 4 * l16 : -1;
        // a segment's 64 columns lie inside the row (lds is a multiple of 256)
        v[u] = j0[u] >= 0 ? s4[j0[u] >> 2]
                          : f32x4{-__builtin_inff(), -__builtin_inff(), -__builtin_inff(),
                                  -__builtin_inff()};
      }
#pragma unroll
      for (int u = 0; u < SB; ++u) {
        const float m = fmaxf(fmaxf(v[u][0], v[u][1]), fmaxf(v[u][2], v[u][3]));
        if (j0[u] >= 0 && m >= tau_f) {
#pragma unroll
          for (int e4 = 0; e4 < 4; ++e4)
            if (j0[u] + e4 < nc) take(v[u][e4], j0[u] + e4, tau);
        }
      }
    }
    __syncthreads();
    return n_cand;
  };

  bool ok = false;
  int c = 0;
  if (nc <= RS_CAP || has_b) {
    c = collect(floor_key);  // everything above the bound
    ok = c <= RS_CAP;        // fewer than k entries is allowed
  } else {
    // No bound yet: a threshold that at least k and, where they differ, at most k + 8
    // of the segment maxima reach, so at least k scores do; unless one segment holds many of the top
    // scores, few more than k do.
    // (Ballots over as many maxima per thread as the chunk has, down to a threshold
    // that few more reach: 300 queries, 9000 x 2048, k = 1, the whole call 48 us; 62
    // with ballots over 4096 places down to the k-th itself, 54 with a sort.)
    auto kth_max = [&](auto per_thread) {
      constexpr int V = decltype(per_thread)::value;
      uint32_t key[V];
#pragma unroll
      for (int u = 0; u < V; ++u) {
        const int g = t + 256 * u;
        const uint32_t x = g < n_sc ? fkey(sm[g]) : 0u;
        key[u] = selectable(x) ? x : 0u;
      }
      int reach;
      return block_kth<V>([&](int u) { return key[u]; }, k, 8, kcnt, reach);
    };
    const uint32_t kth = n_sc <= 256    ? kth_max(std::integral_constant<int, 1>{})
                         : n_sc <= 1024 ? kth_max(std::integral_constant<int, 4>{})
                                        : kth_max(std::integral_constant<int, RS_MAXSEG / 256>{});
    const uint32_t tau = kth ? kth : floor_key;
    c = collect(tau);
    ok = c <= RS_CAP;
  }
  if (!ok) {
    {
      uint32_t v[RS_SMP / 256];
#pragma unroll
      for (int u = 0; u < RS_SMP / 256; ++u) {
        const int64_t j = (int64_t)(u * 256 + t) * nc / RS_SMP;
        const bool written = !has_b || sm[j / RS_SEG] >= floor_f;
        const uint32_t key = written ? fkey(s[j]) : 0u;
        v[u] = selectable(key) && key >= floor_key ? key : 0u;
      }
#pragma unroll
      for (int u = 0; u < RS_SMP / 256; ++u) smp[u * 256 + t] = v[u];
    }
    bitonic_desc(smp, RS_SMP);
    int lo = 0, hi = RS_SMP - 1;
    int rho = (int)(((int64_t)(2 * k + 256) * RS_SMP + nc - 1) / nc) - 1;
    rho = rho < 0 ? 0 : (rho > hi ? hi : rho);
    while (lo <= hi) {
      const uint32_t tau = smp[rho];
      if (tau == 0u) {  // fewer selectable samples than rho + 1
        hi = rho - 1;
      } else {
        c = collect(tau);
        if (c >= k && c <= RS_CAP) {
          ok = true;
          break;
        }
        if (c < k) lo = rho + 1;
        else hi = rho - 1;
      }
      rho = (lo + hi) / 2;
    }
  }
  float kth = -__builtin_inff();
  if (ok) {
    int n_sort = 64;  // power of two >= max(c, k)
    while (n_sort < c || n_sort < k) n_sort <<= 1;
    for (int j = c + t; j < n_sort; j += 256) cand[j] = 0ull;
    bitonic_desc(cand, n_sort);
    for (int j = t; j < k; j += 256) {
      const uint64_t e = cand[j];
      ds[j] = e ? fkey_inv((uint32_t)(e >> 32)) : -__builtin_inff();
      di[j] = e ? index_base + (int64_t)(0xffffffffu - (uint32_t)e) : -1;
    }
    const uint64_t e = cand[k - 1];
    kth = e ? fkey_inv((uint32_t)(e >> 32)) : -__builtin_inff();
  } else {
    // exact: the r-th entry is the largest key (above the floor) below the
    // (r-1)-th
    uint64_t prev = ~0ull;
    for (int r = 0; r < k; ++r) {
      uint64_t best = 0ull;
      if (prev != 0ull)
        for (int64_t j = t; j < nc; j += 256) {
          if (has_b && !(sm[j / RS_SEG] >= floor_f)) continue;  // not written
          const uint32_t key = fkey(s[j]);
          if (selectable(key) && key >= floor_key) {
            const uint64_t e = rs_key(key, j);
            if (e < prev && e > best) best = e;
          }
        }
      best = block_max_u64(best, red_u);
      if (t == 0) {
        ds[r] = best ? fkey_inv((uint32_t)(best >> 32)) : -__builtin_inff();
        di[r] = best ? index_base + (int64_t)(0xffffffffu - (uint32_t)best) : -1;
      }
      if (r == k - 1 && best) kth = fkey_inv((uint32_t)(best >> 32));
      prev = best;
    }
  }
  // running bound for the next chunk (its GEMM skips segments below it)
  if (t == 0) thr[q] = has_b && bnd > kth ? bnd : kth;
}

// ---------------------------------------------------------------------------
// split-K plan
// ---------------------------------------------------------------------------
// Partial scores of (query block, row tile, D-slice) -> spart[slice][q][row]
// (nqp = 64 n_qb query rows of n_g scores per slice).
template <bool F16, int QT>
__global__ __launch_bounds__(256) void score_splitk_kernel(
    const char* __restrict__ Q, int64_t n_q, int64_t ldq, const char* __restrict__ G,
    int64_t n_g, int64_t ldg, int n_grp, int n_qb, int n_tiles, int n_split,
    float* __restrict__ spart) {
  const int64_t nqp = (int64_t)n_qb * SQB;
  constexpr int EB = STag<F16>::bytes;
  __shared__ i32x4 xpose[4][2 * 128];
  uint32_t b = blockIdx.x;
  const int qb = (int)(b % (uint32_t)n_qb);
  b /= (uint32_t)n_qb;
  const int tile = (int)(b % (uint32_t)n_tiles);
  const int split = (int)(b / (uint32_t)n_tiles);
  const int g_begin = (int)((int64_t)n_grp * split / n_split);
  const int g_end = (int)((int64_t)n_grp * (split + 1) / n_split);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int lane = threadIdx.x & 63;
  const int64_t q0 = (int64_t)qb * SQB;
  int64_t nq_blk = n_q - q0;
  nq_blk = nq_blk > SQB ? SQB : nq_blk;
  const __amdgpu_buffer_rsrc_t rq = make_rsrc(Q + q0 * ldq * EB, (uint32_t)(nq_blk * ldq * EB));
  const int64_t r0 = (int64_t)tile * STN + 32 * wave;
  int64_t nrow = n_g - r0;
  nrow = nrow < 0 ? 0 : (nrow > 32 ? 32 : nrow);
  const __amdgpu_buffer_rsrc_t rg = make_rsrc(G + r0 * ldg * EB, (uint32_t)(nrow * ldg * EB));
  f32x4 acc[QT][2];
#pragma unroll
  for (int qt = 0; qt < QT; ++qt)
#pragma unroll
    for (int rt = 0; rt < 2; ++rt) acc[qt][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
  score_tile<F16, QT>(rq, ldq, rg, ldg, g_begin, g_end, lane, &xpose[wave][0], acc);
  float* dst = spart + (int64_t)split * n_g * nqp;
#pragma unroll
  for (int qt = 0; qt < QT; ++qt)
#pragma unroll
    for (int rt = 0; rt < 2; ++rt)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t q = q0 + 16 * qt + 4 * (lane >> 4) + r;
        const int64_t row = r0 + 16 * rt + (lane & 15);
        if (row < n_g && q < n_q) dst[q * n_g + row] = acc[qt][rt][r];
      }
}

// ---------------------------------------------------------------------------
// merge
// ---------------------------------------------------------------------------
struct Cand {
  float s;
  int64_t i;
};

__device__ inline Cand cand_none() { return Cand{-__builtin_inff(), -1}; }

__device__ inline bool better(const Cand& a, const Cand& b) {
  if (a.i < 0) return false;
  if (b.i < 0) return true;
  return a.s > b.s || (a.s == b.s && a.i < b.i);
}

__device__ inline Cand wave_best(Cand c) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    Cand o;
    o.s = __shfl_xor(c.s, off, kWave);
    o.i = __shfl_xor(c.i, off, kWave);
    if (better(o, c)) c = o;
  }
  return c;
}


// Split-K plan with at most 256 store rows (a batch of new rows scored and
// merged into a running list) and k <= 8, or 12 for 16 rows: one wave per query sums
// the slices of its scores in slice order and takes the k best of those rows and
// of the previous list (merge) by k rounds of wave arg-max, writing the list in
// place.  Replaces the partition select and the merge launches.  A round takes
// 0.6 to 1.2 us; for larger k the threshold and the sort of the kernel below, ~10 us
// whatever k, are faster (16 queries, rounds / threshold, the whole call: 256 x 1024 k
// = 8 17 / 15, k = 100 112 / 19; 40 x 256 13 / 12, 78 / 22; one row of 64 10 / 14, k =
// 12 12 / 14, k = 100 64 / 18).
inline bool small_select(int64_t n_g, int k) { return n_g <= 256 && k <= (n_g <= 16 ? 12 : 8); }
__global__ __launch_bounds__(64) void score_small_select_kernel(
    const float* __restrict__ spart, int64_t nqp, int64_t n_g, int n_split, int k, int merge,
    int64_t index_base, float* top_s, int64_t* top_i) {
  const int64_t q = blockIdx.x;
  const int lane = threadIdx.x;
  const int64_t plane = n_g * nqp;
  Cand c[6];
  // rows lane + 64 m; slices summed in order, 8 slices of all four rows in
  // flight at once
  float acc[4];
  bool live[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    live[m] = lane + 64 * m < n_g;
    acc[m] = live[m] ? spart[q * n_g + lane + 64 * m] : 0.f;
  }
  int sp = 1;
  for (; sp + 8 <= n_split; sp += 8) {
    float x[4][8];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int u = 0; u < 8; ++u)
        x[m][u] = live[m] ? spart[(sp + u) * plane + q * n_g + lane + 64 * m] : 0.f;
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
      for (int u = 0; u < 8; ++u) acc[m] += x[m][u];
  }
  for (; sp < n_split; ++sp)
#pragma unroll
    for (int m = 0; m < 4; ++m)
      if (live[m]) acc[m] += spart[sp * plane + q * n_g + lane + 64 * m];
#pragma unroll
  for (int m = 0; m < 4; ++m)  // NaN and -inf are never selected
    c[m] = live[m] && acc[m] > -__builtin_inff() ? Cand{acc[m], index_base + lane + 64 * m}
                                                 : Cand{-__builtin_inff(), -1};
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const int e = lane + 64 * m;
    c[4 + m] = Cand{-__builtin_inff(), -1};
    if (merge && e < k) c[4 + m] = Cand{top_s[q * k + e], top_i[q * k + e]};
  }
  for (int r = 0; r < k; ++r) {
    Cand lb = c[0];
#pragma unroll
    for (int m = 1; m < 6; ++m)
      if (better(c[m], lb)) lb = c[m];
    const Cand wb = wave_best(lb);
    if (lane == 0) {
      top_s[q * k + r] = wb.i >= 0 ? wb.s : -__builtin_inff();
      top_i[q * k + r] = wb.i;
    }
    if (wb.i >= 0) {
#pragma unroll
      for (int m = 0; m < 6; ++m)
        if (c[m].i == wb.i && c[m].s == wb.s) c[m].i = -1;  // indices are unique
    }
  }
}

constexpr int SEL_NT = 1024;    // threads of the selection kernels below

// Bitonic sort of n (a power of two) candidates, best first
// ((score desc, index asc), empty entries last).
__device__ inline void bitonic_cand(Cand* a, int n) {
  for (int size = 2; size <= n; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      __syncthreads();
      for (int t = threadIdx.x; t < n / 2; t += SEL_NT) {
        const int i = 2 * t - (t & (stride - 1));
        const int j = i + stride;
        const Cand x = a[i], y = a[j];
        if ((i & size) == 0 ? better(y, x) : better(x, y)) {
          a[i] = y;
          a[j] = x;
        }
      }
    }
  __syncthreads();
}

// Sorts the n candidates of buf (which holds the next power of two of them) and
// writes the k best as a list.
__device__ inline void write_best(Cand* buf, int n, int k, float* os, int64_t* oi) {
  int n2 = 1;
  while (n2 < n || n2 < k) n2 <<= 1;
  for (int e = n + (int)threadIdx.x; e < n2; e += SEL_NT) buf[e] = cand_none();
  bitonic_cand(buf, n2);
  for (int j = threadIdx.x; j < k; j += SEL_NT) {
    const Cand c = buf[j];
    os[j] = c.i >= 0 ? c.s : -__builtin_inff();
    oi[j] = c.i >= 0 ? c.i : -1;
  }
}

// Split-K plan with more than 256 rows or a larger k (a store of fewer than 32768
// rows; fewer than k of them pass whole):
// one workgroup per query sums every row's slices (slice order) into registers,
// rows u 1024 + t in thread t.  The k-th largest of the threads' best rows is
// reached by k distinct rows, so the k best of all are at or above it; those
// (random stores: k to 2 k rows), and the previous list when merging, are
// gathered into LDS and sorted.  Where many more qualify (an all-zero query, many
// copies of a row, the best rows in few threads), the k-th row of all is found by
// score and, among equal scores, by index, and only the k best are gathered (8 x
// 20000 x 2048, k = 100, all-zero queries: k rounds of arg-max over the registers
// 690 us, now 50; sorted segment maxima, before, 178).  What bounds it is latency:
// 1024 threads with VPT loads in flight each (at VPT = 32 ten registers spill); 256
// threads over parts of 8192 rows with sorted segment maxima, and a merge of the
// parts, took 96 us for 10 queries x 11335 rows, k = 100, and 30 us for 64 x 4096, k
// = 10.
constexpr int SEL_CAP = 1024;  // entries gathered and sorted in LDS: 3 k + 64 rows and a list
template <int VPT>
__global__ __launch_bounds__(SEL_NT) void score_split_select_kernel(
    const float* __restrict__ spart, int64_t nqp, int64_t n_g, int n_split, int k, int merge,
    int64_t index_base, float* top_s, int64_t* top_i) {
  __shared__ Cand buf[SEL_CAP];
  __shared__ int kcnt[48];
  __shared__ int cnt;
  constexpr int NWAVE = SEL_NT / kWave;
  __shared__ int tied_before[VPT][NWAVE];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (threadIdx.x == 0) cnt = 0;  // (block_kth's barriers follow)
  constexpr int SL = VPT == 32 ? 1 : VPT == 16 ? 2 : 8;  // slices loaded at once
  const int64_t q = blockIdx.x;
  const int t = threadIdx.x;
  const int64_t plane = n_g * nqp;
  const float* base = spart + q * n_g;
  float v[VPT];
#pragma unroll
  for (int u = 0; u < VPT; ++u) v[u] = 0.f;
  for (int sp = 0; sp < n_split; sp += SL) {
    float x[SL][VPT];
#pragma unroll
    for (int a = 0; a < SL; ++a) {
      const float* src = base + (sp + a) * plane;
      // 32 rows a thread: through a descriptor of the slice, whose 32-bit offsets
      // leave the registers to the scores (rows past the end read as zeros)
      const __amdgpu_buffer_rsrc_t r = make_rsrc(src, (uint32_t)n_g * 4u);
#pragma unroll
      for (int u = 0; u < VPT; ++u) {
        const int j = u * SEL_NT + t;
        if (VPT == 32)
          x[a][u] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (uint32_t)j * 4u, 0, 0));
        else
          x[a][u] = j < (int)n_g && sp + a < n_split ? src[j] : 0.f;
      }
    }
#pragma unroll
    for (int a = 0; a < SL; ++a)
#pragma unroll
      for (int u = 0; u < VPT; ++u) v[u] += x[a][u];
  }
  // NaN and -inf are never selected (key 0)
  auto key_of = [&](int u) -> uint32_t {
    const uint32_t key = fkey(v[u]);
    return u * SEL_NT + t < (int)n_g && selectable(key) ? key : 0u;
  };
  uint32_t best_key = 0u;
#pragma unroll
  for (int u = 0; u < VPT; ++u) {
    const uint32_t key = key_of(u);
    best_key = key > best_key ? key : best_key;
  }
  int reach;
  uint32_t tau = block_kth<1>([&](int) { return best_key; }, k, 16, kcnt, reach);
  tau = tau ? tau : 1u;
  // Rows of at least tau, or (tied) those above it and, of those whose key is tau,
  // the first `ties` in index order: tied_before[u][wave] counts the ties before
  // this wave's rows u.
  int ties = 0;
  auto gather = [&](auto tied) {
    int64_t row0 = index_base + t;
    asm volatile("" : "+v"(row0));  // (the rows' indices are not held in registers meanwhile)
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
      const uint32_t key = key_of(u);
      bool pass = key >= tau;
      if (decltype(tied)::value) {
        const uint64_t at_tau = __builtin_amdgcn_ballot_w64(key == tau);
        const int at = tied_before[u][wave] + __builtin_popcountll(at_tau & ((1ull << lane) - 1ull));
        pass = key > tau || (key == tau && at < ties);
      }
      if (pass) {
        const int pos = atomicAdd(&cnt, 1);
        if (pos < SEL_CAP) buf[pos] = Cand{v[u], row0 + u * SEL_NT};
      }
    }
    __syncthreads();
    return cnt;
  };
  auto rows_above = [&]() -> int {
    int n = 0;
#pragma unroll
    for (int u = 0; u < VPT; ++u) n += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key_of(u) > tau));
    return block_total(n, kcnt);
  };
  const int prev = merge ? k : 0;
  // more rows than this cost more to gather and sort than to count out
  const int most = 3 * k + 64;
  int n = reach > k + 16 ? most + 1 : gather(std::false_type{});
  if (n > most) {  // uniform
    int above = rows_above();
    if (above >= k) {  // the best rows sit in few threads: the k-th of all rows
      tau = block_kth<VPT>(key_of, k, 0, kcnt, reach);
      above = rows_above();
    }
#pragma unroll
    for (int u = 0; u < VPT; ++u) {
      const int tied = __builtin_popcountll(__builtin_amdgcn_ballot_w64(key_of(u) == tau));
      if (lane == 0) tied_before[u][wave] = tied;
    }
    __syncthreads();
    if (wave == 0) {  // counts -> counts before, in row order (u, wave)
      constexpr int E = VPT * NWAVE > kWave ? VPT * NWAVE / kWave : 1;  // per lane
      int* c = &tied_before[0][0] + lane * E;
      const bool mine = lane * E < VPT * NWAVE;
      int sum = 0;
      for (int e = 0; mine && e < E; ++e) sum += c[e];
      int run = sum;
#pragma unroll
      for (int off = 1; off < kWave; off <<= 1) {
        const int o = __shfl_up(run, off, kWave);
        run += lane >= off ? o : 0;
      }
      run -= sum;
      for (int e = 0; mine && e < E; ++e) {
        const int x = c[e];
        c[e] = run;
        run += x;
      }
    }
    ties = k - above;
    if (t == 0) cnt = 0;
    __syncthreads();
    n = gather(std::true_type{});  // k
  }
  float* os = top_s + q * k;
  int64_t* oi = top_i + q * k;
  for (int e = t; e < prev; e += SEL_NT) {
    const Cand c{os[e], oi[e]};
    buf[n + e] = c.i >= 0 ? c : cand_none();
  }
  write_best(buf, n + prev, k, os, oi);
}

// One workgroup per query merges n_parts + merge <= 1024 sorted lists.  The
// first d entries of every list (as many as 4096 entries allow, so at least k in
// all) are loaded side by side; the k-th best of them is a lower bound on the
// k-th best overall, and the entries at or above it (a prefix of each list; past
// d entries the list's last thread goes on alone) are gathered into LDS and
// sorted.  Where more than a few entries share the k-th score (an all-zero query:
// every score is 0) the bound is by index too, so that at most k + slack of the
// loaded entries pass, at most (k + slack) / d lists go on, and all of them fit.
// rows: the lists' indices are index_base .. index_base + rows - 1.
// Latency-bound: one thread per list walking its prefix, between two sorts of 256
// threads, took 30-41 us at k = 100 over 512 lists as over two.
constexpr int MERGE_E = 4;       // entries per thread of the first load
constexpr int MERGE_CAP = 4096;  // k + (k / d) (k - d) <= 4096 for k <= 128, d >= 4
__global__ __launch_bounds__(SEL_NT) void score_merge_kernel(const float* __restrict__ part_s,
                                                             const int64_t* __restrict__ part_i,
                                                             int n_parts, int k, int merge,
                                                             int64_t index_base, uint32_t rows,
                                                             float* top_s, int64_t* top_i) {
  __shared__ Cand buf[MERGE_CAP];
  __shared__ int kcnt[48];
  __shared__ int cnt;
  const int64_t q = blockIdx.x;
  const int t = threadIdx.x;
  const int n_src = n_parts + (merge ? 1 : 0);
  auto list_s = [&](int src) { return src < n_parts ? part_s + (q * n_parts + src) * (int64_t)k : top_s + q * (int64_t)k; };
  auto list_i = [&](int src) { return src < n_parts ? part_i + (q * n_parts + src) * (int64_t)k : top_i + q * (int64_t)k; };
  auto entry = [&](int src, int j) { return Cand{list_s(src)[j], list_i(src)[j]}; };
  // A caller's previous list may hold -inf, or anything, under a valid index.
  // -0 and +0 are equal scores: + 0.f makes both +0.
  auto key_of = [](const Cand& c) -> uint32_t { return c.i < 0 ? 0u : c.s == c.s ? fkey(c.s + 0.f) : 1u; };
  const int room = n_src > 0 ? MERGE_E * SEL_NT / n_src : k;
  const int d = room < k ? room : k;
  Cand e4[MERGE_E];
  uint32_t key[MERGE_E];
#pragma unroll
  for (int m = 0; m < MERGE_E; ++m) {
    const int e = t + SEL_NT * m, src = e / d;
    e4[m] = src < n_src ? entry(src, e - src * d) : cand_none();
    key[m] = key_of(e4[m]);
  }
  const int slack = k + 16 + (k + 16) / d * (k - d) <= MERGE_CAP ? 16 : 0;
  int reach;
  uint32_t tau = block_kth<MERGE_E>([&](int m) { return key[m]; }, k, slack, kcnt, reach);
  // Index order as 32-bit keys, larger is earlier: this call's rows, and before and
  // after them the previous list's other entries (j: their place in it).
  auto before = [&](const Cand& c, int j) -> uint32_t {
    const int64_t r = c.i - index_base;
    return rows + 256u - (r < 0 ? (uint32_t)j : r < (int64_t)rows ? 128u + (uint32_t)r : 128u + rows + (uint32_t)j);
  };
  uint32_t tie = 0u;  // of the entries whose key is tau, those with before() >= tie
  if (reach > k + slack) {
    int above = 0;
#pragma unroll
    for (int m = 0; m < MERGE_E; ++m) above += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key[m] > tau));
    above = block_total(above, kcnt);
    tie = block_kth<MERGE_E>([&](int m) { return key[m] == tau ? before(e4[m], (t + SEL_NT * m) % d) : 0u; },
                             k - above, 0, kcnt, reach, 32 - __builtin_clz(rows + 256u));
  }
  tau = tau ? tau : 1u;
  if (t == 0) cnt = 0;
  __syncthreads();
  auto passes = [&](const Cand& c, int j) {
    const uint32_t ck = key_of(c);
    return ck > tau || (ck == tau && before(c, j) >= tie);
  };
  auto take = [&](const Cand& c) {
    const int pos = atomicAdd(&cnt, 1);
    if (pos < MERGE_CAP) buf[pos] = c;
  };
#pragma unroll
  for (int m = 0; m < MERGE_E; ++m)
    if (key[m] >= tau && passes(e4[m], (t + SEL_NT * m) % d)) {
      take(e4[m]);
      const int e = t + SEL_NT * m, src = e / d;
      if (e - src * d == d - 1)
        for (int j = d; j < k; ++j) {
          const Cand c = entry(src, j);
          if (!passes(c, j)) break;
          take(c);
        }
    }
  __syncthreads();
  // (more than the buffer holds only from a previous list that names an index
  // many times)
  write_best(buf, cnt < MERGE_CAP ? cnt : MERGE_CAP, k, top_s + q * (int64_t)k, top_i + q * (int64_t)k);
}

// The merge for small k: k rounds of block arg-max over the heads of up to 1024
// lists, four a thread.  Takes ~1.3 us a round whatever the scores: 16 queries, 512
// lists, the whole call 61 us at k = 1 (the kernel above 66), 119 at k = 5 (122), 95
// at k = 10 (92); with an all-zero query 59 at k = 4 (72).
constexpr int MERGE_ROUNDS_K = 8;
__global__ __launch_bounds__(256) void score_merge_rounds_kernel(const float* __restrict__ part_s,
                                                                 const int64_t* __restrict__ part_i,
                                                                 int n_parts, int k, int merge,
                                                                 float* top_s, int64_t* top_i) {
  __shared__ Cand wb[2][4];
  __shared__ Cand out[MERGE_ROUNDS_K];
  const int64_t q = blockIdx.x;
  const int t = threadIdx.x;
  const float* src_s[4];
  const int64_t* src_i[4];
  int head[4];
  Cand cur[4];
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int src = t + 256 * m;
    const bool prev = merge && src == n_parts;
    src_s[m] = prev ? top_s + q * (int64_t)k : part_s + (q * n_parts + src) * (int64_t)k;
    src_i[m] = prev ? top_i + q * (int64_t)k : part_i + (q * n_parts + src) * (int64_t)k;
    head[m] = prev || src < n_parts ? 0 : k;
    cur[m] = head[m] < k ? Cand{src_s[m][0], src_i[m][0]} : cand_none();
  }
  for (int j = 0; j < k; ++j) {
    Cand mine = cur[0];
#pragma unroll
    for (int m = 1; m < 4; ++m)
      if (better(cur[m], mine)) mine = cur[m];
    const Cand w = wave_best(mine);
    if ((t & 63) == 0) wb[j & 1][t >> 6] = w;
    __syncthreads();
    Cand best = wb[j & 1][0];
#pragma unroll
    for (int v = 1; v < 4; ++v)
      if (better(wb[j & 1][v], best)) best = wb[j & 1][v];
    if (t == 0) out[j] = best;
    // the list whose head won advances (indices are unique across lists)
#pragma unroll
    for (int m = 0; m < 4; ++m)
      if (best.i >= 0 && cur[m].i == best.i && cur[m].s == best.s) {
        ++head[m];
        cur[m] = head[m] < k ? Cand{src_s[m][head[m]], src_i[m][head[m]]} : cand_none();
      }
  }
  __syncthreads();
  if (t < k) {
    const Cand c = out[t];
    top_s[q * (int64_t)k + t] = c.i >= 0 ? c.s : -__builtin_inff();
    top_i[q * (int64_t)k + t] = c.i >= 0 ? c.i : -1;
  }
}

}  // namespace

// Streaming-plan launch shape: list capacity KMAX (64 or 128: one or two
// list registers per query), ring depth RING, K-groups per stage GPS, list
// slots per wave QPW (a block's queries / 4: register budget), workgroups
// per CU and tile height TR x 64 rows.  The lists live in registers, so the
// LDS holds only the ring (RING x GPS x (64 TR + 64) rows x 128 B); two
// workgroups per CU were 10-20% faster than one at k > 64, and 128-row
// tiles (a three-stage ring of 24 KB slots) beat 64-row tiles (four 16 KB
// slots) by 4% at 16 queries and 13% at 64 (2M x 8192 fp16: 78-83% of HBM
// bandwidth at 16 to 64 queries and k up to 128).
struct StreamCfg {
  int kmax, ring, gps, qpw, per_cu, tr;
};
static StreamCfg stream_cfg(int64_t n_q, int k) {
  const int64_t qb = n_q < SQ ? n_q : SQ;
  const int qpw = qb <= 16 ? 4 : (qb <= 32 ? 8 : 16);
  const int kmax = k <= 64 ? 64 : 128;
  // 128-row tiles: half the query bytes per store byte through the ring
  return {kmax, 3, 1, qpw, 2, 2};
}

static size_t align256(size_t b) { return (b + 255) / 256 * 256; }
constexpr int64_t BOUND_ROWS = 16384;  // prefix rows whose segment maxima bound the k-th best

ScorePlan plan_score(int64_t n_q, int64_t n_g, int64_t D, int k, int elem_bytes, bool fewest_bytes) {
  ScorePlan P{};
  P.D = D;
  P.n_qb = (int)((n_q + SQB - 1) / SQB);
  P.n_grp = (int)(D * elem_bytes / 128);
  if (n_q <= 0 || n_g <= 0) return P;
  // (the streaming plan at 128-384 queries measured 1.2-2.8x slower)
  // GEMM plan: score chunks of at most ~256 MB (MALL-resident between the
  // GEMM and the selection) and RS_MAXCHUNK rows, at most GEMM_MAX_PARTS
  // chunks (the merge takes 1024 sources, one of them the previous list);
  // a store too large for that takes the streaming plan, whose partitions
  // grow with the store
  constexpr int64_t GEMM_MAX_PARTS = 1023;
  if (elem_bytes == 2 && D % GKS == 0 && n_q >= 128 && n_g >= 4096 &&
      n_g <= RS_MAXCHUNK * GEMM_MAX_PARTS) {
    // Tiles: 256 x 256, or 128 queries x 256 rows (the ring core) where the
    // last 256-query tile would be at most half used (n_q % 256 in [1, 128])
    // and the query count is small enough that store rows, not queries, set
    // the work (the narrow tile reads each store row once per 128 queries).
    const int64_t rem = n_q % 256;
    const bool narrow = rem >= 1 && rem <= 128 && n_q <= 384;
    const int64_t rt = narrow ? GRR : GT;
    int64_t chunk = ((int64_t)256 << 20) / (n_q * 4);
    chunk = chunk > RS_MAXCHUNK ? RS_MAXCHUNK : chunk;
    const int64_t min_chunk = (n_g + GEMM_MAX_PARTS - 1) / GEMM_MAX_PARTS;  // <= RS_MAXCHUNK
    chunk = chunk < min_chunk ? min_chunk : chunk;
    chunk = chunk < 4096 ? 4096 : chunk;
    chunk = (chunk + rt - 1) / rt * rt;
    const int64_t all = (n_g + rt - 1) / rt * rt;
    chunk = chunk > all ? all : chunk;
    P.gemm = narrow ? 2 : 1;
    P.chunk = chunk;
    P.n_parts = (int)((n_g + chunk - 1) / chunk);
    P.rows_per_part = chunk;
    P.split = 1;
    // scores, segment maxima (one per 64 rows), running bound per query
    P.spart_bytes = (size_t)n_q * (size_t)chunk * 4 + (size_t)n_q * (size_t)(chunk / RS_SEG) * 4 +
                    (size_t)n_q * 4;
    P.list_entries = (size_t)n_q * (size_t)P.n_parts * (size_t)k;
    return P;
  }
  const int64_t n_tiles = (n_g + STN - 1) / STN;
  // Too few (query block, row tile) pairs to occupy 256 CUs: split D.
  int64_t split = 1;
  if (P.n_qb * n_tiles < 256) {
    split = (256 + P.n_qb * n_tiles - 1) / (P.n_qb * n_tiles);
    const int64_t max_split = P.n_grp / 8 > 1 ? P.n_grp / 8 : 1;  // >= 8 groups per slice
    split = split > max_split ? max_split : split;
    const int64_t cap = ((int64_t)256 << 20) / ((int64_t)n_g * P.n_qb * SQB * 4);
    split = split > cap ? cap : split;
  }
  // Rows of fewer than 16 groups are not split, but take the same two kernels
  // where the workspace holds their scores (a workspace of the streaming plan's
  // size takes that one): streaming / these, 8 queries x 256 rows x 256 in fp32
  // 34 / 13 us, 64 x 2000 x 512, k = 100, 346 / 28, 100 x 10000 x 64 151 / 18, 1
  // x 32000 x 64 15.1 / 14.3.
  if (split >= 2 || (P.n_qb * n_tiles < 256 && !fewest_bytes)) {
    // partial slices, then one selection workgroup per query straight into
    // the output (no partition lists): n_g < 256 x 128 rows here
    P.split = (int)split;
    P.split_plan = 1;
    P.n_tiles = (int)n_tiles;
    P.rows_per_part = n_g;
    P.n_parts = 0;  // no partition lists
    P.spart_bytes = (size_t)split * (size_t)n_g * (size_t)P.n_qb * SQB * 4;
  } else {
    P.split = 1;
    // streaming plan: 64 queries per workgroup; two workgroups per CU when
    // the ring and the lists fit in half the LDS, else one; as many
    // partitions as workgroups fit at once (an exact multiple of the CU
    // count: 248 workgroups ran ~13% slower than 256 on k <= 32)
    P.n_qb = (int)((n_q + SQ - 1) / SQ);
    int64_t per_wave = (int64_t)stream_cfg(n_q, k).per_cu * 256;
    per_wave = per_wave > 1016 ? 1016 : per_wave;  // the merge takes <= 1024 sources
    int64_t parts = (per_wave + P.n_qb - 1) / P.n_qb;
    const int64_t srt = (int64_t)SR * stream_cfg(n_q, k).tr;  // rows per tile
    const int64_t t64 = (n_g + srt - 1) / srt;
    parts = parts > t64 ? t64 : parts;
    parts = parts > per_wave ? per_wave : (parts < 1 ? 1 : parts);
    int64_t rpp = (n_g + parts - 1) / parts;
    rpp = (rpp + srt - 1) / srt * srt;
    P.rows_per_part = rpp;
    P.n_parts = (int)((n_g + rpp - 1) / rpp);
    P.spart_bytes = 0;
    // the bound pass (~0.1 ms) pays when the lists see many insertions: a
    // large store and many (query, list entry) pairs
    if (n_g >= 16 * BOUND_ROWS && n_q * k >= 1024) {
      P.bound_rows = BOUND_ROWS;
      const size_t nb = (size_t)(BOUND_ROWS / SR);
      P.spart_bytes = align256((size_t)n_q * nb * 4) + align256((size_t)n_q * nb * 8) + align256((size_t)n_q * 4);
    }
  }
  P.list_entries = (size_t)n_q * (size_t)P.n_parts * (size_t)k;
  return P;
}

// bound[q] = k-th largest of the nb segment maxima of query q (-inf when
// fewer than k are finite).  One workgroup per query; nb <= 1024.
__global__ __launch_bounds__(256) void score_bound_kernel(const float* __restrict__ seg_s, int nb, int k,
                                                          float* __restrict__ bound) {
  __shared__ int kcnt[48];
  const int64_t q = blockIdx.x;
  uint32_t key[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int i = (int)threadIdx.x + 256 * u;
    const uint32_t x = i < nb ? fkey(seg_s[q * nb + i]) : 0u;
    key[u] = selectable(x) ? x : 0u;
  }
  int reach;
  const uint32_t kth = block_kth<4>([&](int u) { return key[u]; }, k, 0, kcnt, reach);
  if (threadIdx.x == 0) bound[q] = kth ? fkey_inv(kth) : -__builtin_inff();
}

hipError_t launch_score_topk(bool f16, const ScorePlan& plan, const void* Q, int64_t n_q,
                             int64_t ldq, const void* G, int64_t n_g, int64_t ldg, int k,
                             int64_t index_base, int merge, float* top_s, int64_t* top_i,
                             float* part_s, int64_t* part_i, float* spart, hipStream_t s) {
  const int n_parts = n_g > 0 ? plan.n_parts : 0;
  if (n_g > 0 && plan.gemm) {
    const int tq = plan.gemm == 2 ? GRQ : GT, tr = plan.gemm == 2 ? GRR : GT;
    const int n_qt = (int)((n_q + tq - 1) / tq);
    const int n_st = plan.n_grp;  // 64-element fp16 stages (128 bytes)
    const int64_t n_seg = plan.chunk / RS_SEG;
    float* segmax = spart + n_q * plan.chunk;
    float* thr = segmax + n_q * n_seg;
    for (int c = 0; c < plan.n_parts; ++c) {
      const int64_t r0 = (int64_t)c * plan.chunk;
      const int64_t nc = n_g - r0 < plan.chunk ? n_g - r0 : plan.chunk;
      const int n_items = n_qt * (int)((nc + tr - 1) / tr);
      const int per_xcd = (n_items + 7) / 8;
      const bool nt = n_qt == 1;
      hipLaunchKernelGGL(plan.gemm == 2 ? (nt ? score_gemm_r_kernel<F16Tag, true>
                                              : score_gemm_r_kernel<F16Tag, false>)
                                        : (nt ? score_gemm_kernel<F16Tag, true>
                                              : score_gemm_kernel<F16Tag, false>),
                         dim3((unsigned)(8 * per_xcd)), dim3(256), 0, s, (const _Float16*)Q, n_q,
                         ldq, (const _Float16*)G + r0 * ldg, nc, ldg, n_qt, n_items, per_xcd, n_st,
                         spart, plan.chunk, segmax, n_seg, (const float*)thr, c > 0 ? 1 : 0);
      hipLaunchKernelGGL(score_rselect_kernel, dim3((unsigned)n_q), dim3(256), 0, s,
                         (const float*)spart, plan.chunk, (const float*)segmax, n_seg, thr, nc, k, c,
                         plan.n_parts, index_base + r0, part_s, part_i);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  } else if (n_g > 0 && !plan.split_plan) {
    // lower bound on each query's k-th best score: the k-th largest of the
    // maxima of the first bound_rows / 64 row segments (k distinct rows reach
    // it).  The maxima come from this kernel run with k = 1 over one-tile
    // partitions.
    const float* bound = nullptr;
    if (plan.bound_rows > 0) {
      const int nb = (int)(plan.bound_rows / SR);
      char* w = reinterpret_cast<char*>(spart);
      float* seg_s = reinterpret_cast<float*>(w);
      int64_t* seg_i = reinterpret_cast<int64_t*>(w + align256((size_t)n_q * nb * 4));
      float* bnd = reinterpret_cast<float*>(w + align256((size_t)n_q * nb * 4) + align256((size_t)n_q * nb * 8));
      const StreamCfg cb = stream_cfg(n_q, 1);
      const int pp = (nb + 7) / 8 * 8;
      dim3 gb((unsigned)(plan.n_qb * pp)), bb(256);
      bool ok = false;
#define ATTR_SB(KM, RG, GP, QW)                                                                  \
  if (cb.qpw == QW) {                                                                          \
    ok = true;                                                                                   \
    if (f16)                                                                                     \
      hipLaunchKernelGGL((score_stream_kernel<true, KM, RG, GP, QW, 1>), gb, bb, 0, s,           \
                         (const char*)Q, n_q, ldq, (const char*)G, plan.bound_rows, ldg,        \
                         plan.n_grp, 1, (int64_t)SR, nb, plan.n_qb, (const float*)nullptr, seg_s, \
                         seg_i, (int64_t)0);                                                     \
    else                                                                                         \
      hipLaunchKernelGGL((score_stream_kernel<false, KM, RG, GP, QW, 1>), gb, bb, 0, s,          \
                         (const char*)Q, n_q, ldq, (const char*)G, plan.bound_rows, ldg,        \
                         plan.n_grp, 1, (int64_t)SR, nb, plan.n_qb, (const float*)nullptr, seg_s, \
                         seg_i, (int64_t)0);                                                     \
  }
      ATTR_SB(64, 4, 1, 4)
      ATTR_SB(64, 4, 1, 8)
      ATTR_SB(64, 4, 1, 16)
#undef ATTR_SB
      if (!ok) return hipErrorInvalidConfiguration;
      hipLaunchKernelGGL(score_bound_kernel, dim3((unsigned)n_q), dim3(256), 0, s, (const float*)seg_s, nb,
                         k, bnd);
      hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
      bound = bnd;
    }
    const int parts_pad = (plan.n_parts + 7) / 8 * 8;
    dim3 grid((unsigned)(plan.n_qb * parts_pad)), block(256);
#define ATTR_SS(KM, RG, GP, QW, TRR)                                                             \
  if (c.kmax == KM && c.ring == RG && c.gps == GP && c.qpw == QW && c.tr == TRR) {               \
    launched = true;                                                                             \
    if (f16)                                                                                     \
      hipLaunchKernelGGL((score_stream_kernel<true, KM, RG, GP, QW, TRR>), grid, block, 0, s,     \
                         (const char*)Q, n_q, ldq, (const char*)G, n_g, ldg, plan.n_grp, k,      \
                         plan.rows_per_part, plan.n_parts, plan.n_qb, bound, part_s, part_i,     \
                         index_base);                                                            \
    else                                                                                         \
      hipLaunchKernelGGL((score_stream_kernel<false, KM, RG, GP, QW, TRR>), grid, block, 0, s,    \
                         (const char*)Q, n_q, ldq, (const char*)G, n_g, ldg, plan.n_grp, k,      \
                         plan.rows_per_part, plan.n_parts, plan.n_qb, bound, part_s, part_i,     \
                         index_base);                                                            \
  }
    const StreamCfg c = stream_cfg(n_q, k);
    bool launched = false;
    ATTR_SS(64, 3, 1, 4, 2)
    ATTR_SS(64, 3, 1, 8, 2)
    ATTR_SS(64, 3, 1, 16, 2)
    ATTR_SS(128, 3, 1, 4, 2)
    ATTR_SS(128, 3, 1, 8, 2)
    ATTR_SS(128, 3, 1, 16, 2)
    if (!launched) return hipErrorInvalidConfiguration;
#undef ATTR_SS
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  } else if (n_g > 0) {
    dim3 grid((unsigned)((int64_t)plan.n_qb * plan.n_tiles * plan.split)), block(256);
#define ATTR_SK(F, QT)                                                                               \
  hipLaunchKernelGGL((score_splitk_kernel<F, QT>), grid, block, 0, s, (const char*)Q, n_q, ldq,      \
                     (const char*)G, n_g, ldg, plan.n_grp, plan.n_qb, plan.n_tiles, plan.split, spart)
    if (n_q <= 16) {
      if (f16) ATTR_SK(true, 1);
      else ATTR_SK(false, 1);
    } else if (n_q <= 32) {
      if (f16) ATTR_SK(true, 2);
      else ATTR_SK(false, 2);
    } else {
      if (f16) ATTR_SK(true, 4);
      else ATTR_SK(false, 4);
    }
#undef ATTR_SK
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (small_select(n_g, k)) {
      hipLaunchKernelGGL(score_small_select_kernel, dim3((unsigned)n_q), dim3(64), 0, s,
                         (const float*)spart, (int64_t)plan.n_qb * SQB, n_g, plan.split, k,
                         merge, index_base, top_s, top_i);
      return hipGetLastError();
    }
#define ATTR_SEL(V)                                                                              \
  hipLaunchKernelGGL(score_split_select_kernel<V>, dim3((unsigned)n_q), dim3(SEL_NT), 0, s,     \
                     (const float*)spart, (int64_t)plan.n_qb * SQB, n_g, plan.split, k, merge,  \
                     index_base, top_s, top_i)
    if (n_g <= SEL_NT) ATTR_SEL(1);
    else if (n_g <= 4 * SEL_NT) ATTR_SEL(4);
    else if (n_g <= 16 * SEL_NT) ATTR_SEL(16);
    else if (n_g <= 32 * SEL_NT) ATTR_SEL(32);
    else return hipErrorInvalidConfiguration;  // the plan splits fewer than 32768 rows
#undef ATTR_SEL
    return hipGetLastError();
  }
  if (k <= MERGE_ROUNDS_K) {
    hipLaunchKernelGGL(score_merge_rounds_kernel, dim3((unsigned)n_q), dim3(256), 0, s, (const float*)part_s,
                       (const int64_t*)part_i, n_parts, k, merge, top_s, top_i);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(score_merge_kernel, dim3((unsigned)n_q), dim3(SEL_NT), 0, s,
                     (const float*)part_s, (const int64_t*)part_i, n_parts, k, merge, index_base, (uint32_t)n_g, top_s,
                     top_i);
  return hipGetLastError();
}

}  // namespace attr
