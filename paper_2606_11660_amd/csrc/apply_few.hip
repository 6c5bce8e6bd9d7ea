// Full preconditioner on few rows: y = M x for a session's queries or a
// small batch of store rows (M = H^{-1/2}, fp32, see apply_full.hip), with
// the unit norm.
//
// With few rows the work is reading M (4 D^2 bytes) once.  The general path
// writes M's two fp16 halves to memory first (a pass for max|M|, one that
// reads M and writes the halves, and the GEMM that reads them back: four
// times M's bytes, and a GEMM of D / 256 workgroups at up to 256 rows).
// Here each workgroup reads 64 rows of M over one K-slice straight from the
// caller's matrix, splits the values into fp16 hi + lo on the way to LDS and
// multiplies them with its rows of X; M is read once per 256 rows of X.
//  * M is loaded by 16 lanes per 256-byte row piece (64 values), PD stages
//    ahead into registers; X's MFMA fragments come straight from L2 into
//    registers, also PD stages ahead (every workgroup reads all of X's rows:
//    64 rows of M per workgroup make X's traffic half of what 32 would).
//  * The split needs a power-of-two scale that keeps hi inside fp16's range
//    and lo above its subnormals.  Instead of a pass for max|M|, each row of
//    M carries a running exponent: the 16 lanes that hold a row's 64 values
//    reduce their maximum and, should it pass 2^15 on the row's scale, lower
//    the exponent (2 bits of headroom below); the waves then scale their sums
//    of that row by the same power of two (exact).  hi + lo keeps 22 bits of
//    every value within 2^-12 of its row's running maximum, and an absolute
//    2^-37 of that maximum below.  (The general path's floor is 2^-39 of max|M|:
//    lower in the rows that hold max|M|, higher where a row's own maximum is less
//    than a quarter of it.)
//  * One barrier per two stages (four LDS stage buffers).
// The sums go to fp32 partials per K-slice, [slice][row][D]; a second kernel
// adds the slices in order, forms the row's norm and writes Y with a single
// rounding (no fp16 intermediate).  Deterministic.
// 256 rows x 8192: 628 us on the general path (max|M| 152, split 149, GEMM
// 316, norm 7) -> 93-103 us (this kernel 79 us, 3.4 TB/s of M, packing X 5,
// final 6.5); up to 64 rows the kernel reads M at 5.7 TB/s.  At 256 rows the
// fragments of X pass through the L2 once per 64 columns of Y (537 MB), and the
// third of them that misses it comes beside M's 268 MB: 443 MB, 5.65 TB/s.
// Tried: more stages in flight (6, 8), one barrier per stage, two workgroups
// per CU at 64 rows, MFMAs and split interleaved by hand: no change.
#include "common.h"
#include "kernels.h"

namespace attr {
namespace {

constexpr int FCOL = 64;  // rows of M (columns of Y) per workgroup
constexpr int FKS = 64;   // K per stage
constexpr int FPD = 4;    // stages of M and X in flight
constexpr int FBS = 2;    // stages per barrier
constexpr int FUNSET = 1000;  // exponent of a row of M that was all zero so far

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

// largest of v over the 16 lanes of this lane's DPP row
__device__ inline uint32_t row16_max(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false));  // row_ror:8
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, false));
  return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, false));
}

// X into MFMA fragment order: fragment (K-half h of 32 values, 16-row tile t)
// is 64 lanes x 16 bytes, lane (ri, rg) holding values 32 h + 8 rg .. + 7 of
// row 16 t + ri, at fragment index h n_tiles + t.  Fragments loaded from X
// itself touch 16 rows a power of two apart, which fall on few channels of
// the L2 that every workgroup reads them from.  Rows past the end are zeros.
__global__ __launch_bounds__(256) void apply_few_pack_kernel(const _Float16* __restrict__ X,
                                                             int64_t n_rows, int64_t ldx, int64_t D,
                                                             int n_tiles, i32x4* __restrict__ xpk) {
  // a workgroup takes 16 rows x 128 values: 16 lanes read 256 bytes of a row
  const int t = (int)(blockIdx.x % (uint32_t)n_tiles);
  const int64_t c = (int64_t)(blockIdx.x / (uint32_t)n_tiles) * 16 + (threadIdx.x & 15);  // 8-value chunk
  const int ri = threadIdx.x >> 4;
  if (c >= D / 8) return;
  const int64_t row = (int64_t)t * 16 + ri;
  i32x4 v{0, 0, 0, 0};
  if (row < n_rows) v = *reinterpret_cast<const i32x4*>(X + row * ldx + c * 8);
  xpk[((c >> 2) * n_tiles + t) * kWave + (c & 3) * 16 + ri] = v;
}

// XT: 16-row tiles of X per wave pair (64 XT rows of X per workgroup).  NT: M
// is read once (a single row block), with the non-temporal cache policy.
// Eight waves: wave w takes the X rows of group w % 4 against K-half w / 4 of
// every stage, so two waves share a SIMD (one splits M while the other feeds
// the matrix core) and each needs half the X registers; with four waves of
// twice the registers the sums moved between the two register files at every
// stage, because a changed exponent scales them with vector instructions.
template <int XT, bool NT>
__global__ __launch_bounds__(512, 2) void apply_few_kernel(const _Float16* __restrict__ X,
                                                           int64_t n_rows, int64_t ldx, int64_t D,
                                                           const i32x4* __restrict__ xpk,
                                                           const float* __restrict__ M, int n_ct,
                                                           int n_sl, int n_rb, int n_units,
                                                           float* __restrict__ part) {
  // M stages (hi, then lo), later the second K-half's sums
  constexpr int NB = 2 * FBS;  // stage buffers: stage i in buffer i % NB
  __shared__ i32x4 sm[2 * NB * FCOL * 8];
  static_assert(XT * 1024 <= 2 * NB * FCOL * 8, "the exchange of the sums fits");
  __shared__ int sexp[NB][FCOL];
  __shared__ int schg[NB][8];
  auto sm_hi = [&](int b) { return sm + b * (FCOL * 8); };
  auto sm_lo = [&](int b) { return sm + (NB + b) * (FCOL * 8); };
  // the row blocks of one unit (64 rows of M, one K-slice) are consecutive
  // on one XCD, so that M comes from memory once and then from its L2
  const uint32_t jb = blockIdx.x >> 3;
  const int unit = (int)(jb / (uint32_t)n_rb) * 8 + (int)(blockIdx.x & 7u);
  const int rb = (int)(jb % (uint32_t)n_rb);
  if (unit >= n_units) return;  // uniform
  const int ct = unit % n_ct, sl = unit / n_ct;
  const int n_st = (int)(D / FKS);
  // slices of whole groups of FPD stages (the last group of D may be short)
  const int n_gr = (n_st + FPD - 1) / FPD;
  const int s0 = FPD * (int)((int64_t)n_gr * sl / n_sl);
  int s1 = FPD * (int)((int64_t)n_gr * (sl + 1) / n_sl);
  s1 = s1 > n_st ? n_st : s1;
  const int ns = s1 - s0;  // >= 1
  // each column tile starts at another stage of the slice and wraps: started
  // together, the workgroups would read M's rows, a power of two apart, from
  // the same few memory channels all the way (8192 x 8192, one row of X:
  // 74 -> 51 us a call)
  const int rot = (int)((uint32_t)ct * 37u % (uint32_t)ns);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int xw = wave & 3, kh = wave >> 2;
  const int lane = threadIdx.x & 63;
  const int ri = lane & 15, rg = lane >> 4;
  const int64_t c0 = (int64_t)ct * FCOL;

  // X: rows xr0 .. + 16 XT of this wave, from the packed fragments or (xpk
  // NULL) from X itself, where rows past the end read as zeros
  const int64_t xr0 = ((int64_t)rb * 4 + xw) * (16 * XT);
  int64_t nx = n_rows - xr0;
  nx = nx < 0 ? 0 : (nx > 16 * XT ? 16 * XT : nx);
  const uint32_t xtiles = (uint32_t)n_rb * 4u * XT;  // 16-row tiles of all row blocks
  const __amdgpu_buffer_rsrc_t rx =
      xpk ? make_rsrc(xpk, xtiles * 32u * (uint32_t)D)
          : make_rsrc(X + (nx > 0 ? xr0 * ldx : 0), (uint32_t)(nx * ldx * 2));
  const uint32_t xoff = xpk ? ((uint32_t)kh * xtiles + (uint32_t)(xr0 >> 4)) * 1024u + (uint32_t)lane * 16u
                            : (uint32_t)((int64_t)ri * ldx * 2 + kh * 64 + rg * 16);
  const uint32_t xtile = xpk ? 1024u : (uint32_t)(16 * ldx * 2);
  const uint32_t xstage = xpk ? xtiles * 2048u : (uint32_t)(FKS * 2);
  // M: load u of this lane takes row 8 wave + 4 u + rg of the tile, values
  // 4 ri .. + 3 of the stage's 64
  const __amdgpu_buffer_rsrc_t rm = make_rsrc(M + c0 * D, (uint32_t)(FCOL * D * 4));
  const uint32_t moff = (uint32_t)(((int64_t)(8 * wave + rg) * D + 4 * ri) * 4);
  const uint32_t mrow4 = (uint32_t)(4 * D * 4);

  i32x4 mreg[FPD][2], xreg[FPD][XT];
  // a stage past the slice's end is loaded from past both descriptors' ranges:
  // zeros, and no memory access (every load is issued unconditionally, so the
  // compiler counts the loads in flight instead of draining them at a branch)
  auto issue = [&](int i, i32x4 (&mr)[2], i32x4 (&xr)[XT]) {
    const bool live = i < ns;
    int st = s0 + rot + i;
    st = st >= s1 ? st - ns : st;
    const uint32_t mo = live ? moff + (uint32_t)st * (FKS * 4) : 0xc0000000u;
    const uint32_t xo = live ? xoff + (uint32_t)st * xstage : 0xc0000000u;
#pragma unroll
    for (int u = 0; u < 2; ++u)
      mr[u] = NT ? load16_stream(rm, mo + (uint32_t)u * mrow4) : load16_cached(rm, mo + (uint32_t)u * mrow4);
#pragma unroll
    for (int t = 0; t < XT; ++t) xr[t] = load16_cached(rx, xo + (uint32_t)t * xtile);
  };

  // running exponents: of the rows this lane splits (e[u]) and of the rows
  // its accumulators belong to (cur[mt][r]: row 16 mt + 4 rg + r)
  int e[2], cur[4][4];
#pragma unroll
  for (int u = 0; u < 2; ++u) e[u] = FUNSET;
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int r = 0; r < 4; ++r) cur[mt][r] = FUNSET;
  f32x4 acc[4][XT];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int t = 0; t < XT; ++t) acc[mt][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  // split a stage's M values into LDS buffer b; schg[b][wave] says whether an
  // exponent of this wave's rows moved
  auto split = [&](const i32x4 (&mr)[2], int b) {
    bool any = false;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const i32x4 w = mr[u];
      const f32x4 v = __builtin_bit_cast(f32x4, w);
      // |v| ordered as integers (a NaN passes as the largest: its exponent reads 0)
      const uint32_t m4 = row16_max(max(max((uint32_t)w.x & 0x7fffffffu, (uint32_t)w.y & 0x7fffffffu),
                                        max((uint32_t)w.z & 0x7fffffffu, (uint32_t)w.w & 0x7fffffffu)));
      const int ex = __builtin_amdgcn_frexp_expf(__uint_as_float(m4));  // max = f 2^ex, f in [0.5, 1)
      const bool up = m4 != 0u && ex + e[u] > 15;
      e[u] = up ? 13 - ex : e[u];
      any |= up;
      const float a0 = ldexpf(v.x, e[u]), a1 = ldexpf(v.y, e[u]);
      const float a2 = ldexpf(v.z, e[u]), a3 = ldexpf(v.w, e[u]);
      const f16x2 h0 = __builtin_convertvector(f32x2{a0, a1}, f16x2);
      const f16x2 h1 = __builtin_convertvector(f32x2{a2, a3}, f16x2);
      // a - hi is exact in fp32
      const f16x2 l0 = __builtin_convertvector(f32x2{a0 - (float)h0.x, a1 - (float)h0.y}, f16x2);
      const f16x2 l1 = __builtin_convertvector(f32x2{a2 - (float)h1.x, a3 - (float)h1.y}, f16x2);
      const int row = 8 * wave + 4 * u + rg;
      const int slot = (row * 8 + ((ri >> 1) ^ (row & 7))) * 2 + (ri & 1);  // 8-byte units
      reinterpret_cast<f16x4*>(sm_hi(b))[slot] = f16x4{h0.x, h0.y, h1.x, h1.y};
      reinterpret_cast<f16x4*>(sm_lo(b))[slot] = f16x4{l0.x, l0.y, l1.x, l1.y};
      sexp[b][row] = e[u];  // the same value from 16 lanes
    }
    schg[b][wave] = __builtin_amdgcn_ballot_w64(any) != 0;
  };

#pragma unroll
  for (int u = 0; u < FPD; ++u) issue(u, mreg[u], xreg[u]);
#pragma unroll
  for (int u = 0; u < FBS; ++u) split(mreg[u], u);
  wait_lgkm0();
  __builtin_amdgcn_s_barrier();

  static_assert(FPD == NB, "a ring slot's LDS buffer has its number");
  for (int g0 = 0; g0 < ns; g0 += FPD) {
#pragma unroll
    for (int u = 0; u < FPD; ++u) {
      const int i = g0 + u;  // stage s0 + i (zeros past s1), in LDS buffer u
      const int b = u;
      const i32x4 ch0 = reinterpret_cast<const i32x4*>(schg[b])[0];
      const i32x4 ch1 = reinterpret_cast<const i32x4*>(schg[b])[1];
      i32x4 fh[4], fl[4];
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        const int at = (16 * mt + ri) * 8 + ((4 * kh + rg) ^ (ri & 7));
        fh[mt] = sm_hi(b)[at];
        fl[mt] = sm_lo(b)[at];
      }
      if (__builtin_amdgcn_readfirstlane(ch0.x | ch0.y | ch0.z | ch0.w | ch1.x | ch1.y | ch1.z | ch1.w)) {
        // some row's exponent moved: bring its sums onto the new scale
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int en = sexp[b][16 * mt + 4 * rg + r];
            const int d = en - cur[mt][r];
            cur[mt][r] = en;
#pragma unroll
            for (int t = 0; t < XT; ++t) acc[mt][t][r] = ldexpf(acc[mt][t][r], d);
          }
        // the scaled sums leave this block as whole vectors: merged element
        // by element with the untouched ones, they cost a copy of every
        // accumulator at every stage
#pragma unroll
        for (int mt = 0; mt < 4; ++mt)
#pragma unroll
          for (int t = 0; t < XT; ++t) asm volatile("" : "+v"(acc[mt][t]));
      }
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int t = 0; t < XT; ++t) acc[mt][t] = mma16(F16Tag{}, fh[mt], xreg[u][t], acc[mt][t]);
#pragma unroll
      for (int mt = 0; mt < 4; ++mt)
#pragma unroll
        for (int t = 0; t < XT; ++t) acc[mt][t] = mma16(F16Tag{}, fl[mt], xreg[u][t], acc[mt][t]);
      split(mreg[(u + FBS) % FPD], (u + FBS) % FPD);
      // slot u's X has been used and its M was split FBS stages ago
      issue(i + FPD, mreg[u], xreg[u]);
      if (u % FBS == FBS - 1) {
        wait_lgkm0();
        __builtin_amdgcn_s_barrier();
      }
    }
  }

  // the two K-halves' sums (on the same scales) meet in LDS; the last barrier
  // ended every read of the stage buffers
  f32x4* ex = reinterpret_cast<f32x4*>(sm) + (xw * 4 * XT) * kWave + lane;
  if (kh == 1) {
#pragma unroll
    for (int mt = 0; mt < 4; ++mt)
#pragma unroll
      for (int t = 0; t < XT; ++t) ex[(mt * XT + t) * kWave] = acc[mt][t];
  }
  __syncthreads();
  if (kh == 1) return;
  // acc[mt][t][r]: column c0 + 16 mt + 4 rg + r of Y, row xr0 + 16 t + ri
#pragma unroll
  for (int t = 0; t < XT; ++t) {
    const int row = 16 * t + ri;
    if (row < nx) {
      float* dst = part + ((int64_t)sl * n_rows + xr0 + row) * D + c0 + 4 * rg;
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        f32x4 v = acc[mt][t] + ex[(mt * XT + t) * kWave];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = ldexpf(v[r], -cur[mt][r]);
        *reinterpret_cast<f32x4*>(dst + 16 * mt) = v;
      }
    }
  }
}

template <typename YT>
__device__ inline void put4(YT* p, const f32x4& v);
template <>
__device__ inline void put4<float>(float* p, const f32x4& v) {
  *reinterpret_cast<f32x4*>(p) = v;
}
template <>
__device__ inline void put4<_Float16>(_Float16* p, const f32x4& v) {
  f16x4 h;
#pragma unroll
  for (int q = 0; q < 4; ++q) h[q] = (_Float16)v[q];
  *reinterpret_cast<f16x4*>(p) = h;
}

// One workgroup per row: the slices' partial rows summed in slice order, the
// norm from those sums (fp64 across threads), Y written once.  The first
// FIN_REG column groups of a thread stay in registers between the norm and
// the write; wider rows sum theirs again.
constexpr int FIN_REG = 8;  // x 4 columns x 256 threads = 8192 columns
template <typename YT>
__global__ __launch_bounds__(256) void apply_few_final_kernel(const float* __restrict__ part, int n_sl,
                                                              int64_t n_rows, int64_t D, int unit,
                                                              YT* __restrict__ Y, int64_t ldy) {
  __shared__ double red[4];
  const int64_t r = blockIdx.x;
  const f32x4* p = reinterpret_cast<const f32x4*>(part + r * D);
  const int64_t plane = n_rows * D / 4;  // D is a multiple of 64
  const int n4 = (int)(D / 4);
  auto sum_of = [&](int c) {
    f32x4 s = p[c];
    for (int j = 1; j < n_sl; ++j) s += p[j * plane + c];
    return s;
  };
  f32x4 keep[FIN_REG];
  double ss = 0.0;
#pragma unroll
  for (int j = 0; j < FIN_REG; ++j) {
    const int c = (int)threadIdx.x + 256 * j;
    if (c < n4) {
      keep[j] = sum_of(c);
#pragma unroll
      for (int q = 0; q < 4; ++q) ss += (double)keep[j][q] * (double)keep[j][q];
    }
  }
  for (int c = (int)threadIdx.x + 256 * FIN_REG; c < n4; c += 256) {
    const f32x4 s = sum_of(c);
#pragma unroll
    for (int q = 0; q < 4; ++q) ss += (double)s[q] * (double)s[q];
  }
  float sc = 1.f;
  if (unit) {
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
    __syncthreads();
    ss = (red[0] + red[1]) + (red[2] + red[3]);
    // a zero row stays zero; a row with a NaN keeps it and is zero elsewhere, as
    // on the general path
    sc = ss > 0.0 ? (float)(1.0 / sqrt(ss)) : 0.f;
  }
  YT* y = Y + r * ldy;
#pragma unroll
  for (int j = 0; j < FIN_REG; ++j) {
    const int c = (int)threadIdx.x + 256 * j;
    if (c < n4) put4<YT>(y + 4 * c, keep[j] * sc);
  }
  for (int c = (int)threadIdx.x + 256 * FIN_REG; c < n4; c += 256) put4<YT>(y + 4 * c, sum_of(c) * sc);
}

}  // namespace

// Calls that take this path: up to 2^23 values of X, where the general path's
// passes over M and its part-filled GEMM still cost more, and no more rows
// than D, so that the partials fit the general path's workspace.  At
// D = 8192: 1 / 64 / 256 / 1024 rows take 51 / 59 / 103 / 352 us here (5.2 /
// 4.5 / 2.6 TB/s of M for the first three) and 390-420 us there; from 1536
// rows the general path is as fast (474 us, here 503).  At D = 4096: 193 us
// against ~200 at 2048 rows; at D = 1024, 30 against 70 us at 1024 rows.
constexpr int64_t kApplyFewValues = (int64_t)1 << 23;

ApplyFewPlan plan_apply_few(int64_t n_rows, int64_t D) {
  ApplyFewPlan P{};
  P.use = n_rows <= D && n_rows * D <= kApplyFewValues;
  if (!P.use) return P;
  P.xt = n_rows <= 64 ? 1 : (n_rows <= 128 ? 2 : 4);
  P.n_rb = (int)((n_rows + 64 * P.xt - 1) / (64 * P.xt));
  P.n_ct = (int)(D / FCOL);
  // The workspace is the general path's (at least 4 D^2 bytes): partials and
  // packed rows stay within that.  Up to 16 rows only one wave pair loads X:
  // packing is not worth a launch.
  const int64_t xrows = (int64_t)P.n_rb * 64 * P.xt;
  const bool pack = n_rows > 16 && 4 * n_rows + 2 * xrows <= 4 * D;
  const int64_t room = 4 * D - (pack ? 2 * xrows : 0);  // partial bytes per column, all slices
  // K-slices (whole groups of FPD stages): the count with the least modelled
  // time, in stages: whole rounds of one workgroup per CU, each the stages of
  // a slice plus ~6 to start and end, plus writing and reading one partial
  // per slice (~7 MB per stage time).
  const int64_t n_gr = (D / FKS + FPD - 1) / FPD;
  int64_t best = INT64_MAX;
  P.n_sl = 1;
  for (int64_t sl = 1; sl <= n_gr && sl <= 64 && 4 * sl * n_rows <= room; ++sl) {
    const int64_t rounds = (sl * P.n_ct * P.n_rb + 255) / 256;
    const int64_t cost = rounds * (FPD * ((n_gr + sl - 1) / sl) + 6) + sl * n_rows * D * 8 / 7000000;
    if (cost < best) {
      best = cost;
      P.n_sl = (int)sl;
    }
  }
  P.part_bytes = (size_t)P.n_sl * (size_t)n_rows * (size_t)D * 4;
  P.pack_bytes = pack ? (size_t)xrows * (size_t)D * 2 : 0;
  return P;
}

hipError_t launch_apply_few(const ApplyFewPlan& P, const void* X, int64_t n_rows, int64_t ldx,
                            int64_t D, const float* M, int y_dtype, void* Y, int64_t ldy, int unit,
                            void* ws, hipStream_t s) {
  float* part = static_cast<float*>(ws);
  const int n_units = P.n_ct * P.n_sl;
  i32x4* xpk = nullptr;
  if (P.pack_bytes) {
    xpk = reinterpret_cast<i32x4*>(static_cast<char*>(ws) + P.part_bytes);
    const int n_tiles = 4 * P.n_rb * P.xt;
    hipLaunchKernelGGL(apply_few_pack_kernel, dim3((unsigned)(n_tiles * ((D + 127) / 128))), dim3(256), 0,
                       s, (const _Float16*)X, n_rows, ldx, D, n_tiles, xpk);
  }
  dim3 grid((unsigned)((n_units + 7) / 8 * 8 * P.n_rb)), block(512);
#define ATTR_AF(T, N)                                                                              \
  hipLaunchKernelGGL((apply_few_kernel<T, N>), grid, block, 0, s, (const _Float16*)X, n_rows, ldx, D, \
                     (const i32x4*)xpk, M, P.n_ct, P.n_sl, P.n_rb, n_units, part)
  if (P.xt == 1) ATTR_AF(1, true);
  else if (P.xt == 2) ATTR_AF(2, true);
  else if (P.n_rb == 1) ATTR_AF(4, true);
  else ATTR_AF(4, false);
#undef ATTR_AF
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  block = dim3(256);
  if (y_dtype == 2)
    hipLaunchKernelGGL(apply_few_final_kernel<_Float16>, dim3((unsigned)n_rows), block, 0, s,
                       (const float*)part, P.n_sl, n_rows, D, unit, (_Float16*)Y, ldy);
  else
    hipLaunchKernelGGL(apply_few_final_kernel<float>, dim3((unsigned)n_rows), block, 0, s,
                       (const float*)part, P.n_sl, n_rows, D, unit, (float*)Y, ldy);
  return hipGetLastError();
}

}  // namespace attr
