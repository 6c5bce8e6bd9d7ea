// Row-wise processing of compressed gradient rows and the diagonal
// second-moment accumulator.
//
// rowscale: y = unit_normalise(m .* x) cast to the store dtype (the
// "processing" step of section "Attribution Pipelines": unit normalisation
// and the diagonal preconditioner; grad-cosine in the method-family table).
// One workgroup per row or two rows; they stay in registers between the norm
// and the write, so X is read once and Y written once (HBM-bound).
//
// colsumsq: h_j += sum_i x_ij^2, the diagonal of the second moment G^T G.
// Column blocks x row panels; fp32 sums over 8-row groups are added into an
// fp64 accumulator per thread, panel sums are combined in fp64 in panel
// order and rounded once into h (deterministic, no atomics).
#include "common.h"
#include "kernels.h"

namespace attr {
namespace {

template <typename T>
__device__ inline void load8(const T* p, float (&v)[8]);
template <>
__device__ inline void load8<float>(const float* p, float (&v)[8]) {
  const f32x4 a = *(const f32x4*)p;
  const f32x4 b = *(const f32x4*)(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
template <>
__device__ inline void load8<_Float16>(const _Float16* p, float (&v)[8]) {
  const f16x8 a = *(const f16x8*)p;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (float)a[e];
}

// Streaming (non-temporal) load of a row chunk read exactly once.
template <typename T>
__device__ inline void load8_nt(const T* p, float (&v)[8]);
template <>
__device__ inline void load8_nt<float>(const float* p, float (&v)[8]) {
  const f32x4 a = __builtin_nontemporal_load((const f32x4*)p);
  const f32x4 b = __builtin_nontemporal_load((const f32x4*)(p + 4));
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
  v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
template <>
__device__ inline void load8_nt<_Float16>(const _Float16* p, float (&v)[8]) {
  const f16x8 a = __builtin_nontemporal_load((const f16x8*)p);
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (float)a[e];
}

template <typename T>
__device__ inline void store8(T* p, const float (&v)[8]);
template <>
__device__ inline void store8<float>(float* p, const float (&v)[8]) {
  __builtin_nontemporal_store(f32x4{v[0], v[1], v[2], v[3]}, (f32x4*)p);
  __builtin_nontemporal_store(f32x4{v[4], v[5], v[6], v[7]}, (f32x4*)(p + 4));
}
template <>
__device__ inline void store8<_Float16>(_Float16* p, const float (&v)[8]) {
  f16x8 a;
#pragma unroll
  for (int e = 0; e < 8; ++e) a[e] = (_Float16)v[e];
  __builtin_nontemporal_store(a, (f16x8*)p);
}

__device__ inline float block_sum256(float v, float* sh) {
  v = wave_sum(v);
  const int wave = threadIdx.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[wave] = v;
  __syncthreads();
  return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

__device__ inline float row_scale(float ss, int unit) {
  if (!unit) return 1.f;
  return ss > 0.f ? (float)(1.0 / sqrt((double)ss)) : 0.f;
}

// CH > 0: up to CH chunks of 8 elements per thread stay in registers.
// CH == 0: any width, two passes over the row (second pass hits cache).
// seg_e (with row_ss): X holds y 2^-e per 128-column segment, e = seg_e[r * n_ss
// + segment]; the scale of such a segment is 2^e / ||y||.
template <typename TX, typename TY, int CH>
__global__ __launch_bounds__(256) void rowscale_kernel(const TX* __restrict__ X, int64_t ldx,
                                                       int64_t D, const float* __restrict__ m,
                                                       int unit, const float* __restrict__ row_ss,
                                                       const int8_t* __restrict__ seg_e,
                                                       int64_t n_ss, TY* Y, int64_t ldy) {
  __shared__ float sh[4];
  const int64_t r = blockIdx.x;
  const TX* x = X + r * ldx;
  TY* y = Y + r * ldy;
  const int n8 = (int)(D / 8);
  float ss = 0.f;
  if (CH > 0) {
    float v[CH > 0 ? CH : 1][8];
#pragma unroll
    for (int j = 0; j < (CH > 0 ? CH : 1); ++j) {
      const int ch = threadIdx.x + j * 256;
      if (ch < n8) {
        load8_nt<TX>(x + (int64_t)ch * 8, v[j]);
        if (m) {
          float mm[8];
          load8<float>(m + (int64_t)ch * 8, mm);
#pragma unroll
          for (int e = 0; e < 8; ++e) v[j][e] *= mm[e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += v[j][e] * v[j][e];
      }
    }
    if (row_ss) {
      ss = 0.f;
      for (int64_t p = 0; p < n_ss; ++p) ss += row_ss[r * n_ss + p];
    } else if (unit) {
      ss = block_sum256(ss, sh);
    }
    const float sc = row_scale(ss, unit);
#pragma unroll
    for (int j = 0; j < (CH > 0 ? CH : 1); ++j) {
      const int ch = threadIdx.x + j * 256;
      if (ch < n8) {
        const float scj = seg_e ? ldexpf(sc, (int)seg_e[r * n_ss + (ch >> 4)]) : sc;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[j][e] *= scj;
        store8<TY>(y + (int64_t)ch * 8, v[j]);
      }
    }
  } else {
    if (row_ss) {
      for (int64_t p = 0; p < n_ss; ++p) ss += row_ss[r * n_ss + p];
    } else if (unit) {
      for (int ch = threadIdx.x; ch < n8; ch += 256) {
        float v[8];
        load8<TX>(x + (int64_t)ch * 8, v);
        if (m) {
          float mm[8];
          load8<float>(m + (int64_t)ch * 8, mm);
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] *= mm[e];
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += v[e] * v[e];
      }
      ss = block_sum256(ss, sh);
    }
    const float sc = row_scale(ss, unit);
    for (int ch = threadIdx.x; ch < n8; ch += 256) {
      float v[8];
      load8<TX>(x + (int64_t)ch * 8, v);
      if (m) {
        float mm[8];
        load8<float>(m + (int64_t)ch * 8, mm);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] *= mm[e];
      }
      const float scj = seg_e ? ldexpf(sc, (int)seg_e[r * n_ss + (ch >> 4)]) : sc;
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] *= scj;
      store8<TY>(y + (int64_t)ch * 8, v);
    }
  }
}

// Two rows per workgroup (rows 2b and 2b + 1, same column chunks per
// thread): the scale m is read once for both and twice the bytes are in
// flight per workgroup.  Same per-row arithmetic and order as above.
template <typename TX, typename TY, int CH>
__global__ __launch_bounds__(256) void rowscale2_kernel(const TX* __restrict__ X, int64_t ldx,
                                                        int64_t n_rows, int64_t D,
                                                        const float* __restrict__ m, int unit,
                                                        const float* __restrict__ row_ss,
                                                        int64_t n_ss, TY* Y, int64_t ldy) {
  __shared__ float sh[2][4];
  const int64_t r0 = 2 * (int64_t)blockIdx.x;
  const bool two = r0 + 1 < n_rows;
  const int n8 = (int)(D / 8);
  float v[2][CH][8];
  float ss[2] = {0.f, 0.f};
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int ch = threadIdx.x + j * 256;
    if (ch < n8) {
      load8_nt<TX>(X + r0 * ldx + (int64_t)ch * 8, v[0][j]);
      if (two) load8_nt<TX>(X + (r0 + 1) * ldx + (int64_t)ch * 8, v[1][j]);
    }
  }
#pragma unroll
  for (int j = 0; j < CH; ++j) {
    const int ch = threadIdx.x + j * 256;
    if (ch < n8) {
      if (m) {
        float mm[8];
        load8<float>(m + (int64_t)ch * 8, mm);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          v[0][j][e] *= mm[e];
          v[1][j][e] *= mm[e];
        }
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        ss[0] += v[0][j][e] * v[0][j][e];
        ss[1] += v[1][j][e] * v[1][j][e];
      }
    }
  }
  if (row_ss) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      ss[h] = 0.f;
      if (h == 0 || two)
        for (int64_t p = 0; p < n_ss; ++p) ss[h] += row_ss[(r0 + h) * n_ss + p];
    }
  } else if (unit) {
    const float a = wave_sum(ss[0]), b = wave_sum(ss[1]);
    if ((threadIdx.x & 63) == 0) {
      sh[0][threadIdx.x >> 6] = a;
      sh[1][threadIdx.x >> 6] = b;
    }
    __syncthreads();
    ss[0] = (sh[0][0] + sh[0][1]) + (sh[0][2] + sh[0][3]);
    ss[1] = (sh[1][0] + sh[1][1]) + (sh[1][2] + sh[1][3]);
  }
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h == 1 && !two) break;
    const float sc = row_scale(ss[h], unit);
    TY* y = Y + (r0 + h) * ldy;
#pragma unroll
    for (int j = 0; j < CH; ++j) {
      const int ch = threadIdx.x + j * 256;
      if (ch < n8) {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[h][j][e] *= sc;
        store8<TY>(y + (int64_t)ch * 8, v[h][j]);
      }
    }
  }
}

// The same for rows of more than 8192 columns: R rows per workgroup of TPR
// threads, CH chunks of 8 elements per thread and row, kept as loaded between
// the norm and the write, so that every row's loads are in flight at once; the
// scale is read once per R rows.  Bound by the memory's mixed read and write
// rate (torch's copy of a 4.9 GB tensor moves 4.9 TB/s).  Against one row per 256 threads,
// which reads 48 KB of scale with every 24 KB row: 200000 x 12288 DIAG in fp16
// 1817 -> 1730 us (5.7 TB/s), 20000 x 24096 574 -> 386 us (5.0 TB/s) and, without
// a scale, 459 -> 338 us.  Four rows, 256 threads, or a loop over rows with the
// scale in registers were no faster (1776, 1743, 1742 us).
// Raw: the 8 elements of a chunk as loaded.
template <typename T>
struct RawChunk;
template <>
struct RawChunk<float> {
  f32x4 a, b;
  __device__ inline void load(const float* p) {
    a = __builtin_nontemporal_load((const f32x4*)p);
    b = __builtin_nontemporal_load((const f32x4*)(p + 4));
  }
  __device__ inline void get(float (&v)[8]) const {
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
};
template <>
struct RawChunk<_Float16> {
  f16x8 a;
  __device__ inline void load(const _Float16* p) { a = __builtin_nontemporal_load((const f16x8*)p); }
  __device__ inline void get(float (&v)[8]) const {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (float)a[e];
  }
};

template <typename TX, typename TY, int TPR, int CH, int R, bool DIAG>
__global__ __launch_bounds__(TPR) void rowscale_rows_kernel(
    const TX* X, int64_t ldx, int64_t n_rows, int64_t D, const float* __restrict__ m, int unit,
    TY* Y, int64_t ldy) {
  constexpr int NW = TPR / 64;
  __shared__ float sh[R][NW];
  const int t = (int)threadIdx.x;
  const int n8 = (int)(D / 8);
  const int64_t r0 = (int64_t)blockIdx.x * R;
  RawChunk<TX> x[R][CH];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int j = 0; j < CH; ++j)
      if (r0 + i < n_rows && t + j * TPR < n8) x[i][j].load(X + (r0 + i) * ldx + (int64_t)(t + j * TPR) * 8);
  float mm[DIAG ? CH : 1][8];
  if (DIAG) {
#pragma unroll
    for (int j = 0; j < CH; ++j)
      if (t + j * TPR < n8) load8<float>(m + (int64_t)(t + j * TPR) * 8, mm[DIAG ? j : 0]);
  }
  auto value = [&](int i, int j, float (&v)[8]) {
    x[i][j].get(v);
    if (DIAG) {
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] *= mm[DIAG ? j : 0][e];
    }
  };
  float ss[R];
#pragma unroll
  for (int i = 0; i < R; ++i) ss[i] = 0.f;
  if (unit) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
#pragma unroll
      for (int j = 0; j < CH; ++j)
        if (r0 + i < n_rows && t + j * TPR < n8) {
          float v[8];
          value(i, j, v);
#pragma unroll
          for (int e = 0; e < 8; ++e) ss[i] += v[e] * v[e];
        }
      ss[i] = wave_sum(ss[i]);
      if ((t & 63) == 0) sh[i][t >> 6] = ss[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < R; ++i) {
      ss[i] = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) ss[i] += sh[i][w];
    }
  }
#pragma unroll
  for (int i = 0; i < R; ++i) {
    if (r0 + i >= n_rows) break;  // uniform
    const float sc = row_scale(ss[i], unit);
#pragma unroll
    for (int j = 0; j < CH; ++j)
      if (t + j * TPR < n8) {
        float v[8];
        value(i, j, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] *= sc;
        store8<TY>(Y + (r0 + i) * ldy + (int64_t)(t + j * TPR) * 8, v);
      }
  }
}

template <typename TX, typename TY>
hipError_t launch_rowscale_t(const void* X, int64_t ldx, int64_t n_rows, int64_t D,
                             const float* m, int unit, const float* row_ss, const int8_t* seg_e,
                             int64_t n_ss, void* Y, int64_t ldy, hipStream_t s) {
  const int64_t n8 = D / 8;
  const TX* x = (const TX*)X;
  TY* y = (TY*)Y;
#define ATTR_RR(T, C, R, DG)                                                                       \
  {                                                                                                \
    hipLaunchKernelGGL((rowscale_rows_kernel<TX, TY, T, C, R, DG>), dim3((unsigned)((n_rows + R - 1) / R)), \
                       dim3(T), 0, s, x, ldx, n_rows, D, m, unit, y, ldy);                         \
    return hipGetLastError();                                                                      \
  }
  // Which calls take rowscale_rows_kernel (general / this kernel, us; one and two rows
  // per workgroup give the same bits, so a row's do not depend on the other rows).
  constexpr bool XF = sizeof(TX) == 4, YF = sizeof(TY) == 4;
  if (!row_ss && n8 <= 4096) {
    // With a scale: fp32 rows to fp32 do not gain (60000 x 16384 1531 / 1668).  One row
    // per workgroup while there are few (general / one / two): 64 x 24096 fp16 9.7 / 5.8 /
    // 8.2, fp32 to fp16 7.7 / 6.6 / 11.9; 1000 x 12288 fp16 11.4 / 12.9 / 11.1; 20000 x
    // 12288 fp32 to fp16 291 / 274 / 267.  fp32 to fp16 stays up to 11% behind for 300
    // to 700 rows (part of a second wave of workgroups: 512 x 12288 8.1 / 8.7 / 10.6).
    if constexpr (!(XF && YF)) {
      if (m && n8 > 1024) {  // (up to 1024: the two-row kernel below)
        const bool narrow = n8 <= 2048;
        const int64_t one = XF ? (narrow ? 8192 : 1024) : YF ? (narrow ? 10000 : n_rows + 1) : narrow ? 512 : 256;
        if (n_rows <= one) {
          if (n8 <= 1536) ATTR_RR(512, 3, 1, true)
          if (n8 <= 2048) ATTR_RR(512, 4, 1, true)
          if (n8 <= 3072) ATTR_RR(1024, 3, 1, true)
          ATTR_RR(1024, 4, 1, true)
        }
        if (n8 <= 1536) ATTR_RR(512, 3, 2, true)
        if (n8 <= 2048) ATTR_RR(512, 4, 2, true)
        if constexpr (XF == YF || XF) {
          if (n8 <= 3072) ATTR_RR(1024, 3, 2, true)
          ATTR_RR(1024, 4, 2, true)
        }
      }
    }
    // Without a scale one row per 256 threads is as fast up to 16384 columns, and
    // faster for large stores of fp16 rows to fp32 (20000 x 32768 822 / 1157).
    if constexpr (XF || !YF) {
      if (!m && n8 > 2048) {
        if (n8 <= 3072) ATTR_RR(1024, 3, 1, false)
        ATTR_RR(1024, 4, 1, false)
      }
    }
  }
#undef ATTR_RR
  dim3 grid((unsigned)n_rows), block(256);
#define ATTR_RS(CH) \
  hipLaunchKernelGGL((rowscale_kernel<TX, TY, CH>), grid, block, 0, s, x, ldx, D, m, unit, row_ss, \
                     seg_e, n_ss, y, ldy)
  if (m && !seg_e && n8 <= 1024 && n_rows >= 2) {  // the scale is read once per two rows
    dim3 g2((unsigned)((n_rows + 1) / 2));
#define ATTR_R2(CH)                                                                        \
  hipLaunchKernelGGL((rowscale2_kernel<TX, TY, CH>), g2, block, 0, s, x, ldx, n_rows, D, m, \
                     unit, row_ss, n_ss, y, ldy)
    if (n8 <= 256) ATTR_R2(1);
    else if (n8 <= 512) ATTR_R2(2);
    else ATTR_R2(4);
#undef ATTR_R2
    return hipGetLastError();
  }
  if (n8 <= 256) ATTR_RS(1);
  else if (n8 <= 512) ATTR_RS(2);
  else if (n8 <= 1024) ATTR_RS(4);
  else if (n8 <= 2048) ATTR_RS(8);
  else if (n8 <= 4096) ATTR_RS(16);
  else ATTR_RS(0);
#undef ATTR_RS
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// colsumsq
// ---------------------------------------------------------------------------
constexpr int kColThreads = 256;
// columns per workgroup: one 16-byte load per thread and row (fp32 rows in two
// 16-byte halves per thread touched every cache line twice: 247043 x 4544 in
// fp32 895 -> 745 us, 4.9 -> 6.0 TB/s)
constexpr int col_block(int elem_bytes) { return kColThreads * (16 / elem_bytes); }
constexpr int kColRows = 8;  // rows in flight per thread (16: no faster)

// VE: elements per 16-byte load
template <typename TX, int VE>
__global__ __launch_bounds__(256) void colsumsq_kernel(const TX* __restrict__ X, int64_t ldx,
                                                       int64_t n_rows, int64_t D,
                                                       int64_t rows_per_panel,
                                                       double* __restrict__ part) {
  typedef TX vec __attribute__((ext_vector_type(VE)));
  const int64_t c0 = ((int64_t)blockIdx.x * kColThreads + threadIdx.x) * VE;
  const int64_t panel = blockIdx.y;
  if (c0 >= D) return;
  const int64_t r0 = panel * rows_per_panel;
  int64_t r1 = r0 + rows_per_panel;
  r1 = r1 > n_rows ? n_rows : r1;
  double acc[VE];
#pragma unroll
  for (int e = 0; e < VE; ++e) acc[e] = 0.0;
  auto load = [&](int64_t r) {
    return __builtin_bit_cast(vec, __builtin_nontemporal_load((const i32x4*)(X + r * ldx + c0)));
  };
  int64_t r = r0;
  for (; r + kColRows <= r1; r += kColRows) {
    vec v[kColRows];
#pragma unroll
    for (int u = 0; u < kColRows; ++u) v[u] = load(r + u);
    // fp32 sums over 8 rows
#pragma unroll
    for (int e = 0; e < VE; ++e) {
      float f = 0.f;
#pragma unroll
      for (int u = 0; u < kColRows; ++u) f += (float)v[u][e] * (float)v[u][e];
      acc[e] += (double)f;
    }
  }
  for (; r < r1; ++r) {
    const vec v = load(r);
#pragma unroll
    for (int e = 0; e < VE; ++e) acc[e] += (double)((float)v[e] * (float)v[e]);
  }
#pragma unroll
  for (int e = 0; e < VE; ++e) part[panel * D + c0 + e] = acc[e];
}

// h_j += sum over panels of part[p][j]: a workgroup takes 64 columns, wave w of
// nw sums panels p = w (mod nw) in increasing order (each panel read as 512
// contiguous bytes per wave), and the sums are added in wave order: a fixed
// order, so the result is deterministic.  Sixteen waves from 512 panels on (few
// columns, so few workgroups: with four, the 2048 panels of 1672 columns were a
// chain of 128 load rounds on 27 workgroups, 45 us).
constexpr int kFinWaves = 16;
__global__ __launch_bounds__(64 * kFinWaves) void colsumsq_final_kernel(const double* __restrict__ part,
                                                                        int64_t n_panels, int64_t D,
                                                                        float* __restrict__ H) {
  __shared__ double red[kFinWaves][64];
  const int w = threadIdx.x >> 6, c = threadIdx.x & 63, nw = blockDim.x >> 6;
  const int64_t j = (int64_t)blockIdx.x * 64 + c;
  double s = 0.0;
  if (j < D) {
    int64_t p = w;
    for (; p + 3 * nw < n_panels; p += 4 * nw) {
      double v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = part[(p + u * nw) * D + j];
#pragma unroll
      for (int u = 0; u < 4; ++u) s += v[u];
    }
    for (; p < n_panels; p += nw) s += part[p * D + j];
  }
  red[w][c] = s;
  __syncthreads();
  if (w == 0 && j < D) {
    for (int u = 1; u < nw; ++u) s += red[u][c];
    H[j] = (float)((double)H[j] + s);
  }
}

}  // namespace

hipError_t launch_rowscale(int x_dtype, int y_dtype, const void* X, int64_t ldx,
                           int64_t n_rows, int64_t D, const float* m, int unit,
                           const float* row_ss, const int8_t* seg_e, int64_t n_ss, void* Y,
                           int64_t ldy, hipStream_t s) {
  if (x_dtype == 0 && y_dtype == 0)
    return launch_rowscale_t<float, float>(X, ldx, n_rows, D, m, unit, row_ss, seg_e, n_ss, Y, ldy, s);
  if (x_dtype == 0 && y_dtype == 2)
    return launch_rowscale_t<float, _Float16>(X, ldx, n_rows, D, m, unit, row_ss, seg_e, n_ss, Y, ldy,
                                              s);
  if (x_dtype == 2 && y_dtype == 0)
    return launch_rowscale_t<_Float16, float>(X, ldx, n_rows, D, m, unit, row_ss, seg_e, n_ss, Y, ldy,
                                              s);
  return launch_rowscale_t<_Float16, _Float16>(X, ldx, n_rows, D, m, unit, row_ss, seg_e, n_ss, Y,
                                               ldy, s);
}

int colsumsq_panels(int64_t n_rows, int64_t D) {
  const int64_t ncb = (D + col_block(2) - 1) / col_block(2);
  int64_t panels = (2048 + ncb - 1) / ncb;
  const int64_t max_by_rows = (n_rows + 63) / 64;  // at least 64 rows per panel
  if (panels > max_by_rows) panels = max_by_rows;
  if (panels < 1) panels = 1;
  if (panels > 65535) panels = 65535;
  return (int)panels;
}

hipError_t launch_colsumsq(int x_dtype, const void* X, int64_t ldx, int64_t n_rows, int64_t D,
                           float* H, double* part, hipStream_t s) {
  const int panels = colsumsq_panels(n_rows, D);
  const int64_t rpp = (n_rows + panels - 1) / panels;
  const int cb = col_block(x_dtype == 0 ? 4 : 2);
  dim3 grid((unsigned)((D + cb - 1) / cb), (unsigned)panels), block(kColThreads);
  if (x_dtype == 0)
    hipLaunchKernelGGL((colsumsq_kernel<float, 4>), grid, block, 0, s, (const float*)X, ldx, n_rows, D, rpp, part);
  else if (x_dtype == 1)
    hipLaunchKernelGGL((colsumsq_kernel<__bf16, 8>), grid, block, 0, s, (const __bf16*)X, ldx, n_rows, D, rpp, part);
  else
    hipLaunchKernelGGL((colsumsq_kernel<_Float16, 8>), grid, block, 0, s, (const _Float16*)X, ldx, n_rows, D, rpp, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  dim3 g2((unsigned)((D + 63) / 64));
  hipLaunchKernelGGL(colsumsq_final_kernel, g2, dim3(panels >= 512 ? 64 * kFinWaves : 256), 0, s, (const double*)part, (int64_t)panels, D, H);
  return hipGetLastError();
}

}  // namespace attr
