// LayerNorm forward and backward over rows of width d (bf16 or fp32 rows, fp32 statistics).
//   forward:  mu = mean(x), var = mean((x-mu)^2) (biased), rstd = 1/sqrt(var+eps),
//             y = (x-mu)*rstd*gamma + beta; mu and rstd are saved per row.
//   backward: g = dy*gamma; dx = rstd*(g - mean(g) - xhat*mean(g*xhat)) (+ add);
//             dgamma = sum_rows dy*xhat; dbeta = sum_rows dy.
// One wavefront owns a row (in the backward pass only up to 1024 elements; wider rows are shared by the four
// waves of a workgroup): each lane keeps its 16-byte chunks of the row in registers, statistics are
// butterfly reductions over the 64 lanes (wave_math.h, fixed order).  The column sums of the backward pass are
// accumulated per workgroup over a fixed range of rows, written as partial sums, and added over
// workgroups in index order by a second kernel: no atomics, so results do not depend on timing.
#include "kernels.h"
#include "wave_math.h"

namespace hydra {
namespace {

// MAXC = 8-element chunks a lane may own: d <= 8*64*MAXC (2 -> 1024, 4 -> 2048, 8 -> 4096)
constexpr int LN_ROWS_PER_WG = 64;  // rows per workgroup in the backward pass
// Rows wider than this are taken by a whole workgroup at a time (ln_bwd_wide_kernel), 32 rows per workgroup.
constexpr int LN_WAVE_ROW_MAX = 1024;
constexpr int LN_WIDE_ROWS_PER_WG = 32;

__device__ __forceinline__ bf16_t f2bf(float v) {
  __bf16 h = (__bf16)v;
  return __builtin_bit_cast(bf16_t, h);
}
// two floats -> two bf16 in one word (round to nearest even): one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  typedef __attribute__((ext_vector_type(2))) float f32x2_t;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
  const f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

template <typename T>
__device__ __forceinline__ void ld8(const T* p, float (&v)[8]);
template <>
__device__ __forceinline__ void ld8<float>(const float* p, float (&v)[8]) {
  float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
template <>
__device__ __forceinline__ void ld8<bf16_t>(const bf16_t* p, float (&v)[8]) {
  uint4 a = *reinterpret_cast<const uint4*>(p);
  uint32_t w[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}
// the 16-byte pieces of 8 elements as they lie in memory -> 8 floats
template <typename T>
__device__ __forceinline__ void unpack8(const uint4 (&raw)[sizeof(T) == 2 ? 1 : 2], float (&v)[8]) {
  if constexpr (sizeof(T) == 2) {
    const uint32_t w[4] = {raw[0].x, raw[0].y, raw[0].z, raw[0].w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[2 * q] = __uint_as_float(w[q] << 16);
      v[2 * q + 1] = __uint_as_float(w[q] & 0xffff0000u);
    }
  } else {
    v[0] = __uint_as_float(raw[0].x); v[1] = __uint_as_float(raw[0].y); v[2] = __uint_as_float(raw[0].z); v[3] = __uint_as_float(raw[0].w);
    v[4] = __uint_as_float(raw[1].x); v[5] = __uint_as_float(raw[1].y); v[6] = __uint_as_float(raw[1].z); v[7] = __uint_as_float(raw[1].w);
  }
}
template <typename T>
__device__ __forceinline__ void st8(T* p, const float (&v)[8]);
template <>
__device__ __forceinline__ void st8<float>(float* p, const float (&v)[8]) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
  *reinterpret_cast<float4*>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
template <>
__device__ __forceinline__ void st8<bf16_t>(bf16_t* p, const float (&v)[8]) {
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) w[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
  *reinterpret_cast<uint4*>(p) = make_uint4(w[0], w[1], w[2], w[3]);
}

// R = rows per wave.  Their loads are all issued before the first is reduced, and gamma and beta (fp32: four times the bytes of a
// 16-bit row) are read once for the R rows.  A row's result does not depend on R.  Four rows (two of fp32) where that still
// leaves every SIMD eight waves: 4 x [16384, 768] bf16 49 -> 34 us (5.9 TB/s); fewer rows stay one to a wave.
template <typename T, int LN_MAXC, int R>
__global__ __launch_bounds__(256) void ln_fwd_kernel(const LnArgs a) {
  const int g = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int row0 = (blockIdx.x * 4 + wave) * R;
  if (row0 >= a.rows) return;
  const int nrow = min(R, a.rows - row0);
  const T* x = static_cast<const T*>(a.x[g]) + (size_t)row0 * a.ld;
  T* y = static_cast<T*>(a.y[g]) + (size_t)row0 * a.ld;
  const int nch = a.d >> 3;
  constexpr int RW = sizeof(T) == 2 ? 1 : 2;  // 16-byte pieces per 8 elements
  uint4 raw[R][LN_MAXC][RW];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int i = 0; i < LN_MAXC; ++i) {
      const int c = lane + 64 * i;
#pragma unroll
      for (int q = 0; q < RW; ++q) {
        raw[r][i][q] = make_uint4(0, 0, 0, 0);
        if (c < nch && r < nrow) raw[r][i][q] = reinterpret_cast<const uint4*>(x + (size_t)r * a.ld)[c * RW + q];
      }
    }
  const float* gamma = a.gamma[g];
  const float* beta = a.beta[g];
  float ga[LN_MAXC][8], be[LN_MAXC][8];
#pragma unroll
  for (int i = 0; i < LN_MAXC; ++i) {
    const int c = lane + 64 * i;
    if (c < nch) {
      ld8<float>(gamma + 8 * c, ga[i]);
      ld8<float>(beta + 8 * c, be[i]);
    }
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (r >= nrow) break;
    float v[LN_MAXC][8];
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < LN_MAXC; ++i) {
      unpack8<T>(raw[r][i], v[i]);
      if (lane + 64 * i < nch) {
#pragma unroll
        for (int e = 0; e < 8; ++e) s += v[i][e];
      }
    }
    const float mu = wave_sum(s) / (float)a.d;
    float q = 0.f;
#pragma unroll
    for (int i = 0; i < LN_MAXC; ++i)
      if (lane + 64 * i < nch) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float t = v[i][e] - mu;
          q += t * t;
        }
      }
    const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)a.d + a.eps);
#pragma unroll
    for (int i = 0; i < LN_MAXC; ++i) {
      const int c = lane + 64 * i;
      if (c < nch) {
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (v[i][e] - mu) * rstd * ga[i][e] + be[i][e];
        st8<T>(y + (size_t)r * a.ld + 8 * c, o);
      }
    }
    if (lane == 0) {
      a.mean[g][row0 + r] = mu;
      a.rstd[g][row0 + r] = rstd;
    }
  }
}

// dx and per-workgroup partial column sums, rows of up to 1024 elements.  Workgroup b owns rows [b*64, b*64+64); wave w of NW takes
// rows b*64 + w, + NW, ...; partial sums go to part[g][b][2][d].
// A wave takes its rows in batches of NB: all loads of a batch (x, dy, the additive term, the statistics) are issued
// before its first row is reduced, so that the batch costs one round trip to memory.  Small launches are bound by a
// wave's serial rows, large ones by memory; 4 waves of 16 rows, the next row's loads ahead of the current one's
// reduction, against this form (us): 4 x [1024, 256] bf16 18.1 | 8.7, 4 x [4096, 512] 22 | 13.8, 4 x [1024, 768] 20.7 | 14.5,
// 4 x [16384, 512] 51 | 46, 4 x [16384, 768] 87 | 86 (4.7 TB/s: a device copy's rate), fp32 165 | 161.
template <typename T, int LN_MAXC, int NW, int NB>
__global__ __launch_bounds__(NW * 64) void ln_bwd_kernel(const LnBwdArgs a) {
  extern __shared__ float red[];  // [NW][2][d]
  const int g = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int nch = a.d >> 3;
  constexpr int RW = sizeof(T) == 2 ? 1 : 2;  // 16-byte pieces per 8 elements
  static_assert(LN_ROWS_PER_WG % (NW * NB) == 0, "whole batches");
  const int row0 = blockIdx.x * LN_ROWS_PER_WG + wave;
  const T* X = static_cast<const T*>(a.x[g]);
  const T* DY = static_cast<const T*>(a.dy[g]);
  const T* ADD = static_cast<const T*>(a.add[g]);
  T* DX = static_cast<T*>(a.dx[g]);
  const float* mean = a.mean[g];
  const float* rs = a.rstd[g];
  const float* gamma = a.gamma[g];
  float ga[LN_MAXC][8], sg[LN_MAXC][8], sb[LN_MAXC][8];
#pragma unroll
  for (int i = 0; i < LN_MAXC; ++i) {
    const int c = lane + 64 * i;
#pragma unroll
    for (int e = 0; e < 8; ++e) sg[i][e] = sb[i][e] = ga[i][e] = 0.f;
    if (c < nch) ld8<float>(gamma + 8 * c, ga[i]);
  }
  for (int r0 = 0; r0 < LN_ROWS_PER_WG; r0 += NW * NB) {
    if (row0 + r0 >= a.rows) break;
    uint4 rx[NB][LN_MAXC][RW], rdy[NB][LN_MAXC][RW], radd[NB][LN_MAXC][RW];
    float mu[NB], rstd[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int row = row0 + r0 + b * NW;
      const bool live = row < a.rows;
      const size_t o = (size_t)(live ? row : row0) * a.ld;
      mu[b] = live ? mean[row] : 0.f;
      rstd[b] = live ? rs[row] : 0.f;
#pragma unroll
      for (int i = 0; i < LN_MAXC; ++i) {
        const int c = lane + 64 * i;
        if (live && c < nch) {
#pragma unroll
          for (int q = 0; q < RW; ++q) {
            rx[b][i][q] = reinterpret_cast<const uint4*>(X + o)[c * RW + q];
            rdy[b][i][q] = reinterpret_cast<const uint4*>(DY + o)[c * RW + q];
            if (ADD) radd[b][i][q] = reinterpret_cast<const uint4*>(ADD + o)[c * RW + q];
          }
        }
      }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int row = row0 + r0 + b * NW;
      if (row >= a.rows) break;
      float xh[LN_MAXC][8], gg[LN_MAXC][8];
      float s1 = 0.f, s2 = 0.f;
#pragma unroll
      for (int i = 0; i < LN_MAXC; ++i) {
        if (lane + 64 * i < nch) {
          float xv[8], dv[8];
          unpack8<T>(rx[b][i], xv);
          unpack8<T>(rdy[b][i], dv);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            xh[i][e] = (xv[e] - mu[b]) * rstd[b];
            gg[i][e] = dv[e] * ga[i][e];
            s1 += gg[i][e];
            s2 += gg[i][e] * xh[i][e];
            sg[i][e] += dv[e] * xh[i][e];
            sb[i][e] += dv[e];
          }
        }
      }
      const float c1 = wave_sum(s1) / (float)a.d, c2 = wave_sum(s2) / (float)a.d;
#pragma unroll
      for (int i = 0; i < LN_MAXC; ++i) {
        const int c = lane + 64 * i;
        if (c < nch) {
          float o[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = rstd[b] * (gg[i][e] - c1 - xh[i][e] * c2);
          if (ADD) {
            float av[8];
            unpack8<T>(radd[b][i], av);
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] += av[e];
          }
          st8<T>(DX + (size_t)row * a.ld + 8 * c, o);
        }
      }
    }
  }
  // the waves' partial sums are added in wave order
#pragma unroll
  for (int i = 0; i < LN_MAXC; ++i) {
    const int c = lane + 64 * i;
    if (c < nch) {
      st8<float>(&red[(wave * 2 + 0) * a.d + 8 * c], sg[i]);
      st8<float>(&red[(wave * 2 + 1) * a.d + 8 * c], sb[i]);
    }
  }
  __syncthreads();
  float* part = a.part[g] + (size_t)blockIdx.x * 2 * a.d;
  for (int j = threadIdx.x; j < 2 * a.d; j += NW * 64) {  // red is [wave][2 d]
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += red[w * 2 * a.d + j];
    part[j] = t;
  }
}

// Small launches: one kernel instead of two.  The row statistics are inputs here, so the column sums need nothing from the
// rows' own pass: workgroups past the row blocks add up 32 columns each over all rows, straight from x and dy (which
// the row blocks read at the same time), instead of partial sums that a second launch collects.  Row blocks: 16 waves,
// one row each.  Column blocks: thread (row group, chunk of 8 columns) adds every 256th row in ascending order, the row
// groups of a wave are added by a butterfly and the 16 waves in wave order.
// Two launches | this one, us: 4 x [1024, 256] bf16 8.9 + 2.8 | 7.0, 4 x [152, 256] 8.4 + 2.8 | 4.5, 4 x [1024, 768] 14.6 + 3.9 |
// 11.0, fp32 4 x [1024, 256] 9.2 + 2.8 | 7.9, and a launch gap less.  A column block reads its columns of all rows through one
// compute unit, which sets the limit: 4 x [2048, 256] 9.4 + 2.8 | 10.7, 8 x [2048, 512] 13.8 + 3.9 | 25.6.
constexpr int LN_SMALL_ROWS = 1280, LN_SMALL_COLS = 32;
template <typename T, int LN_MAXC>
__global__ __launch_bounds__(1024) void ln_bwd_small_kernel(const LnBwdArgs a, int row_blocks) {
  __shared__ float red[16][2][LN_SMALL_COLS];
  const int g = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  constexpr int RW = sizeof(T) == 2 ? 1 : 2;  // 16-byte pieces per 8 elements
  const T* X = static_cast<const T*>(a.x[g]);
  const T* DY = static_cast<const T*>(a.dy[g]);
  const float* mean = a.mean[g];
  const float* rs = a.rstd[g];
  if ((int)blockIdx.x < row_blocks) {
    const int row = blockIdx.x * 16 + wave;
    if (row >= a.rows) return;
    const T* ADD = static_cast<const T*>(a.add[g]);
    const float* gamma = a.gamma[g];
    const int nch = a.d >> 3;
    const size_t o = (size_t)row * a.ld;
    uint4 rx[LN_MAXC][RW], rdy[LN_MAXC][RW], radd[LN_MAXC][RW];
    float ga[LN_MAXC][8];
    const float mu = mean[row], rstd = rs[row];
#pragma unroll
    for (int i = 0; i < LN_MAXC; ++i) {
      const int c = lane + 64 * i;
      if (c < nch) {
#pragma unroll
        for (int q = 0; q < RW; ++q) {
          rx[i][q] = reinterpret_cast<const uint4*>(X + o)[c * RW + q];
          rdy[i][q] = reinterpret_cast<const uint4*>(DY + o)[c * RW + q];
          if (ADD) radd[i][q] = reinterpret_cast<const uint4*>(ADD + o)[c * RW + q];
        }
        ld8<float>(gamma + 8 * c, ga[i]);
      }
    }
    float xh[LN_MAXC][8], gg[LN_MAXC][8];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int i = 0; i < LN_MAXC; ++i)
      if (lane + 64 * i < nch) {
        float xv[8], dv[8];
        unpack8<T>(rx[i], xv);
        unpack8<T>(rdy[i], dv);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          xh[i][e] = (xv[e] - mu) * rstd;
          gg[i][e] = dv[e] * ga[i][e];
          s1 += gg[i][e];
          s2 += gg[i][e] * xh[i][e];
        }
      }
    const float c1 = wave_sum(s1) / (float)a.d, c2 = wave_sum(s2) / (float)a.d;
#pragma unroll
    for (int i = 0; i < LN_MAXC; ++i) {
      const int c = lane + 64 * i;
      if (c < nch) {
        float out[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) out[e] = rstd * (gg[i][e] - c1 - xh[i][e] * c2);
        if (ADD) {
          float av[8];
          unpack8<T>(radd[i], av);
#pragma unroll
          for (int e = 0; e < 8; ++e) out[e] += av[e];
        }
        st8<T>(static_cast<T*>(a.dx[g]) + o + 8 * c, out);
      }
    }
    return;
  }
  const int col0 = ((int)blockIdx.x - row_blocks) * LN_SMALL_COLS, c = col0 / 8 + (tid & 3);  // chunk of 8 columns
  const bool live = 8 * c < a.d;
  float sg[8], sb[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) sg[e] = sb[e] = 0.f;
  constexpr int NB = 4;  // rows whose loads are in flight together
  for (int r0 = tid >> 2; r0 < a.rows; r0 += 256 * NB) {
    uint4 rx[NB][RW], rdy[NB][RW];
    float mu[NB], rstd[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const int row = r0 + 256 * b;
      mu[b] = rstd[b] = 0.f;
#pragma unroll
      for (int q = 0; q < RW; ++q) rx[b][q] = rdy[b][q] = make_uint4(0, 0, 0, 0);
      if (row < a.rows && live) {
        mu[b] = mean[row];
        rstd[b] = rs[row];
#pragma unroll
        for (int q = 0; q < RW; ++q) {
          rx[b][q] = reinterpret_cast<const uint4*>(X + (size_t)row * a.ld)[c * RW + q];
          rdy[b][q] = reinterpret_cast<const uint4*>(DY + (size_t)row * a.ld)[c * RW + q];
        }
      }
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      if (r0 + 256 * b >= a.rows) break;
      float xv[8], dv[8];
      unpack8<T>(rx[b], xv);
      unpack8<T>(rdy[b], dv);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        sg[e] += dv[e] * ((xv[e] - mu[b]) * rstd[b]);
        sb[e] += dv[e];
      }
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    sg[e] = wave_sum_mod4(sg[e]);
    sb[e] = wave_sum_mod4(sb[e]);
  }
  if (lane < 4) {
    st8<float>(&red[wave][0][8 * lane], sg);
    st8<float>(&red[wave][1][8 * lane], sb);
  }
  __syncthreads();
  if (tid < 2 * LN_SMALL_COLS) {
    const int which = tid / LN_SMALL_COLS, col = tid % LN_SMALL_COLS;
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) t += red[w][which][col];
    if (col0 + col < a.d) (which ? a.dbeta[g] : a.dgamma[g])[col0 + col] = t;
  }
}

// Rows of more than 1024 elements: a wave per row would need 32 or 64 values of x-hat and g per lane (one or two waves
// per SIMD, and up to 128 KB of LDS for the cross-wave column sums).  Here the four waves of a workgroup share each
// row: thread t owns chunks t, t + 256 (MAXW of them), the two row sums cross the waves through LDS (added in wave
// order), and every column belongs to exactly one thread, which adds its dgamma/dbeta terms over the workgroup's 32
// rows in row order and writes them to part[g][b][2][d] itself.  16-bit rows are prefetched one row ahead.
template <typename T, int MAXW>
__global__ __launch_bounds__(256) void ln_bwd_wide_kernel(const LnBwdArgs a) {
  __shared__ float xs[2][4][2];  // [row parity][wave][s1, s2]
  const int g = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nch = a.d >> 3;
  constexpr bool PF = sizeof(T) == 2;
  constexpr int RW = sizeof(T) == 2 ? 1 : 2;  // 16-byte pieces per 8 elements
  const float* gamma = a.gamma[g];
  float ga[MAXW][8], sg[MAXW][8], sb[MAXW][8];
#pragma unroll
  for (int i = 0; i < MAXW; ++i) {
    const int c = tid + 256 * i;
#pragma unroll
    for (int e = 0; e < 8; ++e) sg[i][e] = sb[i][e] = ga[i][e] = 0.f;
    if (c < nch) ld8<float>(gamma + 8 * c, ga[i]);
  }
  uint4 nx[MAXW][RW], ndy[MAXW][RW], nadd[MAXW][RW];
  float nmu = 0.f, nrstd = 0.f;
  const bool has_add = a.add[g] != nullptr;
  auto fetch_row = [&](int row) {
    const uint4* x = reinterpret_cast<const uint4*>(static_cast<const T*>(a.x[g]) + (size_t)row * a.ld);
    const uint4* dy = reinterpret_cast<const uint4*>(static_cast<const T*>(a.dy[g]) + (size_t)row * a.ld);
    const uint4* add = has_add ? reinterpret_cast<const uint4*>(static_cast<const T*>(a.add[g]) + (size_t)row * a.ld) : nullptr;
#pragma unroll
    for (int i = 0; i < MAXW; ++i) {
      const int c = tid + 256 * i;
      if (c < nch) {
#pragma unroll
        for (int q = 0; q < RW; ++q) {
          nx[i][q] = x[c * RW + q];
          ndy[i][q] = dy[c * RW + q];
          if (has_add) nadd[i][q] = add[c * RW + q];
        }
      }
    }
    nmu = a.mean[g][row];
    nrstd = a.rstd[g][row];
  };
  const int row0 = blockIdx.x * LN_WIDE_ROWS_PER_WG;
  const int nrow = min(LN_WIDE_ROWS_PER_WG, a.rows - row0);  // the same for every thread: the barriers below are uniform
  if (PF && nrow > 0) fetch_row(row0);
  for (int r = 0; r < nrow; ++r) {
    const int row = row0 + r;
    if (!PF) fetch_row(row);
    uint4 cx[MAXW][RW], cdy[MAXW][RW], cadd[MAXW][RW];
#pragma unroll
    for (int i = 0; i < MAXW; ++i)
#pragma unroll
      for (int q = 0; q < RW; ++q) { cx[i][q] = nx[i][q]; cdy[i][q] = ndy[i][q]; cadd[i][q] = nadd[i][q]; }
    const float mu = nmu, rstd = nrstd;
    if (PF && r + 1 < nrow) fetch_row(row + 1);
    float xh[MAXW][8], gg[MAXW][8];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int i = 0; i < MAXW; ++i) {
      const int c = tid + 256 * i;
      if (c < nch) {
        float xv[8], dv[8];
        unpack8<T>(cx[i], xv);
        unpack8<T>(cdy[i], dv);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          xh[i][e] = (xv[e] - mu) * rstd;
          gg[i][e] = dv[e] * ga[i][e];
          s1 += gg[i][e];
          s2 += gg[i][e] * xh[i][e];
          sg[i][e] += dv[e] * xh[i][e];
          sb[i][e] += dv[e];
        }
      }
    }
    // Two LDS slots by row parity and one barrier per row: a wave can write the slot of row r + 2 only after the
    // barrier of row r + 1, which every wave reaches after it has read the slot of row r.
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    if (lane == 0) {
      xs[r & 1][wave][0] = s1;
      xs[r & 1][wave][1] = s2;
    }
    __syncthreads();
    float t1 = 0.f, t2 = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      t1 += xs[r & 1][w][0];
      t2 += xs[r & 1][w][1];
    }
    const float c1 = t1 / (float)a.d, c2 = t2 / (float)a.d;
    T* dx = static_cast<T*>(a.dx[g]) + (size_t)row * a.ld;
#pragma unroll
    for (int i = 0; i < MAXW; ++i) {
      const int c = tid + 256 * i;
      if (c < nch) {
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = rstd * (gg[i][e] - c1 - xh[i][e] * c2);
        if (has_add) {
          float av[8];
          unpack8<T>(cadd[i], av);
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] += av[e];
        }
        st8<T>(dx + 8 * c, o);
      }
    }
  }
  float* part = a.part[g] + (size_t)blockIdx.x * 2 * a.d;
#pragma unroll
  for (int i = 0; i < MAXW; ++i) {
    const int c = tid + 256 * i;
    if (c < nch) {
      st8<float>(part + 8 * c, sg[i]);
      st8<float>(part + a.d + 8 * c, sb[i]);
    }
  }
}

// dgamma[col] = sum_b part[b][0][col], dbeta[col] = sum_b part[b][1][col].  A workgroup owns 16 columns; thread
// (w, col) adds the w-th of 16 contiguous ranges of b in ascending order and the 16 range sums are then added in
// ascending w: a fixed order that depends on the number of row blocks only.
__global__ __launch_bounds__(256) void ln_reduce_kernel(const LnBwdArgs a, int nblocks) {
  __shared__ float sh[16][17];
  const int g = blockIdx.y, cl = threadIdx.x & 15, w = threadIdx.x >> 4;
  const int j = blockIdx.x * 16 + cl, n2 = 2 * a.d;
  const int per = (nblocks + 15) / 16, b0 = w * per, b1 = min(nblocks, b0 + per);
  const float* part = a.part[g];
  float t = 0.f;
  if (j < n2)
    for (int b = b0; b < b1; ++b) t += part[(size_t)b * n2 + j];
  sh[w][cl] = t;
  __syncthreads();
  if (w == 0 && j < n2) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) s += sh[i][cl];
    if (j < a.d) a.dgamma[g][j] = s;
    else a.dbeta[g][j - a.d] = s;
  }
}

}  // namespace

int ln_bwd_blocks(int rows, int d) {
  const int per = d > LN_WAVE_ROW_MAX ? LN_WIDE_ROWS_PER_WG : LN_ROWS_PER_WG;
  return (rows + per - 1) / per;
}

static bool ln_shape_ok(int G, int rows, int d, int ld) {
  return G >= 1 && G <= MAXG && rows >= 1 && d >= 8 && !(d & 7) && d <= 4096 && ld >= d && !(ld & 7);
}

template <typename T, int C, int R>
static hipError_t ln_fwd_run(const LnArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((ln_fwd_kernel<T, C, R>), dim3((a.rows + 4 * R - 1) / (4 * R), a.G), dim3(256), 0, s, a);
  return hipGetLastError();
}
template <typename T>
static hipError_t ln_fwd_pick(const LnArgs& a, hipStream_t s) {
  if (a.d <= 1024) return (long)a.rows * a.G >= 32768 ? ln_fwd_run<T, 2, sizeof(T) == 2 ? 4 : 2>(a, s) : ln_fwd_run<T, 2, 1>(a, s);
  if (a.d <= 2048) return ln_fwd_run<T, 4, 1>(a, s);
  return ln_fwd_run<T, 8, 1>(a, s);
}

hipError_t launch_ln_fwd(const LnArgs& a, hipStream_t s) {
  if (!ln_shape_ok(a.G, a.rows, a.d, a.ld)) return hipErrorInvalidValue;
  return a.dtype == GEMM_F32 ? ln_fwd_pick<float>(a, s) : ln_fwd_pick<bf16_t>(a, s);
}

template <typename T>
static hipError_t ln_bwd_pick(const LnBwdArgs& a, hipStream_t s) {
  const dim3 grid(ln_bwd_blocks(a.rows, a.d), a.G);
  if (a.d <= LN_WAVE_ROW_MAX) {
    // 64 rows over 16 waves (one batch each) where a lane owns at most 8 columns, over 8 waves beyond (the cross-wave sums
    // need NW x 8 d bytes of LDS: 64 KB either way); many wide fp32 rows over 4 waves (2 x [9000, 800]
    // 49 us, over 8 waves 52.5; bf16 3 x [14483, 616] over 8 waves 52 us, over 4 57)
    if (a.d <= 512) hipLaunchKernelGGL((ln_bwd_kernel<T, 1, 16, sizeof(T) == 2 ? 4 : 2>), grid, dim3(1024), (size_t)16 * 8 * a.d, s, a);
    else if (sizeof(T) == 4 && a.rows > 4096) hipLaunchKernelGGL((ln_bwd_kernel<T, 2, 4, 2>), grid, dim3(256), (size_t)4 * 8 * a.d, s, a);
    else hipLaunchKernelGGL((ln_bwd_kernel<T, 2, 8, 2>), grid, dim3(512), (size_t)8 * 8 * a.d, s, a);
  } else if (a.d <= 2048) {
    hipLaunchKernelGGL((ln_bwd_wide_kernel<T, 1>), grid, dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL((ln_bwd_wide_kernel<T, 2>), grid, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

template <typename T>
static hipError_t ln_bwd_small_run(const LnBwdArgs& a, hipStream_t s) {
  const int row_blocks = (a.rows + 15) / 16;
  const dim3 grid(row_blocks + (a.d + LN_SMALL_COLS - 1) / LN_SMALL_COLS, a.G);
  if (a.d <= 512) hipLaunchKernelGGL((ln_bwd_small_kernel<T, 1>), grid, dim3(1024), 0, s, a, row_blocks);
  else hipLaunchKernelGGL((ln_bwd_small_kernel<T, 2>), grid, dim3(1024), 0, s, a, row_blocks);
  return hipGetLastError();
}

hipError_t launch_ln_bwd(const LnBwdArgs& a, hipStream_t s) {
  if (!ln_shape_ok(a.G, a.rows, a.d, a.ld)) return hipErrorInvalidValue;
  // by the shape of one problem alone: the order of the column sums must not depend on the group
  if (a.rows <= LN_SMALL_ROWS && a.d <= LN_WAVE_ROW_MAX)
    return a.dtype == GEMM_F32 ? ln_bwd_small_run<float>(a, s) : ln_bwd_small_run<bf16_t>(a, s);
  hipError_t e = a.dtype == GEMM_F32 ? ln_bwd_pick<float>(a, s) : ln_bwd_pick<bf16_t>(a, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(ln_reduce_kernel, dim3((2 * a.d + 15) / 16, a.G), dim3(256), 0, s, a, ln_bwd_blocks(a.rows, a.d));
  return hipGetLastError();
}

// nothing to set up: the wave-per-row kernel needs at most 64 KB of LDS
hipError_t ln_init() { return hipSuccess; }

}  // namespace hydra
