// LayerNorm forward and backward over rows of width d (bf16 or fp32 rows, fp32 statistics).
//   forward:  mu = mean(x), var = mean((x-mu)^2) (biased), rstd = 1/sqrt(var+eps),
//             y = (x-mu)*rstd*gamma + beta; mu and rstd are saved per row.
//   backward: g = dy*gamma; dx = rstd*(g - mean(g) - xhat*mean(g*xhat)) (+ add);
//             dgamma = sum_rows dy*xhat; dbeta = sum_rows dy.
// One wavefront owns a row (in the backward pass only up to 1024 elements; wider rows are shared by the four
// waves of a workgroup): each lane keeps its 16-byte chunks of the row in registers, statistics are
// butterfly reductions over the 64 lanes (wave_math.h, fixed order).  The column sums of the backward pass are
// accumulated over blocks of 64 (wide rows: 32) rows, and the blocks' partial sums are added in a fixed order, as a rule by
// a second kernel: no atomics, so results do not depend on timing.  Rows of up to 1024 elements: rows r, r + 4, ... of a
// block are one chain of multiply-adds, the four chains are added in order, then the blocks in 16 ranges and the ranges.
// Several kernels take that order, so which of them runs never changes a bit.
#include <type_traits>

#include "kernels.h"
#include "launch_rules.h"
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
// 16-bit row) are read once for the R rows.  A row's result does not depend on R: its multiply-adds are written out, not left to
// the compiler.  Four rows (two of fp32) where that still leaves every SIMD eight waves: 4 x [16384, 768] bf16 49 -> 34 us (5.9
// TB/s); fewer rows stay one to a wave.
template <typename T, int LN_MAXC, int R>
__global__ __launch_bounds__(256) void ln_fwd_kernel(const LnArgs a) {
#pragma clang fp contract(off)
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
          if (i == 0 && e == 0) {  // the first two: t0 t0 + (t1 t1, rounded)
            const float t1 = v[0][1] - mu;
            q = fmaf(t, t, t1 * t1);
          } else if (i > 0 || e > 1) {
            q = fmaf(t, t, q);
          }
        }
      }
    const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)a.d + a.eps);
#pragma unroll
    for (int i = 0; i < LN_MAXC; ++i) {
      const int c = lane + 64 * i;
      if (c < nch) {
        float o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = fmaf((v[i][e] - mu) * rstd, ga[i][e], be[i][e]);
        st8<T>(y + (size_t)r * a.ld + 8 * c, o);
      }
    }
    if (lane == 0) {
      a.mean[g][row0 + r] = mu;
      a.rstd[g][row0 + r] = rstd;
    }
  }
}

// dx and per-workgroup partial column sums, rows of up to 1024 elements.  Workgroup b owns rows [b*64, b*64+64); wave w takes rows
// b*64 + w, +4, +8, ... in ascending order; partial sums go to part[g][b][2][d].
struct LnRows {  // a problem's matrices, read from the arguments once
  const void *x, *dy, *add;
  void* dx;
  const float *mean, *rstd;
  int d, ld;
};
template <typename T, int C, int W = 64>
struct LnRow {  // one row's operands as they lie in memory: chunks lane, lane + W, ...
  static constexpr int RW = sizeof(T) == 2 ? 1 : 2;  // 16-byte pieces per 8 elements
  uint4 x[C][RW], dy[C][RW], add[C][RW];
  float mu, rstd;
  __device__ __forceinline__ void fetch(const LnBwdArgs& a, int g, int row, int lane, int nch) {
    const uint4* px = reinterpret_cast<const uint4*>(static_cast<const T*>(a.x[g]) + (size_t)row * a.ld);
    const uint4* pd = reinterpret_cast<const uint4*>(static_cast<const T*>(a.dy[g]) + (size_t)row * a.ld);
    const uint4* pa = reinterpret_cast<const uint4*>(static_cast<const T*>(a.add[g]) + (size_t)row * a.ld);
    mu = a.mean[g][row];
    rstd = a.rstd[g][row];
#pragma unroll
    for (int i = 0; i < C; ++i) {
      const int c = lane + W * i;
      if (c < nch) {
#pragma unroll
        for (int q = 0; q < RW; ++q) {
          x[i][q] = px[c * RW + q];
          dy[i][q] = pd[c * RW + q];
          if (a.add[g]) add[i][q] = pa[c * RW + q];
        }
      }
    }
  }
  // The same through descriptors: nothing is conditional (past the row's end, or of a row that is not `there`, zeros), so that the
  // compiler knows how many loads and stores stand behind these and waits for no more than them.  row: the same for the whole wave.
  __device__ __forceinline__ void fetch(const LnRows& a, int row, bool there, int lane) {
    typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
    const int n = there ? a.d * (int)sizeof(T) : 0;
    auto of = [&](const void* m, int bytes) {
      return __builtin_amdgcn_make_buffer_rsrc(static_cast<T*>(const_cast<void*>(m)) + (size_t)row * a.ld, 0, bytes, 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t rx = of(a.x, n), rd = of(a.dy, n), ra = of(a.add, a.add ? n : 0);
    auto one = [&](const float* m) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(m) + row, 0, there ? 4 : 0, 0x00020000);
      return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, 0, 0, 0));
    };
    mu = one(a.mean);
    rstd = one(a.rstd);
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
      for (int q = 0; q < RW; ++q) {
        const int off = ((lane + W * i) * RW + q) * 16;
        x[i][q] = __builtin_bit_cast(uint4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(rx, off, 0, 0));
        dy[i][q] = __builtin_bit_cast(uint4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(rd, off, 0, 0));
        add[i][q] = __builtin_bit_cast(uint4, (u32x4)__builtin_amdgcn_raw_buffer_load_b128(ra, off, 0, 0));
      }
  }
};
// A lane's gamma: in registers, or (AGAIN) read from LDS where it is used, dy * gamma being worked out twice: 24 registers less for
// the kernel whose occupancy they cost.
template <int C>
struct GammaRegs {
  static constexpr bool AGAIN = false;
  const float (&v)[C][8];
  __device__ __forceinline__ void get(int i, int, float (&o)[8]) const {
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = v[i][e];
  }
};
struct GammaLds {
  static constexpr bool AGAIN = true;
  const float* p;
  __device__ __forceinline__ void get(int, int c, float (&o)[8]) const { ld8<float>(p + 8 * c, o); }
};
// Eight elements of a row of dx, dropped where the row has none
template <typename T>
__device__ __forceinline__ void store8_rows(const LnRows& a, int row, int c, const float (&v)[8]) {
  typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(static_cast<T*>(a.dx) + (size_t)row * a.ld, 0, a.d * (int)sizeof(T), 0x00020000);
  if constexpr (sizeof(T) == 2) {
    const u32x4 w = {pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7])};
    __builtin_amdgcn_raw_buffer_store_b128(w, rs, c * 16, 0, 0);
  } else {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const u32x4 w = {__float_as_uint(v[4 * q]), __float_as_uint(v[4 * q + 1]), __float_as_uint(v[4 * q + 2]), __float_as_uint(v[4 * q + 3])};
      __builtin_amdgcn_raw_buffer_store_b128(w, rs, (2 * c + q) * 16, 0, 0);
    }
  }
}
// One row: its dx is stored, its terms are added to the column sums where SUMS.  Every multiply-add is written out, so that all
// kernels give the same bits.
template <typename T, int C, bool SUMS, typename GA>
__device__ __forceinline__ void ln_bwd_row(const LnBwdArgs& a, int g, int row, int lane, int nch, const LnRow<T, C>& r,
                                           const GA& gam, float (&sg)[C][8], float (&sb)[C][8], const LnRows* rows = nullptr) {
#pragma clang fp contract(off)
  // The test for a residual stands here, ahead of the sums, and all loads with it.  At the end, ln_bwd_split_kernel, us, here | there: bf16 4 x [1024, 256]
  // 5.64 | 5.79, 4 x [512, 512] 4.46 | 4.53; few rows 7 x [21, 360] 4.24 | 4.12
  const bool desc = rows != nullptr, has_add = desc ? rows->add != nullptr : a.add[g] != nullptr;
  float xh[C][8], gg[C][8];
  float s1 = 0.f, s2 = 0.f;
#pragma unroll
  for (int i = 0; i < C; ++i) {
    if ((C == 2 && i == 0 && !GA::AGAIN) || lane + 64 * i < nch) {
      float xv[8], dv[8], ga[8];
      unpack8<T>(r.x[i], xv);
      unpack8<T>(r.dy[i], dv);
      gam.get(i, lane + 64 * i, ga);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        xh[i][e] = (xv[e] - r.mu) * r.rstd;
        gg[i][e] = dv[e] * ga[e];
        s1 = fmaf(dv[e], ga[e], s1);
        s2 = fmaf(gg[i][e], xh[i][e], s2);
        if (SUMS) {
          sg[i][e] = fmaf(dv[e], xh[i][e], sg[i][e]);
          sb[i][e] += dv[e];
        }
      }
    }
  }
  const float c1 = wave_sum(s1) / (float)a.d, c2 = wave_sum(s2) / (float)a.d;
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int c = lane + 64 * i;
    float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if ((C == 2 && i == 0 && !GA::AGAIN) || c < nch) {
      if constexpr (GA::AGAIN) {
        float dv[8], ga[8];
        unpack8<T>(r.dy[i], dv);
        gam.get(i, c, ga);
#pragma unroll
        for (int e = 0; e < 8; ++e) gg[i][e] = dv[e] * ga[e];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = r.rstd * fmaf(-xh[i][e], c2, gg[i][e] - c1);
      if (has_add) {
        float av[8];
        unpack8<T>(r.add[i], av);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] += av[e];
      }
      if (!desc) st8<T>(static_cast<T*>(a.dx[g]) + (size_t)row * a.ld + 8 * c, o);
    }
    if (desc) store8_rows<T>(*rows, row, c, o);
  }
}
// Many rows: workgroups of 4 waves, each with its next row's loads in flight while it reduces the current one; bound by memory.  By
// descriptors, two rows' operands in turn.  With conditional loads and the next row's copied over the current one's, a row began when its
// own loads and the last row's stores were through, and read its pointers anew after them.  us, before | now, forward pass with it:
// 4 x [16384, 768] bf16 123.3 | 121.4, 2 x [12000, 640] 50.9 | 47.7, [65536, 128] 50.1 | 45.4, 4 x [16384, 512] 82.6 | 78.7; fp32 4 x [12000, 256]
// 65.2 | 61.5, 2 x [9000, 1000] 118 | 109.  16-bit matrices may start at any element: the target's unaligned access mode holds for descriptors, too
// (a test compares such matrices with ones that start on a word; the old loops, which they had for a while, took longer: backward alone
// 4 x [16384, 768] 98 | 93, 4 x [16384, 512] 56.6 | 54.5, 3 x [8000, 1536] 77 | 72.5, [2000, 3000] 46.2 | 38.2).
// FOUR (bf16 rows wider than 512): gamma in LDS, 124 registers instead of 141, so that four workgroups share a CU and not three;
// ahead where they are one pass that way and two the other: 4 x [16384, 768] (1024 workgroups) 95.7 | 91.1 us.
template <typename T, int C, bool FOUR = false>
__global__ __launch_bounds__(256, FOUR ? 4 : 1) void ln_bwd_kernel(const LnBwdArgs a) {
  extern __shared__ float red[];  // [4][2][d], FOUR: gamma [d]
  float* const gl = red + 8 * a.d;
  const int g = blockIdx.y, lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nch = a.d >> 3;
  const int first = blockIdx.x * LN_ROWS_PER_WG, row0 = first + wave, end = first + min(a.rows - first, LN_ROWS_PER_WG);
  const LnRows rows = {a.x[g], a.dy[g], a.add[g], a.dx[g], a.mean[g], a.rstd[g], a.d, a.ld};
  float ga[C][8], sg[C][8], sb[C][8];
  LnRow<T, C> cur, nxt;
  cur.fetch(rows, row0, row0 < end, lane);
  nxt.fetch(rows, row0 + 4, row0 + 4 < end, lane);
  if constexpr (FOUR)
    for (int j = 4 * threadIdx.x; j < a.d; j += 1024) *reinterpret_cast<float4*>(gl + j) = *reinterpret_cast<const float4*>(a.gamma[g] + j);
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int c = lane + 64 * i;
#pragma unroll
    for (int e = 0; e < 8; ++e) sg[i][e] = sb[i][e] = ga[i][e] = 0.f;
    if (!FOUR && c < nch) ld8<float>(a.gamma[g] + 8 * c, ga[i]);
  }
  if constexpr (FOUR) __syncthreads();
  auto add_row = [&](int row, const LnRow<T, C>& r) {
    if constexpr (FOUR) ln_bwd_row<T, C, true>(a, g, row, lane, nch, r, GammaLds{gl}, sg, sb, &rows);
    else ln_bwd_row<T, C, true>(a, g, row, lane, nch, r, GammaRegs<C>{ga}, sg, sb, &rows);
  };
  // The first row stands ahead of the loop, so that at its head the same loads and stores are on their way from either side
  if (row0 < end) add_row(row0, cur);
  for (int row = row0 + 4; row < end; row += 4) {
    cur.fetch(rows, row + 4, row + 4 < end, lane);
    add_row(row, nxt);
    row += 4;
    if (row >= end) break;
    nxt.fetch(rows, row + 4, row + 4 < end, lane);
    add_row(row, cur);
  }
  // the waves' partial sums are added in wave order
#pragma unroll
  for (int i = 0; i < C; ++i) {
    const int c = lane + 64 * i;
    if (c < nch) {
      st8<float>(&red[(wave * 2 + 0) * a.d + 8 * c], sg[i]);
      st8<float>(&red[(wave * 2 + 1) * a.d + 8 * c], sb[i]);
    }
  }
  __syncthreads();
  float* part = a.part[g] + (size_t)blockIdx.x * 2 * a.d;
  for (int j = threadIdx.x; j < 2 * a.d; j += 256) {  // red is [wave][2 d]
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) t += red[w * 2 * a.d + j];
    part[j] = t;
  }
}

// Up to a workgroup per CU and d <= 512: 16 waves per 64 rows, four rows each, so that a block is a quarter as long.  The row sums
// need no order among rows; the column sums keep the order of ln_bwd_kernel: waves w, 4 + w, 8 + w, 12 + w hold the rows of its
// wave w in turn and hand the sums on through LDS.  us, this | 4 waves of 16 rows: 4 x [2048, 256] bf16 12.1 | 17.5, 4 x [4096, 512]
// (256 blocks) 17.7 | 20.2, 8 x [3094, 224] (392) 22.9 | 22.0, 16 x [2048, 512] (512) 30 | 25.5; fp32 2 x [4096, 512] (128) 19.0 | 20.6,
// 4 x [4096, 256] (256) 16.6 | 20.2, 4 x [3300, 384] (208) 19.5 | 21.4, 4 x [4096, 512] 26.8 | 25.4.  Held to 64 registers, so that two
// workgroups fit a CU, it spills: 27-33 at 8 x [3094, 224].
template <typename T>
__global__ __launch_bounds__(1024) void ln_bwd_chain_kernel(const LnBwdArgs a) {
  __shared__ float4 red[4][4][64];  // [chain][sums of dgamma: columns 0-3, 4-7 of the lane's chunk; of dbeta][lane]
  const int g = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, w = wave & 3, quarter = wave >> 2;
  const int nch = a.d >> 3, row0 = blockIdx.x * LN_ROWS_PER_WG + w + 16 * quarter;
  float ga[1][8], none[1][8];
  LnRow<T, 1> r[4];
#pragma unroll
  for (int b0 = 0; b0 < 4; b0 += 2) {  // two rows in flight: four spill with fp32
#pragma unroll
    for (int b = b0; b < b0 + 2; ++b)
      if (row0 + 4 * b < a.rows) r[b].fetch(a, g, row0 + 4 * b, lane, nch);
    if (b0 == 0 && lane < nch) ld8<float>(a.gamma[g] + 8 * lane, ga[0]);
#pragma unroll
    for (int b = b0; b < b0 + 2; ++b)
      if (row0 + 4 * b < a.rows) ln_bwd_row<T, 1, false>(a, g, row0 + 4 * b, lane, nch, r[b], GammaRegs<1>{ga}, none, none);
  }
  for (int p = 0; p < 4; ++p) {
    if (quarter == p) {
#pragma clang fp contract(off)
      float sg[8], sb[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) sg[e] = sb[e] = 0.f;
      if (p > 0) {
        const float4 t[4] = {red[w][0][lane], red[w][1][lane], red[w][2][lane], red[w][3][lane]};
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          sg[4 * h] = t[h].x; sg[4 * h + 1] = t[h].y; sg[4 * h + 2] = t[h].z; sg[4 * h + 3] = t[h].w;
          sb[4 * h] = t[2 + h].x; sb[4 * h + 1] = t[2 + h].y; sb[4 * h + 2] = t[2 + h].z; sb[4 * h + 3] = t[2 + h].w;
        }
      }
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if (row0 + 4 * b < a.rows && lane < nch) {
          float xv[8], dv[8];
          unpack8<T>(r[b].x[0], xv);
          unpack8<T>(r[b].dy[0], dv);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            sg[e] = fmaf(dv[e], (xv[e] - r[b].mu) * r[b].rstd, sg[e]);
            sb[e] += dv[e];
          }
        }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        red[w][h][lane] = make_float4(sg[4 * h], sg[4 * h + 1], sg[4 * h + 2], sg[4 * h + 3]);
        red[w][2 + h][lane] = make_float4(sb[4 * h], sb[4 * h + 1], sb[4 * h + 2], sb[4 * h + 3]);
      }
    }
    __syncthreads();
  }
  const int which = threadIdx.x >> 9, col = threadIdx.x & 511;
  if (col < a.d) {
    float t = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c) t += reinterpret_cast<const float*>(&red[c][2 * which + ((col >> 2) & 1)][col >> 3])[col & 3];
    a.part[g][((size_t)blockIdx.x * 2 + which) * a.d + col] = t;
  }
}

template <typename T> struct LnQuad { typedef uint4 type; };
template <> struct LnQuad<bf16_t> { typedef uint2 type; };
__device__ __forceinline__ void unpack4(const uint4& r, float (&v)[4]) {
  v[0] = __uint_as_float(r.x); v[1] = __uint_as_float(r.y); v[2] = __uint_as_float(r.z); v[3] = __uint_as_float(r.w);
}
__device__ __forceinline__ void unpack4(const uint2& r, float (&v)[4]) {
  v[0] = __uint_as_float(r.x << 16); v[1] = __uint_as_float(r.x & 0xffff0000u); v[2] = __uint_as_float(r.y << 16); v[3] = __uint_as_float(r.y & 0xffff0000u);
}
// Launches that do not fill the chip: every row gets a wave of its own, and the column sums, which need nothing from the rows' own
// pass (the row statistics are inputs), are added up by workgroups of their own straight from x and dy, which the row
// workgroups read at the same time.  The order is that of ln_bwd_kernel and ln_reduce_kernel, so the bits are the same: thread
// (chain, 4 columns) adds the 16 rows that a wave of ln_bwd_kernel would, four chains make a block's partial sum.  A column
// workgroup takes 20 blocks of 64 rows; where those are all (FINAL), it adds the partial sums up as ln_reduce_kernel does and
// there is no second launch.  dx must not overlap x or dy.
// us, this | ln_bwd_chain_kernel (d <= 512) or ln_bwd_kernel: 4 x [1024, 256] bf16 6.3 | 11.4, 4 x [1024, 768] 11.2 | 22.9, 1 x [4096, 1024]
// 14.8 | 25.1; x and dy are read twice, which sets the limit: 16 x [1024, 256] 16.3 | 14.2, 16 x [1024, 1024] 32.2 | 27.3.
// What bounds the small ones is a thread's own instruction stream.  With eight columns per thread 1 x [64, 64] takes 5.8 us, with a
// test around every load 5.3, as it is 3.7 (a launch: 2.4); eight rows in flight instead of four are level there and cost
// occupancy elsewhere (4 x [1280, 1024] 16.3 | 13.3).
constexpr int LN_SPLIT_BLOCKS = 20, LN_SPLIT_COLS = 32, LN_SPLIT_NT = LN_SPLIT_BLOCKS * 4 * LN_SPLIT_COLS / 4;
template <typename T, int C, bool FINAL>
__global__ __launch_bounds__(LN_SPLIT_NT) void ln_bwd_split_kernel(const LnBwdArgs a, int col_wgs) {
  constexpr int NV = 2 * LN_SPLIT_COLS;
  __shared__ float red[4 * LN_SPLIT_BLOCKS][NV], sum[FINAL ? LN_SPLIT_BLOCKS : 1][NV];
  const int g = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if ((int)blockIdx.x >= col_wgs) {
    const int row = ((int)blockIdx.x - col_wgs) * (LN_SPLIT_NT / 64) + wave, nch = a.d >> 3;
    if (row >= a.rows) return;
    float ga[C][8], none[C][8];
    LnRow<T, C> r;
    r.fetch(a, g, row, lane, nch);
#pragma unroll
    for (int i = 0; i < C; ++i)
      if (lane + 64 * i < nch) ld8<float>(a.gamma[g] + 8 * (lane + 64 * i), ga[i]);
    ln_bwd_row<T, C, false>(a, g, row, lane, nch, r, GammaRegs<C>{ga}, none, none);
    return;
  }
  typedef typename LnQuad<T>::type Q;
  constexpr int NB = 4;  // rows whose loads are in flight together
  const int nblk = (a.rows + LN_ROWS_PER_WG - 1) / LN_ROWS_PER_WG, ncol = (a.d + LN_SPLIT_COLS - 1) / LN_SPLIT_COLS;
  const int blk0 = FINAL ? 0 : (int)blockIdx.x / ncol * LN_SPLIT_BLOCKS, nb = min(nblk - blk0, LN_SPLIT_BLOCKS);
  // workgroups 8 apart, which run on one XCD, take neighbouring columns: 32 columns of 16 bits are half a cache line
  int ci = FINAL ? (int)blockIdx.x : (int)blockIdx.x % ncol;
  if (ci < ncol / 16 * 16) ci = ci / 16 * 16 + (ci % 8) * 2 + (ci / 8) % 2;
  const int col0 = ci * LN_SPLIT_COLS, c = col0 / 4 + (tid & 7);  // 4 columns
  const int chain = tid >> 3;  // rows (blk0 + chain/4) * 64 + chain%4, + 4, ...
  if (chain < 4 * nb) {
#pragma clang fp contract(off)
    // columns past the matrix are read as its first ones, and rows past the block as its last: no branch around a load
    const int first = (blk0 + (chain >> 2)) * LN_ROWS_PER_WG, row0 = first + (chain & 3), end = first + min(a.rows - first, LN_ROWS_PER_WG);
    const size_t col = 4 * c < a.d ? 4 * c : 0;
    const T* X = static_cast<const T*>(a.x[g]) + col;
    const T* DY = static_cast<const T*>(a.dy[g]) + col;
    const float* mean = a.mean[g];
    const float* rs = a.rstd[g];
    float sg[4] = {0.f, 0.f, 0.f, 0.f}, sb[4] = {0.f, 0.f, 0.f, 0.f};
    auto add_rows = [&](auto full) {
      constexpr bool FULL = decltype(full)::value;
#pragma unroll 1
      for (int i0 = 0; i0 < 16; i0 += NB) {
        Q rx[NB], rdy[NB];
        float mu[NB], rstd[NB];
        const int rb = row0 + 4 * i0;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          const int row = FULL ? rb + 4 * b : min(rb + 4 * b, end - 1);
          mu[b] = mean[row];
          rstd[b] = rs[row];
          rx[b] = *reinterpret_cast<const Q*>(X + (size_t)row * a.ld);
          rdy[b] = *reinterpret_cast<const Q*>(DY + (size_t)row * a.ld);
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
          float xv[4], dv[4];
          unpack4(rx[b], xv);
          unpack4(rdy[b], dv);
          const bool in = FULL || rb + 4 * b < end;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float tg = fmaf(dv[e], (xv[e] - mu[b]) * rstd[b], sg[e]), tb = sb[e] + dv[e];
            sg[e] = in ? tg : sg[e];
            sb[e] = in ? tb : sb[e];
          }
        }
      }
    };
    if (__all(end - first == LN_ROWS_PER_WG)) add_rows(std::true_type());
    else add_rows(std::false_type());
    *reinterpret_cast<float4*>(&red[chain][4 * (tid & 7)]) = make_float4(sg[0], sg[1], sg[2], sg[3]);
    *reinterpret_cast<float4*>(&red[chain][LN_SPLIT_COLS + 4 * (tid & 7)]) = make_float4(sb[0], sb[1], sb[2], sb[3]);
  }
  __syncthreads();
  for (int i = tid; i < nb * NV; i += LN_SPLIT_NT) {
    const int b = i / NV, j = i % NV, col = col0 + j % LN_SPLIT_COLS;
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) t += red[4 * b + w][j];
    if (FINAL) sum[b][j] = t;
    else if (col < a.d) a.part[g][(size_t)(blk0 + b) * 2 * a.d + (j / LN_SPLIT_COLS) * a.d + col] = t;
  }
  if (!FINAL) return;
  __syncthreads();
  if (tid < NV) {  // 16 ranges of partial sums, as in ln_reduce_kernel
    const int per = (nb + 15) / 16;
    float t[16], s = 0.f;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
      t[w] = w * per < nb ? sum[w * per][tid] : 0.f;
      if (per == 2) t[w] += 2 * w + 1 < nb ? sum[2 * w + 1][tid] : 0.f;
    }
#pragma unroll
    for (int w = 0; w < 16; ++w) s += t[w];
    const int col = col0 + tid % LN_SPLIT_COLS;
    if (col < a.d) (tid / LN_SPLIT_COLS ? a.dbeta[g] : a.dgamma[g])[col] = s;
  }
}

// Eight elements of a wide row: x-hat, dy * gamma and what they add to the row's and the columns' sums, and their dx.  Every multiply-add is
// written out, as in ln_bwd_row, and none is left to the compiler: which of the kernels below runs depends on how many problems share a
// launch (ln_wide_ahead).  (The residual is added by the kernels: with its test in here the compiler made selections of it, and the
// kernel without look-ahead, whose registers were then dealt out another way, waited at every row for the stores of the one before,
// 2 x [9024, 2048] 132 | 142 us.)
__device__ __forceinline__ void ln_wide_terms(const float (&xv)[8], const float (&dv)[8], const float (&ga)[8], float mu, float rstd, float (&xh)[8],
                                              float (&gg)[8], float& s1, float& s2, float (&sg)[8], float (&sb)[8]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    xh[e] = (xv[e] - mu) * rstd;
    gg[e] = dv[e] * ga[e];
    s1 = fmaf(dv[e], ga[e], s1);
    s2 = fmaf(gg[e], xh[e], s2);
    sg[e] = fmaf(dv[e], xh[e], sg[e]);
    sb[e] += dv[e];
  }
}
__device__ __forceinline__ void ln_wide_dx(const float (&xh)[8], const float (&gg)[8], float rstd, float c1, float c2, float (&o)[8]) {
#pragma clang fp contract(off)
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = rstd * fmaf(-xh[e], c2, gg[e] - c1);
}
// Rows of more than 1024 elements: a wave per row would need 32 or 64 values of x-hat and g per lane (one or two waves
// per SIMD, and up to 128 KB of LDS for the cross-wave column sums).  Here the four waves of a workgroup share each
// row: thread t owns chunks t, t + 256, the two row sums cross the waves through LDS (added in wave
// order), and every column belongs to exactly one thread, which adds its dgamma/dbeta terms over the workgroup's 32
// rows in row order and writes them to part[g][b][2][d] itself.
//
// fp32 rows of up to 2048 elements where this kernel, which asks for a row when it comes to it, is ahead (ln_wide_ahead).
__global__ __launch_bounds__(256) void ln_bwd_wide_f32_kernel(const LnBwdArgs a) {
#pragma clang fp contract(off)
  __shared__ float xs[2][4][2];  // [row parity][wave][s1, s2]
  const int g = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nch = a.d >> 3;
  const float* gamma = a.gamma[g];
  float ga[8], sg[8], sb[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) sg[e] = sb[e] = ga[e] = 0.f;
  if (tid < nch) ld8<float>(gamma + 8 * tid, ga);
  const bool has_add = a.add[g] != nullptr;
  const int row0 = blockIdx.x * LN_WIDE_ROWS_PER_WG;
  const int nrow = min(LN_WIDE_ROWS_PER_WG, a.rows - row0);  // the same for every thread: the barriers below are uniform
  uint4 x[2], dy[2], add[2];
  float mu = 0.f, rstd = 0.f;
  auto fetch_row = [&](int row) {
    const uint4* px = reinterpret_cast<const uint4*>(static_cast<const float*>(a.x[g]) + (size_t)row * a.ld);
    const uint4* pdy = reinterpret_cast<const uint4*>(static_cast<const float*>(a.dy[g]) + (size_t)row * a.ld);
    const uint4* padd = has_add ? reinterpret_cast<const uint4*>(static_cast<const float*>(a.add[g]) + (size_t)row * a.ld) : nullptr;
    if (tid < nch) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        x[q] = px[tid * 2 + q];
        dy[q] = pdy[tid * 2 + q];
        if (has_add) add[q] = padd[tid * 2 + q];
      }
    }
    mu = a.mean[g][row];
    rstd = a.rstd[g][row];
  };
  for (int r = 0; r < nrow; ++r) {
    const int row = row0 + r;
    fetch_row(row);
    float xh[8], gg[8];
    float s1 = 0.f, s2 = 0.f;
    if (tid < nch) {
      float xv[8], dv[8];
      unpack8<float>(x, xv);
      unpack8<float>(dy, dv);
      ln_wide_terms(xv, dv, ga, mu, rstd, xh, gg, s1, s2, sg, sb);
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
    float* dx = static_cast<float*>(a.dx[g]) + (size_t)row * a.ld;
    if (tid < nch) {
      float o[8];
      ln_wide_dx(xh, gg, rstd, c1, c2, o);
      if (has_add) {
        float av[8];
        unpack8<float>(add, av);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] += av[e];
      }
      st8<float>(dx + 8 * tid, o);
    }
  }
  float* part = a.part[g] + (size_t)blockIdx.x * 2 * a.d;
  if (tid < nch) {
    st8<float>(part + 8 * tid, sg);
    st8<float>(part + a.d + 8 * tid, sb);
  }
}

// All others: every row on its way while the one before it is reduced, as in ln_bwd_kernel, and the operands of two rows in turn.  us, a row asked
// for when it is due (bf16: one ahead, under conditions) | this, forward pass with it: 2 x [16384, 4096] bf16 350 | 335, 3 x [8000, 1536] 94.9 | 92.1,
// [2000, 3000] 51.7 | 39.9; fp32 2 x [16384, 4096] 668 | 629, 2 x [4000, 2560] 147 | 105, 2 x [9000, 1288] 138 | 128.
template <typename T, int MAXW>
__global__ __launch_bounds__(256) void ln_bwd_wide_kernel(const LnBwdArgs a) {
#pragma clang fp contract(off)
  __shared__ float xs[2][4][2];  // [row parity][wave][s1, s2]
  const int g = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nch = a.d >> 3;
  typedef LnRow<T, MAXW, 256> Row;
  const int row0 = blockIdx.x * LN_WIDE_ROWS_PER_WG;
  const int nrow = min(LN_WIDE_ROWS_PER_WG, a.rows - row0);  // the same for every thread: the barriers below are uniform
  const LnRows rows = {a.x[g], a.dy[g], a.add[g], a.dx[g], a.mean[g], a.rstd[g], a.d, a.ld};
  Row cur, nxt;
  cur.fetch(rows, row0, true, tid);
  nxt.fetch(rows, row0 + 1, nrow > 1, tid);
  const float* gamma = a.gamma[g];
  float ga[MAXW][8], sg[MAXW][8], sb[MAXW][8];
#pragma unroll
  for (int i = 0; i < MAXW; ++i) {
    const int c = tid + 256 * i;
#pragma unroll
    for (int e = 0; e < 8; ++e) sg[i][e] = sb[i][e] = ga[i][e] = 0.f;
    if (c < nch) ld8<float>(gamma + 8 * c, ga[i]);
  }
  const bool has_add = rows.add != nullptr;
  auto add_row = [&](int r, const Row& in) {
    float xh[MAXW][8], gg[MAXW][8];
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int i = 0; i < MAXW; ++i) {
      if ((MAXW == 2 && i == 0) || tid + 256 * i < nch) {
        float xv[8], dv[8];
        unpack8<T>(in.x[i], xv);
        unpack8<T>(in.dy[i], dv);
        ln_wide_terms(xv, dv, ga[i], in.mu, in.rstd, xh[i], gg[i], s1, s2, sg[i], sb[i]);
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
#pragma unroll
    for (int i = 0; i < MAXW; ++i) {
      const int c = tid + 256 * i;
      float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if ((MAXW == 2 && i == 0) || c < nch) {
        ln_wide_dx(xh[i], gg[i], in.rstd, c1, c2, o);
        if (has_add) {
          float av[8];
          unpack8<T>(in.add[i], av);
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] += av[e];
        }
      }
      store8_rows<T>(rows, row0 + r, c, o);
    }
  };
  add_row(0, cur);  // ahead of the loop, as in ln_bwd_kernel
  for (int r = 1; r < nrow; ++r) {
    cur.fetch(rows, row0 + r + 1, r + 1 < nrow, tid);
    add_row(r, nxt);
    if (++r >= nrow) break;
    nxt.fetch(rows, row0 + r + 1, r + 1 < nrow, tid);
    add_row(r, cur);
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
  // 16 partial sums requested together, past the range its last one again (one after the other, each add waits for its load)
  if (j < n2)
    for (int b = b0; b < b1; b += 16) {
      float v[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = part[(size_t)min(b + i, b1 - 1) * n2 + j];
#pragma unroll
      for (int i = 0; i < 16; ++i) t = b + i < b1 ? t + v[i] : t;
    }
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
  const size_t lds = (size_t)4 * 8 * a.d;
  // at most one 16-wave workgroup per CU; wide fp32 rows gain nothing when every CU has one
  const long blocks = (long)grid.x * a.G;
  const bool chain = a.d <= 512 && blocks <= 256 && (sizeof(T) == 2 || blocks * a.d <= 96 * 1024);
  if (chain) hipLaunchKernelGGL((ln_bwd_chain_kernel<T>), grid, dim3(1024), 0, s, a);
  else if (a.d <= 512) hipLaunchKernelGGL((ln_bwd_kernel<T, 1>), grid, dim3(256), lds, s, a);
  else if (sizeof(T) == 2 && a.d <= LN_WAVE_ROW_MAX && ln_four_to_a_cu(blocks))
    hipLaunchKernelGGL((ln_bwd_kernel<bf16_t, 2, true>), grid, dim3(256), lds + 4 * a.d, s, a);
  else if (a.d <= LN_WAVE_ROW_MAX) hipLaunchKernelGGL((ln_bwd_kernel<T, 2>), grid, dim3(256), lds, s, a);
  else if (sizeof(T) == 4 && a.d <= 2048 && !ln_wide_ahead(blocks, a.d)) hipLaunchKernelGGL(ln_bwd_wide_f32_kernel, grid, dim3(256), 0, s, a);
  else if (a.d <= 2048) hipLaunchKernelGGL((ln_bwd_wide_kernel<T, 1>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((ln_bwd_wide_kernel<T, 2>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

template <typename T, int C>
static hipError_t ln_bwd_split_run(const LnBwdArgs& a, hipStream_t s) {
  const int nblk = ln_bwd_blocks(a.rows, a.d), ranges = (nblk + LN_SPLIT_BLOCKS - 1) / LN_SPLIT_BLOCKS;
  const int col_wgs = (a.d + LN_SPLIT_COLS - 1) / LN_SPLIT_COLS * ranges;
  const dim3 grid(col_wgs + (a.rows + LN_SPLIT_NT / 64 - 1) / (LN_SPLIT_NT / 64), a.G);
  if (ranges == 1) hipLaunchKernelGGL((ln_bwd_split_kernel<T, C, true>), grid, dim3(LN_SPLIT_NT), 0, s, a, col_wgs);
  else hipLaunchKernelGGL((ln_bwd_split_kernel<T, C, false>), grid, dim3(LN_SPLIT_NT), 0, s, a, col_wgs);
  return hipGetLastError();
}

// dx of some problem over its x or dy: the column workgroups of ln_bwd_split_kernel would read those while the row workgroups store
// dx, where the other kernels have read a row before they store it.
static bool ln_bwd_in_place(const LnBwdArgs& a) {
  const uintptr_t n = ((size_t)(a.rows - 1) * a.ld + a.d) * (a.dtype == GEMM_F32 ? 4 : 2);
  for (int g = 0; g < a.G; ++g) {
    const uintptr_t o = (uintptr_t)a.dx[g], x = (uintptr_t)a.x[g], dy = (uintptr_t)a.dy[g];
    if ((o < x + n && x < o + n) || (o < dy + n && dy < o + n)) return true;
  }
  return false;
}
// Whether row and column workgroups side by side are the faster form (a choice never changes a bit of the result, so it may look
// at the group).  us, this | the other form.  d <= 512: up to 3 M elements in one launch (2 M fp32 12.1 | 16.1, 4 M bf16 13.1 | 13.9 and
// 16.3 | 14.2), half of that in two (1.3 M 9.2 | 11.7, 2 M 12.2 | 12.1 and 11.7 | 13.3, fp32 17.4 | 14.4).  Wider: up to 20 MB (bf16 16 MB
// 21.5 | 26.7, 24 MB 31.5 | 26.5; fp32 20 MB 24.4 | 28.7, 31 MB 33.0 | 30.7).
static bool ln_bwd_split(const LnBwdArgs& a) {
  if (a.d > LN_WAVE_ROW_MAX || ln_bwd_in_place(a)) return false;
  const long n = (long)a.G * a.rows * a.d;
  if (a.d > 512) return n * (a.dtype == GEMM_F32 ? 4 : 2) <= 20L << 20;
  return n <= (a.rows <= LN_SPLIT_BLOCKS * LN_ROWS_PER_WG ? 3L << 20 : 3L << 19);
}

hipError_t launch_ln_bwd(const LnBwdArgs& a, hipStream_t s) {
  if (!ln_shape_ok(a.G, a.rows, a.d, a.ld)) return hipErrorInvalidValue;
  const bool f32 = a.dtype == GEMM_F32;
  hipError_t e;
  if (ln_bwd_split(a)) {
    if (a.d <= 512) e = f32 ? ln_bwd_split_run<float, 1>(a, s) : ln_bwd_split_run<bf16_t, 1>(a, s);
    else e = f32 ? ln_bwd_split_run<float, 2>(a, s) : ln_bwd_split_run<bf16_t, 2>(a, s);
    if (a.rows <= LN_SPLIT_BLOCKS * LN_ROWS_PER_WG) return e;
  } else {
    e = f32 ? ln_bwd_pick<float>(a, s) : ln_bwd_pick<bf16_t>(a, s);
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(ln_reduce_kernel, dim3((2 * a.d + 15) / 16, a.G), dim3(256), 0, s, a, ln_bwd_blocks(a.rows, a.d));
  return hipGetLastError();
}

// nothing to set up: the wave-per-row kernel needs at most 32 KB of LDS
hipError_t ln_init() { return hipSuccess; }

}  // namespace hydra
