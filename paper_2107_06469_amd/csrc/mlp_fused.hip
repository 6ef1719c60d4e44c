// Whole shard phases of small fp32 MLPs in one launch each.
//
// A model whose step is a few megaflops (32 rows, layers up to 256 wide) is bound by the chain of dependent launches,
// not by arithmetic or memory: every Linear layer as a launch of its own costs a launch, a round trip to memory for its
// operands and a kernel boundary.  Here the forward pass of a shard (all its layers, and the rows' losses when the shard
// ends the model) is one launch; the backward pass is two: the chain of input gradients through the shard's layers,
// then every weight gradient of the shard at once, each with the parameter update in the same kernel (a workgroup per
// 32 output rows of a layer; the one that has the model's last layer also adds up the step's loss).  In the two chains
// a workgroup takes 4 rows of one model's batch through all the layers, activations staying in LDS between them: rows are
// independent there.  Every sum runs in a fixed order that depends on the layer's shape alone, and the epilogues
// apply the same single-rounded operations as the tiled GEMM kernel's.  Results depend on nothing but the model: not
// on the group, the cut points or the schedule.
//
// Bound by what one compute unit takes in: 256 KB of weights a layer at 36 to 40 bytes a cycle, 3 us.  The same weights go into LDS and out
// again, 512 KB at 128 bytes a cycle, 4100 of those 6300 to 7200 cycles, and the products (32 dependent instructions of 12 cycles per 32
// k) stand beside both.  4 x (4 layers of 256, 32 rows), forward and chain in one launch: 35.8 us, of which
// 23 are those sums; with 16 rows a workgroup (v_mfma_f32_16x16x4_f32, weights through registers, 8 of 256 compute units) 59.4.
// Bringing the weights into L2 beforehand changes nothing, nor does asking for the input rows ahead of them.
#include "act_math.h"
#include "kernels.h"
#include "lds_dma.h"
#include "optim_math.h"

namespace hydra {
namespace {

typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4a;
constexpr int XS = 272;            // LDS row pitch in floats (256 + 16: the four rows of an operand read start 16 banks apart)
constexpr int RB = 4;              // batch rows of a workgroup of the two chain kernels

// acc += W-operand chunk (4 consecutive k of one row n) x X-operand chunk (the same k of one row m) for the weight-gradient
// kernel's 32 x 32 tiles: four instructions, each summing k and k+4 (the two half-waves hold chunks 4 apart)
__device__ __forceinline__ void mma4(f32x16& acc, const float4& w, const float4& x) {
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w.x, x.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w.y, x.y, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w.z, x.z, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w.w, x.w, acc, 0, 0, 0);
}
// The chain kernels' tiles are 4 batch rows x 64 columns, one instruction per k (v_mfma_f32_4x4x1_16b_f32: sixteen blocks of 4 x 4,
// lane l holds column l in four registers, one per row).  x: lane l has row l%4 at k = l/4 of a group of 16; the instruction
// broadcasts the block of its k to all sixteen.  w: the lane's column at the 16 k.  The k are taken in the order 0, 4, 8, 12, 1, 5, ...:
// one multiply-add after the other with the rounding of fmaf, the bits of four v_mfma_f32_16x16x4_f32 whose lane group q supplies k = 4 q + e
// (compared bit by bit; those tiles of 16 rows are what the kernels had before).  12 cycles from one to the next that adds to it.
#define HYDRA_MMA_K(K) acc = __builtin_amdgcn_mfma_f32_4x4x1f32(x, w[K], acc, 4, K, 0);
// the j-th of the four products of k = e, 4 + e, 8 + e, 12 + e
__device__ __forceinline__ void mma1(f32x4a& acc, const float* w, float x, int e, int j) {
  switch (4 * j + e) {
    case 0: HYDRA_MMA_K(0) break;   case 1: HYDRA_MMA_K(1) break;   case 2: HYDRA_MMA_K(2) break;   case 3: HYDRA_MMA_K(3) break;
    case 4: HYDRA_MMA_K(4) break;   case 5: HYDRA_MMA_K(5) break;   case 6: HYDRA_MMA_K(6) break;   case 7: HYDRA_MMA_K(7) break;
    case 8: HYDRA_MMA_K(8) break;   case 9: HYDRA_MMA_K(9) break;   case 10: HYDRA_MMA_K(10) break; case 11: HYDRA_MMA_K(11) break;
    case 12: HYDRA_MMA_K(12) break; case 13: HYDRA_MMA_K(13) break; case 14: HYDRA_MMA_K(14) break; case 15: HYDRA_MMA_K(15) break;
  }
}
#undef HYDRA_MMA_K

__device__ __forceinline__ float4 zero4() { return make_float4(0.f, 0.f, 0.f, 0.f); }

// A pointer read from the activation table in memory carries no address space, and through such a pointer the compiler
// emits flat instructions, which count against the LDS counter as well and may complete out of order: every wait
// after one is a wait for everything.  The table's pointers go to global memory; these types say so.
typedef __attribute__((address_space(1))) float gfloat;
typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) f32x4v gf32x4v;
__device__ __forceinline__ gfloat* global_ptr(float* p) { return (gfloat*)p; }
__device__ __forceinline__ const gfloat* global_ptr(const float* p) { return (const gfloat*)p; }
__device__ __forceinline__ float4 gload4(const gfloat* p) {
  const f32x4v v = *(const gf32x4v*)p;
  return make_float4(v.x, v.y, v.z, v.w);
}

// rows [0, rows) x columns [0, cols) of a row-major matrix into the RB LDS rows of pitch XS, 16 bytes a thread; the rest of the 256
// columns is zero (the products run over k in groups of 16 and must not meet what an earlier kernel left in LDS)
__device__ __forceinline__ void stage_rows(float* xs, const gfloat* src, int ld, int rows, int cols, int tid) {
  const int m = tid >> 6, c = (tid & 63) * 4;
  float4 v = zero4();
  if (m < rows && c < cols) {
    const gfloat* r = src + (size_t)m * ld + c;
    if (c + 4 <= cols) v = gload4(r);
    else {
      v.x = r[0];
      if (c + 1 < cols) v.y = r[1];
      if (c + 2 < cols) v.z = r[2];
    }
  }
  *reinterpret_cast<float4*>(&xs[m * XS + c]) = v;
}

// ---- the chains: units [u0, u1) of 4 batch rows of one model per workgroup (4 waves; wave w owns columns [64w, 64w+64)) ----
// Rows of the batch do not meet before the loss, so a model's rows are split over as many workgroups as there are groups of
// four; then a layer costs its wave a chain of 256 instructions (1.3 us) and the compute unit the 256 KB of its weights (3 us).
// A wave multiplies by its own 64 columns' weights only and stages them for itself: chunks of 32 k go from memory straight into a
// ring of four 8 KB pieces of LDS that no other wave touches, three chunks ahead of the one being multiplied, and the requests run ahead across
// layer ends (weights do not depend on activations).  A chunk's weights are in registers before its products start, while the
// next one's are read.  Nothing inside a layer waits for another wave: the workgroup meets once per layer, when its outputs are in
// the other of two LDS buffers.
constexpr int STG = 8192;            // bytes of a stage: 32 k x 64 columns
constexpr int WLDS = 4 * STG + 5 * 256;  // bytes of a wave: its ring, then 5 x 64 floats (the bias; z of the four rows)
constexpr size_t CHAIN_LDS = 2 * RB * XS * sizeof(float) + 4 * (size_t)WLDS;

// the same value in every lane, told to the compiler (descriptors of buffer loads must sit in scalar registers)
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// orders a wave's own LDS writes before its later LDS reads (the hardware keeps a wave's LDS operations in order; this
// keeps the compiler from moving them)
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// of this wave's loads all but the newest N have landed / its LDS reads are done; nothing moves across
template <int N>
__device__ __forceinline__ void loads_but() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void lds_reads_done() {
  __builtin_amdgcn_s_waitcnt(0xc07f);
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ unsigned lds_addr_of(const void* p) {
  return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const char*)reinterpret_cast<const char*>(p);
}
// chunks of a unit whose sum runs over K (an even number: the register sets alternate)
__device__ __forceinline__ int chunks_of(int K) { return (K + 63) / 64 * 2; }

// The stream of weights of a wave.  FWD: W_u [N][K], the wave's 64 rows, 128 contiguous bytes of each per chunk; the 16-byte piece c
// of row r sits at c ^ (r/2)%8 of its row in LDS (16 rows read at one piece spread over all banks).  Backward: W_u [K][N], 32
// rows of k, 256 contiguous bytes of each.  Rows past the matrix lie behind the end of the descriptor and read as zero; columns past it
// are sent out of range; past the last unit the matrix is empty.
template <bool FWD>
struct WStream {
  const MlpFusedArgs& a;
  const float* P;
  int lane, n0, lu, u_end, k0, lK, lN;  // the next chunk to request: k0.. of unit lu
  unsigned ring, seq;                   // LDS byte address; number of the chunk whose weights are in registers
  // its eight loads: load i at base[i % 2] + i * step of the unit's matrix.  A lane that reads past the matrix's columns has a base
  // past every descriptor's end.
  rsrc_u32x4 rs;
  unsigned base[2], step;
  __device__ __forceinline__ WStream(const MlpFusedArgs& a_, const float* p, int lane_, int wave, int u_first, int u_last, unsigned ring_)
      : a(a_), P(p), lane(lane_), n0(wave * 64), lu(u_first), u_end(u_last + (FWD ? 1 : -1)), ring(ring_), seq(0) { unit(); }
  __device__ __forceinline__ void unit() {
    const bool live = FWD ? lu < u_end : lu > u_end;
    const int rows = lu < a.L ? a.d : a.n_out, cols = FWD ? (lu == 0 ? a.d_in : a.d) : a.d;
    k0 = 0;
    lK = uniform(FWD ? cols : rows);
    lN = uniform(FWD ? rows : cols);
    rs = rsrc_settled(rsrc_words(P + a.w_off[live ? lu : a.u0], 0, live ? (long)lN * lK * 4 : 0));
    step = uniform((FWD ? 8 * lK : 4 * lN) * 4);
    place();
  }
  __device__ __forceinline__ void place() {
    if (FWD) {
      const int c0 = k0 + 4 * ((lane & 7) ^ ((lane >> 4) & 3)), row = n0 + (lane >> 3);  // rows 8 further on: c ^ 4
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        const int col = c0 ^ (16 * o);
        base[o] = col < lK ? (unsigned)(row * lK + col) * 4u : 0x80000000u;
      }
    } else {
      const int col = n0 + 4 * (lane & 15);
      base[0] = base[1] = col < lN ? (unsigned)((k0 + (lane >> 4)) * lN + col) * 4u : 0x80000000u;
    }
  }
  __device__ __forceinline__ void advance() {
    k0 += 32;
    if (k0 >= chunks_of(lK) * 32) {
      lu += FWD ? 1 : -1;
      unit();
    } else if (FWD && k0 + 32 > lK) {  // the columns end inside the chunk
      place();
    } else {
      const unsigned by = FWD ? 128u : 8u * step;
      base[0] += by;
      base[1] += by;
    }
  }
  __device__ __forceinline__ void load(unsigned to, int i) const { load_to_lds_b128(rs, to + i * 1024, base[FWD ? i & 1 : 0] + i * step); }
  __device__ __forceinline__ unsigned stage(unsigned s) const { return ring + (s & 3) * STG; }
  __device__ __forceinline__ void request(unsigned s) {
#pragma unroll
    for (int i = 0; i < 8; ++i) load(stage(s), i);
    advance();
  }
  // an eighth of a chunk's weights of this lane's column, k = 4 c + 0..3
  __device__ __forceinline__ void read(unsigned at, int c, float (&w)[32]) const {
    typedef __attribute__((address_space(3))) const f32x4a lds_f4;
    typedef __attribute__((address_space(3))) const float lds_f;
    if (FWD) {
      const f32x4a v = *(lds_f4*)(uintptr_t)(at + lane * 128 + ((c ^ ((lane >> 1) & 7)) << 4));
#pragma unroll
      for (int e = 0; e < 4; ++e) w[4 * c + e] = v[e];
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) w[4 * c + e] = *(lds_f*)(uintptr_t)(at + (4 * c + e) * 256 + lane * 4);
    }
  }
  __device__ __forceinline__ void start(float (&w)[32]) {  // after it: chunk 0 in registers, chunks 1 to 3 on their way
    loads_but<24>();
#pragma unroll
    for (int c = 0; c < 8; ++c) read(stage(0), c, w);
    lds_reads_done();
  }
  // Chunk c of a unit whose weights are in cur: the next chunk's weights go into nxt, the one four ahead takes cur's stage.  One wave
  // to a SIMD issues an instruction every 4 cycles or so, and the products want one every 12: what moves data stands between them (in
  // front of them it took longer than they do).
  __device__ __forceinline__ void chunk(f32x4a& acc, const float (&x)[16], int c, int K, float (&cur)[32], float (&nxt)[32]) {
    loads_but<16>();
    const unsigned at = stage(seq + 1), to = stage(seq);
    if (32 * c + 32 <= K) {  // a whole chunk
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float* const w = cur + 16 * (i >> 2);
        mma1(acc, w, x[2 * c + (i >> 2)], i & 3, 0);
        __builtin_amdgcn_sched_barrier(0);
        read(at, i, nxt);
        __builtin_amdgcn_sched_barrier(0);
        mma1(acc, w, x[2 * c + (i >> 2)], i & 3, 1);
        __builtin_amdgcn_sched_barrier(0);
        load(to, i);
        __builtin_amdgcn_sched_barrier(0);
        mma1(acc, w, x[2 * c + (i >> 2)], i & 3, 2);
        mma1(acc, w, x[2 * c + (i >> 2)], i & 3, 3);
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {  // a group of 16 k that starts at or past K is not multiplied; inside a group, k at or past K meet zeros on both sides
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        read(at, i, nxt);
        load(to, i);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (32 * c + 16 * (i >> 2) < K) {
#pragma unroll
          for (int j = 0; j < 4; ++j) mma1(acc, cur + 16 * (i >> 2), x[2 * c + (i >> 2)], i & 3, j);
        }
    }
    advance();
    lds_reads_done();
    ++seq;
  }
  // a unit: the sum over K of this lane's column for the four rows in xs
  __device__ __forceinline__ f32x4a sum(const float* xs, int K, float (&w0)[32], float (&w1)[32]) {
    float x[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) x[i] = xs[(lane & 3) * XS + 16 * i + (lane >> 2)];
    lds_reads_done();
    f32x4a acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 8; c += 2)
      if (32 * c < K) {
        chunk(acc, x, c, K, w0, w1);
        chunk(acc, x, c + 1, K, w1, w0);
      }
    return acc;
  }
};
// Four rows of a matrix of a.B rows of ld floats, this lane's column n of N: stores past either end are dropped
struct RowStore {
  __amdgpu_buffer_rsrc_t rs;
  unsigned at, step;
  __device__ __forceinline__ RowStore(gfloat* p, int B, int ld, int r0, int n, int N)
      : rs(__builtin_amdgcn_make_buffer_rsrc((float*)p, 0, uniform(p ? B * ld * 4 : 0), 0x00020000)),
        at(n < N ? (unsigned)(r0 * ld + n) * 4u : 0x80000000u), step((unsigned)ld * 4u) {}
  __device__ __forceinline__ void put(int r, float v) const {
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, at + r * step, 0, 0);
  }
};

// The table does not change under the kernel: read through the constant address space its pointers come by scalar loads, which no
// vector load or store waits behind (through a global pointer they were vector loads, and a wait for one a wait for every chunk).
typedef const __attribute__((address_space(4))) MlpTab* TabPtr;

// ---- forward: the shard's layers, and the rows' losses when it ends the model ----------------------------------------------
// THEN: the chain of input gradients follows in the same kernel (all of the model's units): the first chunks of its weights are
// requested when the last layer's products are done, and the logits' gradient is left in the first LDS buffer for it.
template <bool THEN, typename F>
__device__ __forceinline__ void fwd_body(const MlpFusedArgs& a, float* smem, F&& after_products) {
  const int g = blockIdx.x % a.G, r0 = (blockIdx.x / a.G) * RB;  // model, first batch row
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int rows = a.B - r0 < RB ? a.B - r0 : RB;  // >= 1: the grid has ceil(B / RB) workgroups per model
  const TabPtr tb = (TabPtr)a.tab[g];
  const float* P = a.p[g];
  char* const own = reinterpret_cast<char*>(smem + 2 * RB * XS) + wave * WLDS;
  const float* const lbias = reinterpret_cast<const float*>(own + 4 * STG);
  const int n = wave * 64 + lane;  // this lane's column
  WStream<true> ws(a, P, lane, wave, a.u0, a.u1 - 1, lds_addr_of(own));
  float w0[32], w1[32];
#pragma unroll
  for (int s = 0; s < 4; ++s) ws.request(s);
  stage_rows(smem, global_ptr(a.u0 == 0 ? a.x[g] : tb->h[a.u0 - 1]) + (size_t)r0 * (a.u0 == 0 ? a.ld_in : a.ldd),
             a.u0 == 0 ? a.ld_in : a.ldd, rows, a.u0 == 0 ? a.d_in : a.d, tid);
  ws.start(w0);
  __syncthreads();  // the input rows are in place
  for (int u = a.u0; u < a.u1; ++u) {
    const int K = u == 0 ? a.d_in : a.d, N = u < a.L ? a.d : a.n_out;
    float* const xs = smem + ((u - a.u0) & 1) * RB * XS;
    float* const xn = smem + ((u - a.u0 + 1) & 1) * RB * XS;
    load_to_lds_b32(rsrc_settled(rsrc_words(P + a.b_off[u], 0, (long)N * 4)), lds_addr_of(lbias), (unsigned)n * 4u);
    // where the unit's outputs go: read from the table now, not between the stores at the unit's end
    const bool last = u == a.L;
    const RowStore zs(global_ptr(last ? tb->logits : tb->z[u]), a.B, last ? a.ldv : a.ldd, r0, n, N);
    const RowStore hs(global_ptr(last ? nullptr : tb->h[u]), a.B, a.ldd, r0, n, N);
    gfloat* const dlog = global_ptr(last ? tb->dlogits : nullptr);
    gfloat* const rowl = global_ptr(last ? tb->rowloss : nullptr);
    const f32x4a acc = ws.sum(xs, K, w0, w1);
    loads_but<16>();  // the bias, requested before the unit's chunks (two at least)
    const float bv = lbias[lane];
    if (THEN && last) {
      lds_reads_done();
      loads_but<0>();  // the requests past the last unit: their LDS is used again
      after_products();
    }
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      float v = acc[r] + bv;
      zs.put(r, v);
      if (!last) {
        v = act_fwd(v, a.act);
        hs.put(r, v);
      }
      xn[r * XS + n] = n < N ? v : 0.f;  // columns past N: a wider layer's values may have stood there
    }
    __syncthreads();
    if (last) {
      // Softmax cross-entropy of the workgroup's rows by the first wave, 16 lanes a row: exponentials side by side, then the row's
      // sum in ascending class order by one lane (the step's loss is the sum of the rows' losses; the gradient kernel, which
      // follows, adds them up).  The layer's input buffer is free: it takes the exponentials, and after them the logits' gradient.
      const int C = a.n_out, row = lane >> 4, sub = lane & 15;
      if (wave == 0 && row < rows) {
        const int m = r0 + row;
        const float* const z = xn + row * XS;
        float* const ex = xs + row * XS;
        const int y = a.labels[m];
        float mx = -INFINITY;
        for (int c = sub; c < C; c += 16) mx = fmaxf(mx, z[c]);
#pragma unroll
        for (int k = 8; k > 0; k >>= 1) mx = fmaxf(mx, __shfl_xor(mx, k, 16));
        for (int c = sub; c < C; c += 16) ex[c] = expf(z[c] - mx);
        wave_lds_order();
        float sum = 0.f;
        if (sub == 0)
          for (int c = 0; c < C; ++c) sum += ex[c];
        sum = __shfl(sum, 0, 16);
        const float lse = logf(sum) + mx, inv_sum = 1.f / sum;
        wave_lds_order();
        gfloat* const dz = dlog + (size_t)m * a.ldv;
        for (int c = sub; c < (THEN ? 256 : a.ldv); c += 16) {
          const float v = c < C ? (ex[c] * inv_sum - (c == y ? 1.f : 0.f)) * a.inv_n : 0.f;
          if (c < a.ldv) dz[c] = v;
          if (THEN) ex[c] = v;
        }
        if (sub == 0) rowl[m] = lse - z[y];
      } else if (THEN && wave == 0) {
        for (int c = sub; c < 256; c += 16) xs[row * XS + c] = 0.f;
      }
    }
  }
  if (!THEN) loads_but<0>();  // the requests past the last unit, before their LDS is given back
}

// ---- backward, part 1: dz_{u-1} = (dz_u W_u) * act'(z_{u-1}) for u = u1-1 ... max(u0, 1) -------------------------------------
// W_u is k-major for this product: its rows are the k of the sum.  ws: its first four chunks requested; buf: the LDS buffer that
// holds dz of the last unit.
__device__ __forceinline__ void chain_body(const MlpFusedArgs& a, float* smem, WStream<false>& ws, int buf, int u_hi, int u_lo) {
  const int g = blockIdx.x % a.G, r0 = (blockIdx.x / a.G) * RB;  // model, first batch row
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int rows = a.B - r0 < RB ? a.B - r0 : RB;
  const TabPtr tb = (TabPtr)a.tab[g];
  char* const own = reinterpret_cast<char*>(smem + 2 * RB * XS) + wave * WLDS;
  const float* const gate = reinterpret_cast<const float*>(own + 4 * STG + 256);
  const int n = wave * 64 + lane;    // this lane's column
  const int Kin = a.d;               // width of dz_{u-1} (u >= 1)
  float w0[32], w1[32];
  ws.start(w0);
  __syncthreads();  // dz of the last unit is in place
  for (int u = u_hi; u >= u_lo; --u, buf ^= 1) {
    const int K = u < a.L ? a.d : a.n_out;
    const float* const ds = smem + buf * RB * XS;
    float* const dn = smem + (buf ^ 1) * RB * XS;
    // read the table now: between the stores at the unit's end a pointer read would wait for each of them
    const RowStore dzs(global_ptr(tb->dz[u - 1]), a.B, a.ldd, r0, n, Kin);
    const rsrc_u32x4 zr = rsrc_settled(rsrc_words(tb->z[u - 1], (long)r0 * a.ldd * 4, ((long)(a.B - 1) * a.ldd + Kin) * 4));
#pragma unroll
    for (int r = 0; r < RB; ++r)  // z_{u-1} at the outputs this lane will hold
      load_to_lds_b32(zr, lds_addr_of(gate) + 256 * r, n < Kin ? (unsigned)(r * a.ldd + n) * 4u : 0x80000000u);
    const f32x4a acc = ws.sum(ds, K, w0, w1);
    loads_but<16>();  // z, requested before the unit's chunks (two at least)
#pragma unroll
    for (int r = 0; r < RB; ++r) {
      const float v = acc[r] * act_grad(gate[64 * r + lane], a.act);
      dzs.put(r, v);
      dn[r * XS + n] = r < rows && n < Kin ? v : 0.f;
    }
    __syncthreads();
  }
  loads_but<0>();
}

__global__ __launch_bounds__(256) void mlp_fwd_fused_kernel(const MlpFusedArgs a) {
  extern __shared__ float smem[];
  fwd_body<false>(a, smem, [] {});
}
__global__ __launch_bounds__(256) void mlp_dgrad_chain_kernel(const MlpFusedArgs a) {
  extern __shared__ float smem[];
  const int g = blockIdx.x % a.G, r0 = (blockIdx.x / a.G) * RB, tid = threadIdx.x, wave = uniform(tid >> 6);
  const int u_hi = a.u1 - 1, u_lo = a.u0 > 1 ? a.u0 : 1;
  if (u_hi < u_lo) return;
  const TabPtr tb = (TabPtr)a.tab[g];
  WStream<false> ws(a, a.p[g], tid & 63, wave, u_hi, u_lo, lds_addr_of(smem + 2 * RB * XS) + wave * WLDS);
#pragma unroll
  for (int s = 0; s < 4; ++s) ws.request(s);
  stage_rows(smem, global_ptr(u_hi < a.L ? tb->dz[u_hi] : tb->dlogits) + (size_t)r0 * (u_hi < a.L ? a.ldd : a.ldv),
             u_hi < a.L ? a.ldd : a.ldv, a.B - r0 < RB ? a.B - r0 : RB, u_hi < a.L ? a.d : a.n_out, tid);
  chain_body(a, smem, ws, 0, u_hi, u_lo);
}
// Forward through all of a model's units, then straight on into the chain of input gradients: a workgroup's rows
// need nothing from other workgroups in between (the rows' losses and the gradient of the logits are its own), so
// the two phases of a step that the plan runs back to back are one launch.  The pre-activations that the forward phase wrote to
// memory are read back by the wave that wrote them.  45 scalar registers of the weights' stream are kept in lanes of a vector register: the
// two halves' arguments and descriptors together are more than there are (neither half alone spills any).
__global__ __launch_bounds__(256) void mlp_fwd_chain_kernel(const MlpFusedArgs a) {
  extern __shared__ float smem[];
  const int g = blockIdx.x % a.G, tid = threadIdx.x, wave = uniform(tid >> 6);
  WStream<false> ws(a, a.p[g], tid & 63, wave, a.L, 1, lds_addr_of(smem + 2 * RB * XS) + wave * WLDS);
  fwd_body<true>(a, smem, [&] {
#pragma unroll
    for (int s = 0; s < 4; ++s) ws.request(s);
  });
  if (a.L >= 1) chain_body(a, smem, ws, a.L & 1, a.L, 1);
  else loads_but<0>();
}

// ---- backward, part 2: dW_u = dz_u^T x_u with the update of W_u and b_u, for every unit of the shard -----------------
// grid (strip of 32 output rows, unit, model); wave w takes the 32-column tiles w, w+4 of the strip
template <int OPT>
__global__ __launch_bounds__(256) void mlp_wgrad_update_kernel(const MlpFusedArgs a) {
  const int strip = blockIdx.x, u = a.u0 + blockIdx.y, g = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lrow = lane & 31, lgrp = lane >> 5;
  const int N = u < a.L ? a.d : a.n_out, Kin = u == 0 ? a.d_in : a.d;
  if (strip * 32 >= N) return;
  const TabPtr tb = (TabPtr)a.tab[g];
  if (u == a.L && strip == 0 && tid == 0) {
    // the step's loss: the rows' losses, which the forward kernel's workgroups left, added in ascending order
    const gfloat* rl = global_ptr(tb->rowloss);
    float t = 0.f;
    for (int m = 0; m < a.B; ++m) t += rl[m];
    *a.loss[g] = t * a.inv_n;
  }
  const gfloat* dz = global_ptr(u < a.L ? tb->dz[u] : tb->dlogits);
  const int lddz = u < a.L ? a.ldd : a.ldv;
  const gfloat* xin = global_ptr(u == 0 ? a.x[g] : tb->h[u - 1]);
  const int ldx = u == 0 ? a.ld_in : a.ldd;
  const int n = strip * 32 + lrow;
  const OptimHp hp = a.hp[g];
  // the sum runs over the batch rows: 4 groups of 8; this lane's dz values: rows 8s + 4 lgrp + e of column n
  float4 dv[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int m = 8 * s + 4 * lgrp;
    dv[s] = zero4();
    if (n < N) {
      if (m < a.B) dv[s].x = dz[(size_t)m * lddz + n];
      if (m + 1 < a.B) dv[s].y = dz[(size_t)(m + 1) * lddz + n];
      if (m + 2 < a.B) dv[s].z = dz[(size_t)(m + 2) * lddz + n];
      if (m + 3 < a.B) dv[s].w = dz[(size_t)(m + 3) * lddz + n];
    }
  }
  for (int kt = wave; kt * 32 < Kin; kt += 4) {
    const int k = kt * 32 + lrow;
    float4 xa[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int m = 8 * s + 4 * lgrp;
      xa[s] = zero4();
      if (k < Kin) {
        if (m < a.B) xa[s].x = xin[(size_t)m * ldx + k];
        if (m + 1 < a.B) xa[s].y = xin[(size_t)(m + 1) * ldx + k];
        if (m + 2 < a.B) xa[s].z = xin[(size_t)(m + 2) * ldx + k];
        if (m + 3 < a.B) xa[s].w = xin[(size_t)(m + 3) * ldx + k];
      }
    }
    // the state of the lane's 16 weights depends on addresses only: requested with the operands, not behind the products
    float4 ps[4], ms[4], vs[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int kq = kt * 32 + 8 * q + 4 * lgrp;
      if (a.keep_grads || n >= N || kq >= Kin) continue;
      const size_t ix = (size_t)a.w_off[u] + (size_t)n * Kin + kq;
      ps[q] = *reinterpret_cast<const float4*>(a.p[g] + ix);
      if (OPT == 1) {
        ms[q] = *reinterpret_cast<const float4*>(a.m[g] + ix);
        vs[q] = *reinterpret_cast<const float4*>(a.v[g] + ix);
      }
    }
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll
    for (int s = 0; s < 4; ++s) mma4(acc, xa[s], dv[s]);
    // a lane holds, for output row n = strip*32 + lrow, columns kt*32 + 8q + 4 lgrp + (0..3)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int kq = kt * 32 + 8 * q + 4 * lgrp;
      if (n >= N || kq >= Kin) continue;   // Kin is a multiple of 8: whole vectors
      const size_t ix = (size_t)a.w_off[u] + (size_t)n * Kin + kq;
      const float gr[4] = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
      if (a.keep_grads) {
        *reinterpret_cast<float4*>(a.g[g] + ix) = make_float4(gr[0], gr[1], gr[2], gr[3]);
        continue;
      }
      const float4 pv = ps[q];
      float pe[4] = {pv.x, pv.y, pv.z, pv.w}, me[4] = {0.f, 0.f, 0.f, 0.f}, ve[4] = {0.f, 0.f, 0.f, 0.f};
      if (OPT == 1) {
        const float4 mv = ms[q], vv = vs[q];
        me[0] = mv.x; me[1] = mv.y; me[2] = mv.z; me[3] = mv.w;
        ve[0] = vv.x; ve[1] = vv.y; ve[2] = vv.z; ve[3] = vv.w;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) optim_step<OPT>(pe[e], me[e], ve[e], gr[e], hp);
      if (OPT == 1) {
        *reinterpret_cast<float4*>(a.m[g] + ix) = make_float4(me[0], me[1], me[2], me[3]);
        *reinterpret_cast<float4*>(a.v[g] + ix) = make_float4(ve[0], ve[1], ve[2], ve[3]);
      }
      *reinterpret_cast<float4*>(a.p[g] + ix) = make_float4(pe[0], pe[1], pe[2], pe[3]);
    }
  }
  if (wave == 0) {
    // bias gradient: column sums of dz.  Each half-wave adds its chunks in ascending row order, element by element,
    // then the two halves are added (the order the tiled kernel uses for its row sums)
    float rs = 0.f;
    {
#pragma clang fp contract(off)
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        rs = rs + dv[s].x;
        rs = rs + dv[s].y;
        rs = rs + dv[s].z;
        rs = rs + dv[s].w;
      }
    }
    const float total = rs + __shfl_xor(rs, 32, 64);
    if (lgrp == 0 && n < N) {
      const size_t ix = (size_t)a.b_off[u] + n;
      if (a.keep_grads) {
        a.g[g][ix] = total;
      } else {
        float pe = a.p[g][ix], me = 0.f, ve = 0.f;
        if (OPT == 1) {
          me = a.m[g][ix];
          ve = a.v[g][ix];
        }
        optim_step<OPT>(pe, me, ve, total, hp);
        if (OPT == 1) {
          a.m[g][ix] = me;
          a.v[g][ix] = ve;
        }
        a.p[g][ix] = pe;
      }
    }
  }
}

hipError_t check(const MlpFusedArgs& a) {
  if (a.G < 1 || a.G > MAXG || a.B < 1 || a.B > 32 || a.d_in < 8 || a.d_in > 256 || a.d_in % 8 || a.d < 8 || a.d > 256 ||
      a.d % 8 || a.n_out < 1 || a.n_out > 256 || a.L < 0 || a.L + 1 > MLP_FUSED_MAX_UNITS || a.u0 < 0 || a.u1 > a.L + 1 ||
      a.u0 >= a.u1 || a.ld_in < a.d_in || a.ld_in % 4 || a.ldd < a.d || a.ldd % 4 || a.ldv < a.n_out)
    return hipErrorInvalidValue;
  for (int g = 0; g < a.G; ++g)
    if (!a.p[g] || !a.tab[g] || !a.x[g]) return hipErrorInvalidValue;
  return hipSuccess;
}

}  // namespace

bool mlp_fused_shape_ok(int B, int d_in, int d, int n_out, int n_units) {
  return B >= 1 && B <= 32 && d_in >= 8 && d_in <= 256 && d_in % 8 == 0 && d >= 8 && d <= 256 && d % 8 == 0 && n_out >= 1 &&
         n_out <= 256 && n_units <= MLP_FUSED_MAX_UNITS;
}

hipError_t mlp_fused_init() {
  const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&mlp_fwd_fused_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)CHAIN_LDS);
  if (e != hipSuccess) return e;
  const hipError_t e2 = hipFuncSetAttribute(reinterpret_cast<const void*>(&mlp_dgrad_chain_kernel),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)CHAIN_LDS);
  if (e2 != hipSuccess) return e2;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&mlp_fwd_chain_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)CHAIN_LDS);
}

hipError_t launch_mlp_fwd_fused(const MlpFusedArgs& a, hipStream_t s) {
  hipError_t e = check(a);
  if (e != hipSuccess) return e;
  if (a.u1 == a.L + 1 && !a.labels) return hipErrorInvalidValue;
  hipLaunchKernelGGL(mlp_fwd_fused_kernel, dim3(a.G * ((a.B + RB - 1) / RB)), dim3(256), CHAIN_LDS, s, a);
  return hipGetLastError();
}

hipError_t launch_mlp_fwd_chain(const MlpFusedArgs& a, hipStream_t s) {
  hipError_t e = check(a);
  if (e != hipSuccess) return e;
  if (a.u0 != 0 || a.u1 != a.L + 1 || !a.labels) return hipErrorInvalidValue;  // the whole model, forward and back
  hipLaunchKernelGGL(mlp_fwd_chain_kernel, dim3(a.G * ((a.B + RB - 1) / RB)), dim3(256), CHAIN_LDS, s, a);
  return hipGetLastError();
}

hipError_t launch_mlp_dgrad_chain(const MlpFusedArgs& a, hipStream_t s) {
  hipError_t e = check(a);
  if (e != hipSuccess) return e;
  if (a.u1 - 1 < (a.u0 > 1 ? a.u0 : 1)) return hipSuccess;  // no unit of the shard has an input gradient to produce
  hipLaunchKernelGGL(mlp_dgrad_chain_kernel, dim3(a.G * ((a.B + RB - 1) / RB)), dim3(256), CHAIN_LDS, s, a);
  return hipGetLastError();
}

hipError_t launch_mlp_wgrad_update(const MlpFusedArgs& a, hipStream_t s) {
  hipError_t e = check(a);
  if (e != hipSuccess) return e;
  for (int g = 0; g < a.G; ++g) {
    if (a.keep_grads ? !a.g[g] : (a.opt == 1 && (!a.m[g] || !a.v[g]))) return hipErrorInvalidValue;
    if (a.u1 == a.L + 1 && !a.loss[g]) return hipErrorInvalidValue;  // the launch with the last unit writes the step's loss
  }
  const int widest = a.d > a.n_out ? a.d : a.n_out;
  const dim3 grid((widest + 31) / 32, a.u1 - a.u0, a.G);
  if (a.opt == 1) hipLaunchKernelGGL(mlp_wgrad_update_kernel<1>, grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL(mlp_wgrad_update_kernel<0>, grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace hydra
