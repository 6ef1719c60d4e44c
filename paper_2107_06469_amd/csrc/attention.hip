// Scaled dot-product attention for bf16 activations, forward and backward, block-wise so the S x S
// score matrix never reaches HBM.
//   forward:   P = softmax(q k^T * scale [+ causal mask]),  o = P v,  lse = log sum exp (saved)
//   backward:  delta_i = sum_c do[i,c] o[i,c];  P recomputed from lse;
//              dv = P^T do;  dP = do v^T;  dS = P * (dP - delta);  dq = scale * dS k;  dk = scale * dS^T q
// Memory layout: qkv is [B*S, ld] with q of head h at columns [h*DH, h*DH+DH), k at d + ..., v at 2d + ...
// (d = H*DH); o/do are [B*S, ld_o] with head h at columns [h*DH, ...); dqkv has the layout of qkv.
//
// Matrix-core mapping (v_mfma_f32_32x32x16_bf16, 64-wide wavefronts).  A 32x32 accumulator gives lane l
// column l%32 and rows 8q+4(l/32)+e (q,e = 0..3).  Every product is arranged so that the accumulator of
// the first contraction is already in the lane layout the second contraction needs as its B operand
// (k index = accumulator row), i.e. probabilities never go through LDS:
//   forward and dq:  S^T[j,i] = K Q^T  (lane = query i, rows = keys j)  ->  O^T[c,i] += Vt[c,j] P^T[j,i]
//   dk/dv:           S[i,j]   = Q K^T  (lane = key j, rows = queries i) ->  dV^T[c,j] += dOt[c,i] P[i,j]
// The A operand of the second contraction walks a tile along its slow index (eight keys, or queries, of one
// column).  The tiles stay row-major in LDS (rows of DH values, 16-byte chunks XOR-swizzled by the row) and that
// operand comes from transposing LDS reads (ds_read_b64_tr_b16: within 16 lanes, source lane j supplies four
// consecutive columns of row j/4 and lane i receives column i of rows 0..3), two per fragment, so every tile is
// loaded once and nothing is transposed in memory.  Tiles go from memory straight into one of two LDS buffers (buffer
// loads with LDS as their destination): the loads of tile t+1 are issued when every wave has left tile t-1 and land under
// the products of tile t; one barrier per tile.  Softmax statistics
// of a query live in the two lanes l and l^32 and are combined with one cross-lane exchange.  A wavefront owns 32
// queries (or 32 keys) and loops over tiles of 64 keys (queries) shared through LDS by the four wavefronts of the
// workgroup.  All sums run in a fixed order; dq and dk/dv are separate workgroups so that no atomics are needed.
#include <algorithm>
#include <type_traits>

#include "kernels.h"
#include "launch_rules.h"
#include "lds_dma.h"
#include "wave_math.h"

namespace hydra {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

namespace {

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr float NEG_BIG = -1.0e30f;

// 2^x by the hardware instruction alone: arguments here are <= 0 up to rounding, results below the normal
// range may flush to zero, which is what a softmax weight that small is worth.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// two floats -> two bf16 in one word, round to nearest even: one v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float bf_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

__device__ __forceinline__ f32x16 mfma(const uint4& a, const uint4& b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// ---- LDS tiles of 64 rows x DH columns ---------------------------------------------------------------
// uint4 chunk (row, kc) sits at row*NCH + (kc ^ swz(row)), NCH = DH/8.
// Work item of a workgroup.  The hardware deals consecutive workgroup ids to the 8 XCDs in turn; items are numbered so
// that each XCD gets a contiguous run of them, and the 128-row blocks of one (batch, head) are consecutive items: the
// blocks that read the same K/V (or Q/dO) tiles then run on one XCD and share them through its L2, instead of
// each XCD fetching them from memory.  Returns false for the padding ids at the end of the grid.
// What a workgroup does before its first tile has landed is a third of its life at 8 tiles, so that part is kept short in all kernels:
// three multiplications instead of four integer divisions, every pointer read at once, rows read without branches (rows_at), and
// nothing that waits for one load before the next is issued.  us, before | now: forward 4 x [32 x 12 heads, 512, 64] 172 | 161,
// 8 x 32 heads, 2048, 128, causal 411 | 385; backward 490 | 453, 1239 | 1187, 4 x [8 x 16, 384, 64] 102 | 96.6.  Then descriptors of a tile by 32-bit
// scalar arithmetic from its first row (64-bit from the matrix's before, which took all scalar registers and spilled some on
// every tile), masks by one comparison, 16-byte stores: forward 160 | 145 and 34.3 | 30.8, backward 451 | 430 and 94 | 88.
// Under a causal mask the row blocks of a head have one to n_blk parts of work.  Where attn_pairs says so (launch_rules.h) a workgroup takes
// blocks i and `last` - i one after the other, the longer one first, and asks for the first tile and the fragments of the
// second under the last tile of the first: equal workgroups, half the launch latencies, K and V of a head from one L2.  us, one block | two:
// forward 8 x 32 heads, 2048, 128 362 | 339, backward 1110 | 1036; 2 x [4 x 16, 1024, 128] 66 | 49 and 198 | 156; 16 heads, 8 x 1024, 64 43 | 33
// and 113 | 94.  (Chains of three or four blocks and one resident workgroup for all of its blocks: level under a mask; without one 2 to 8 %
// behind single blocks, whose loads do not all come at once.)
struct AttnGrid { unsigned n_blk, n_bh, n_h, total, per_xcd, r_blk, r_bh, r_h; int last; };  // counts of items, reciprocals (attn_grid); last: -1 without pairs
struct AttnItem { int blk, then, bh, gi, b, h; };
// n / d for the divisor whose reciprocal the host worked out, floor(2^32 / d) (2^32 - 1 for d = 1): one too small at most
__device__ __forceinline__ unsigned div_by(unsigned n, unsigned d, unsigned rcp) {
  const unsigned q = __umulhi(n, rcp);
  return n - q * d >= d ? q + 1 : q;
}
// then: the second block of a pair, -1 where there is none.  HIGH_FIRST: the higher block is the longer one (more keys to a query).
template <bool HIGH_FIRST>
__device__ __forceinline__ bool attn_item(unsigned wg, const AttnGrid& gr, AttnItem& it) {
  // all of the grid's fields by one scalar load, not those behind the test by another
  asm volatile("" ::"s"(gr.total), "s"(gr.per_xcd), "s"(gr.n_blk), "s"(gr.n_bh), "s"(gr.n_h), "s"(gr.r_blk), "s"(gr.r_bh), "s"(gr.r_h), "s"(gr.last));
  const unsigned id = (wg & 7) * gr.per_xcd + (wg >> 3);
  if (id >= gr.total || (wg >> 3) >= gr.per_xcd) return false;
  const unsigned u = div_by(id, gr.n_blk, gr.r_blk), gi = div_by(u, gr.n_bh, gr.r_bh), bh = u - gi * gr.n_bh;
  const unsigned b = div_by(bh, gr.n_h, gr.r_h);
  const int low = (int)(id - u * gr.n_blk), high = gr.last - low;
  const bool pair = gr.last >= 0;
  it = {pair && HIGH_FIRST ? high : low, !pair ? -1 : HIGH_FIRST ? low : high, (int)bh, (int)gi, (int)b, (int)(bh - b * gr.n_h)};
  return true;
}
// Bytes from the start of a head's columns in one row to the end of those columns in the last of `rows` rows (none: 0): what a
// descriptor that begins there spans.  Rows behind it read as zero and are not written, without a branch around the access
// (between branches every load fetched its pointer anew and waited for it).
template <int DH>
__device__ __forceinline__ int span_of(int rows, int ld) { return rows > 0 ? ((rows - 1) * ld + DH) * 2 : 0; }
template <int DH>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rows_at(const bf16_t* first, int rows, int ld) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(first), 0, span_of<DH>(min(rows, 32), ld), 0x00020000);
}
// A lane's row, from a tile's or a block's first, for offsets into such descriptors.  FAR: a sequence shorter than 64 rows may have rows of up to 2 GiB in
// all, and the offsets of the 64 rows of a tile then come round, past 32 bits, to rows that are there; past the sequence a row counts as its end.
// Kernels of their own: the minimum costs the others, whose registers are then dealt out another way, up to 1 %.
template <bool FAR>
__device__ __forceinline__ unsigned lane_row(int row, int S) { return (unsigned)(FAR ? min(row, S) : row); }
__device__ __forceinline__ uint4 row_chunk(__amdgpu_buffer_rsrc_t rs, unsigned voff) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rs, voff, 0, 0));
}

// XOR term of a row's chunk index.  Two access patterns must each spread over all 64 banks: a 128-bit row read
// (16 consecutive rows at one chunk index per pass) and a transposing 64-bit read (per pass of 32 lanes: rows 4g..4g+3 x
// 4 neighbouring chunks x both halves).  A row of DH = 128 fills the banks once: the 16 rows need 16 different terms,
// and 4 consecutive rows must move the group of 4 chunks to the 4 different groups: 4*(row%4) + (row/4)%4.  A row of
// DH = 64 fills half of the banks and rows of equal parity share them: the 8 such rows among 16 need 8 different terms,
// and the 2 among 4 consecutive rows must move the group of 4 chunks to different groups: 4*((row/2)%2) + (row/4)%4.
template <int DH>
__device__ __forceinline__ int swz(int row) {
  if (DH == 128) return 4 * (row & 3) + ((row >> 2) & 3);
  return 4 * ((row >> 1) & 1) + ((row >> 2) & 3);
}

// A tile's way into LDS: load i of wave w fills slots [(4 i + w) 64, + 64), lane l slot l, with the chunk that belongs there.
// Rows past the last one read as zero (the descriptor ends with it; it is made per tile, so that the lane's
// offset is the same for every tile).  ONE: the rows of load i are those of load 0 plus 16 or 32 i, which have the same XOR
// terms, so one offset per lane serves every load and the descriptor, in scalar registers, moves on: for the kernel
// that has no vector register to spare (the others would only spill scalar registers for it).
template <int DH, bool ONE = false, bool SETTLE = false, bool FAR = false>
struct TileDma {
  static constexpr int NCH = DH / 8, N = 64 * NCH / 256, STEP = 256 / NCH;  // loads per wave, rows between them
  unsigned voff[ONE ? 1 : N];
  __device__ __forceinline__ void init(int ld, int S, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < (ONE ? 1 : N); ++i) {
      const int sl = (4 * i + wave) * 64 + lane, row = sl / NCH;
      voff[i] = (lane_row<FAR>(row, S) * (unsigned)ld + (unsigned)((sl % NCH) ^ swz<DH>(row)) * 8u) * 2u;
    }
  }
  // first: the tile's first row at the head's columns; rows: how many there are from it on (at least one)
  __device__ __forceinline__ void issue(const bf16_t* first, int rows, int ld, unsigned lds_addr, int wave) const {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int skip = ONE ? STEP * i : 0;
      const uint64_t p = (uint64_t)(uintptr_t)(first + (size_t)skip * ld);
      rsrc_u32x4 rs = {(unsigned)p, (unsigned)(p >> 32) & 0xffffu, (unsigned)span_of<DH>(min(rows, 64) - skip, ld), 0x00020000u};
      if constexpr (SETTLE) {
        rs.x = __builtin_amdgcn_readfirstlane(rs.x), rs.y = __builtin_amdgcn_readfirstlane(rs.y), rs.z = __builtin_amdgcn_readfirstlane(rs.z);
        rs = rsrc_settled(rs);
      }
      load_to_lds_b128(rs, lds_addr + (unsigned)((4 * i + wave) * 64 * 16), voff[ONE ? 0 : i]);
    }
  }
};
// Every load of this wave has landed.  (A wait written in inline asm the compiler does not count: it waited again, inside the loop, for
// the fragments loaded before it, and with them for the next tile's loads.  For the same reason it stands at the end of every tile,
// on all paths, and ahead of the stores of an item that ends there: their way to memory is under the next item's first tile.)
__device__ __forceinline__ void loads_landed() {
  __builtin_amdgcn_s_waitcnt(0xf70);  // vmcnt(0)
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ unsigned lds_byte_addr(const void* p) {
  return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const char*)reinterpret_cast<const char*>(p);
}

// A operand along the slow index of a row-major tile: lane l gets, for column col0 + l%32, the values of rows
// row0 + 4g + {0..3} and row0 + 8 + 4g + {0..3} (g = l/32), the k order the accumulator rows of the first product
// have.  Two transposing reads: in the 16-lane group, source lane j reads 8 bytes at row 4g + j/4, column
// 16*(group&1) + 4*(j%4) of the block.
// The lane's part of an address is computed once: for rows row0 + l%32 (row0 a multiple of
// NCH) the XOR term depends on the lane alone, so a tile's later row blocks, and a second tile that follows the first
// in LDS, are constant offsets from one pointer per chunk (they go into the instruction's offset field).
template <int DH>
__device__ __forceinline__ const uint4* rows_base(const uint4* tile, int li, int kc) {
  constexpr int NCH = DH / 8;
  return tile + li * NCH + (kc ^ swz<DH>(li));
}
// byte addresses of the two transposing reads (rows r0 and r0 + 8) for row0 = 0; row0 (a multiple of 16) adds
// row0 * NCH * 16 to both
struct ColsBase { unsigned a0, a1; };
template <int DH>
__device__ __forceinline__ ColsBase cols_base(const uint4* tile, int col0, int lane) {
  constexpr int NCH = DH / 8;
  const int j = lane & 15, grp = lane >> 4;
  const int col = col0 + 16 * (grp & 1) + 4 * (j & 3), kc = col >> 3, half = (col >> 2) & 1;
  const int r0 = 4 * (grp >> 1) + (j >> 2), r1 = r0 + 8;
  const unsigned base = lds_byte_addr(tile);
  ColsBase b;
  b.a0 = base + (unsigned)((r0 * NCH + (kc ^ swz<DH>(r0))) * 16 + half * 8);
  b.a1 = base + (unsigned)((r1 * NCH + (kc ^ swz<DH>(r1))) * 16 + half * 8);
  return b;
}
// At DH = 128 a row is 256 bytes and the bits of a chunk's number in an address are XOR-ed with the row's term, so all of a lane's
// bases follow from one of each kind: chunk 2 kk more is address ^ 32 kk; column block c is ^ 64 c, and row r0 + 8 is ^ 32 (its
// term differs in one bit) and 8 rows.  The dk/dv kernel, which has no register to spare, works them out per 32 queries (14
// instructions) instead of keeping 16, so that no K or V fragment goes to scratch (a reload waits for the next tile's loads).
__device__ __forceinline__ void bases128(const uint4* (&rows)[8], ColsBase (&cols)[4]) {
  unsigned r = lds_byte_addr(rows[0]), c0 = cols[0].a0;
  asm("" : "+v"(r));  // not to be hoisted
  asm("" : "+v"(c0));
#pragma unroll
  for (int kk = 1; kk < 8; ++kk)
    rows[kk] = (const uint4*)(__attribute__((address_space(3))) const uint4*)(uintptr_t)(r ^ (unsigned)(kk * 32));
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    cols[c].a0 = c0 ^ (unsigned)(c * 64);
    cols[c].a1 = (c0 ^ (unsigned)(c * 64 + 32)) + 8u * 16u * 16u;
  }
}
template <int DH>
__device__ __forceinline__ uint4 read_cols_at(const ColsBase& b, unsigned off) {
  typedef __attribute__((ext_vector_type(4))) short s16x4;
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(b.a0 + off));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(b.a1 + off));
  const uint2 l = __builtin_bit_cast(uint2, lo), h = __builtin_bit_cast(uint2, hi);
  return make_uint4(l.x, l.y, h.x, h.y);
}

__device__ __forceinline__ uint4 pack_half(const f32x16& p, int x) {
  return make_uint4(pack2(p[8 * x], p[8 * x + 1]), pack2(p[8 * x + 2], p[8 * x + 3]), pack2(p[8 * x + 4], p[8 * x + 5]),
                    pack2(p[8 * x + 6], p[8 * x + 7]));
}

// An accumulator's 32 columns of 32 rows (lane l: row l%32, columns 8q + 4(l/32) + e) as bf16 to the rows that a descriptor
// begins with; off: the lane's row and the block's first column.  The two lanes of a row trade halves so that a lane stores 8 columns
// at once: two stores of 16 bytes (four of 8 before).  Rows past the descriptor's end are dropped.
__device__ __forceinline__ void store_block(const f32x16& v, float f, __amdgpu_buffer_rsrc_t rs, unsigned off, int g) {
  typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
#pragma unroll
  for (int q = 0; q < 4; q += 2) {
    const auto lo = __builtin_amdgcn_permlane32_swap(pack2(v[4 * q] * f, v[4 * q + 1] * f), pack2(v[4 * q + 4] * f, v[4 * q + 5] * f), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(pack2(v[4 * q + 2] * f, v[4 * q + 3] * f), pack2(v[4 * q + 6] * f, v[4 * q + 7] * f), false, false);
    const u32x4 w = {lo[0], hi[0], lo[1], hi[1]};
    __builtin_amdgcn_raw_buffer_store_b128(w, rs, off + (unsigned)(8 * q + 8 * g) * 2u, 0, 0);
  }
}
// One float of each of a wave's 32 rows, from the lower half of the wave
__device__ __forceinline__ void store_stat(float v, float* first, int rows, int li, int g) {
  const uint64_t p = (uint64_t)(uintptr_t)first;
  const uint64_t u = (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane((unsigned)(p >> 32)) << 32 | (unsigned)__builtin_amdgcn_readfirstlane((unsigned)p);
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((float*)(uintptr_t)u, 0, __builtin_amdgcn_readfirstlane(max(min(rows, 32), 0) * 4), 0x00020000);
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, g ? 0x7ffffff0 : li * 4, 0, 0);
}

// ---- forward ---------------------------------------------------------------------------------------------
// Bound by the VALU: a score costs a multiply-add, an exponential (four times a plain instruction's cycles), an addition, half a
// maximum, half a conversion and (where a maximum grew) a multiplication, 8 issue slots for 1.3 of MFMA at DH = 64.  120
// registers (four waves per SIMD; 153 when tiles passed through registers).
template <int DH, bool FAR = false>
__global__ __launch_bounds__(256, DH == 64 ? 4 : 2) void attn_fwd_kernel(const AttnArgs a, const AttnGrid gr) {
  constexpr int NK = DH / 16, NC = DH / 32, NCH = DH / 8;
  extern __shared__ __attribute__((aligned(256))) uint4 lds[];
  // two buffers of K [64][NCH], V [64][NCH]
  uint4* tK = lds;
  uint4* tV = lds + 64 * NCH;
  constexpr int BUF = 2 * 64 * NCH;  // chunks per buffer
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 31, g = lane >> 5;
  AttnItem item;
  if (!attn_item<true>(blockIdx.x, gr, item)) return;
  const int d = a.H * DH, ld = a.ld_qkv;
  const float sc = a.scale * LOG2E;
  TileDma<DH, false, false, FAR> dma;
  dma.init(ld, a.S, wave, lane);
  const unsigned lds0 = lds_byte_addr(lds), q_off = lane_row<FAR>(li, a.S) * (unsigned)ld * 2u + 16u * g;
  auto fetch = [&](const bf16_t* k, int rows, unsigned buf) {  // k: the tile's first key
    dma.issue(k, rows, ld, lds0 + buf, wave);
    dma.issue(k + d, rows, ld, lds0 + buf + 64 * NCH * 16, wave);
  };
  const bf16_t* const base = a.qkv[item.gi] + (size_t)item.b * a.S * ld + item.h * DH;
  fetch(base + d, a.S, 0);
  uint4 qf[NK];
  auto load_q = [&](int blk) {
    const int row0 = blk * 128 + wave * 32;
    const __amdgpu_buffer_rsrc_t q_rows = rows_at<DH>(base + (size_t)row0 * ld, a.S - row0, ld);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) qf[kk] = row_chunk(q_rows, q_off + 32u * kk);
    asm volatile("" ::: "memory");
  };
  load_q(item.blk);
  const uint4* kr[NK];   // K rows l%32, chunk 2kk + g
  ColsBase vc[NC];       // V columns c*32.., rows from 0
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) kr[kk] = rows_base<DH>(tK, li, 2 * kk + g);
#pragma unroll
  for (int c = 0; c < NC; ++c) vc[c] = cols_base<DH>(tV, c * 32, lane);
  f32x16 oacc[NC];
  float m_run, l_run;
  int t = 0, n_tiles;
  const bf16_t* ktile = base + d;
  auto begin = [&] {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[c][r] = 0.f;
    m_run = NEG_BIG, l_run = 0.f, t = 0;
    n_tiles = (a.causal ? min(a.S, item.blk * 128 + 128) + 63 : a.S + 63) / 64;
  };
  begin();
  loads_landed();
  auto tile = [&](auto buf_) {
    constexpr int B = decltype(buf_)::value * BUF;  // chunks to the tile's buffer
    const int j0 = t * 64, row0 = item.blk * 128 + wave * 32, iq = row0 + li;  // this lane's query
    const bool last = t + 1 == n_tiles, more = !last || item.then >= 0;
    __syncthreads();
    ktile = last ? base + d : ktile + (size_t)64 * ld;
    if (more) fetch(ktile, last ? a.S : a.S - j0 - 64, (unsigned)((BUF - B) * 16));
    f32x16 s[2];
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[sub][r] = 0.f;
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) s[sub] = mfma(kr[kk][B + sub * 32 * NCH], qf[kk], s[sub]);
    }
    if (last && more) load_q(item.then);
    // Masking is needed only in tiles that reach past the sequence end or, with a causal mask, past the
    // wave's first query; the scale is folded into the exponent's multiply-add.
    const bool edge = j0 + 64 > a.S || (a.causal && j0 + 63 > row0);
    float mx = NEG_BIG;
    if (edge) {
      const int keys = (a.causal ? min(a.S, iq + 1) : a.S) - j0 - 4 * g;  // keys the query sees, from the lane's first on
#pragma unroll
      for (int sub = 0; sub < 2; ++sub)
#pragma unroll
        for (int r = 0; r < 16; ++r) s[sub][r] = sub * 32 + 8 * (r >> 2) + (r & 3) < keys ? s[sub][r] : NEG_BIG;
    }
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[sub][r]);
    // The output accumulators, the largest part of a wave's registers, are rescaled only when some query's maximum has
    // grown.  (Letting it lag by up to 2^8 makes the kernel 4-5 % faster and the results 0.7 % less exact: the largest
    // weight is then no longer exactly 1 in bf16.)
    const float2 mh = wave_swap32(mx);
    mx = fmaxf(mh.x, mh.y) * sc;
    float alpha = 1.f;
    if (__any(mx > m_run)) {
      const float m_new = fmaxf(m_run, mx);
      alpha = fast_exp2(m_run - m_new);
      m_run = m_new;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[c][r] *= alpha;
    }
    float rs = 0.f;
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = fast_exp2(fmaf(s[sub][r], sc, -m_run));
        s[sub][r] = p;
        rs += p;
      }
    const float2 rh = wave_swap32(rs);  // a query's keys are shared by lanes l and l^32
    l_run = fmaf(l_run, alpha, rh.x + rh.y);
#pragma unroll
    for (int sub = 0; sub < 2; ++sub)
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const uint4 pf = pack_half(s[sub], x);
#pragma unroll
        for (int c = 0; c < NC; ++c) oacc[c] = mfma(read_cols_at<DH>(vc[c], (unsigned)((B + (sub * 32 + 16 * x) * NCH) * 16)), pf, oacc[c]);
      }
    loads_landed();
    ++t;
    if (!last) return true;
    const float inv = 1.f / l_run;
    const __amdgpu_buffer_rsrc_t o_rows = rows_at<DH>(a.o[item.gi] + ((size_t)item.b * a.S + row0) * a.ld_o + item.h * DH, a.S - row0, a.ld_o);
#pragma unroll
    for (int c = 0; c < NC; ++c) store_block(oacc[c], inv, o_rows, lane_row<FAR>(li, a.S) * (unsigned)a.ld_o * 2u + c * 64u, g);
    store_stat((m_run + log2f(l_run)) * LN2, a.lse[item.gi] + (size_t)item.bh * a.S + row0, a.S - row0, li, g);
    item.blk = item.then, item.then = -1;
    begin();
    return more;
  };
  while (tile(std::integral_constant<int, 0>()) && tile(std::integral_constant<int, 1>())) {
  }
}

// ---- backward, dq (also writes delta) ------------------------------------------------------------------
// The lane's part (chunks 2 kk + g of a row's DH columns) of delta = sum of do * o: the two bodies below that compute it take
// the same operations in the same order.  This order, the row sums' (a tile's 64 keys, then the running sum) and dP - delta
// after the product are part of the results: tests hold them to recorded bits.
template <int NK>
__device__ __forceinline__ float delta_part(const uint4 (&dof)[NK], const uint4 (&of)[NK]) {
#pragma clang fp contract(off)
  float delta = 0.f;
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) {
    const uint32_t dw[4] = {dof[kk].x, dof[kk].y, dof[kk].z, dof[kk].w}, ow[4] = {of[kk].x, of[kk].y, of[kk].z, of[kk].w};
#pragma unroll
    for (int e = 0; e < 4; ++e) delta += fmaf(bf_lo(dw[e]), bf_lo(ow[e]), bf_hi(dw[e]) * bf_hi(ow[e]));
  }
  return delta;
}

template <int DH, bool ONE_ITEM, bool SETTLE = ONE_ITEM, bool FAR = false>
__device__ __forceinline__ void dq_body(const AttnBwdArgs& a, const AttnGrid& gr, int wg) {
  constexpr int NK = DH / 16, NC = DH / 32, NCH = DH / 8;
  extern __shared__ __attribute__((aligned(256))) uint4 lds[];
  // two buffers of K [64][NCH], V [64][NCH]
  uint4* tK = lds;
  constexpr int BUF = 2 * 64 * NCH;  // chunks per buffer
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 31, g = lane >> 5;
  AttnItem item;
  if (!attn_item<true>(wg, gr, item)) return;
  const int d = a.H * DH, ld = a.ld_qkv;
  const float sc = a.scale * LOG2E;
  TileDma<DH, false, SETTLE, FAR> dma;
  dma.init(ld, a.S, wave, lane);
  const unsigned lds0 = lds_byte_addr(lds);
  // every pointer at once, so that their loads are one wait
  const size_t seq = (size_t)item.b * a.S;
  const bf16_t* const base = a.qkv[item.gi] + seq * ld + item.h * DH;
  const bf16_t* const dobase = a.dout[item.gi] + seq * a.ld_o + item.h * DH;
  const bf16_t* const obase = a.o[item.gi] + seq * a.ld_o + item.h * DH;
  const float* const lse = a.lse[item.gi] + (size_t)item.bh * a.S;
  float* const delta_out = a.delta[item.gi] + (size_t)item.bh * a.S;
  bf16_t* const dqbase = a.dqkv[item.gi] + seq * ld + item.h * DH;
  auto fetch = [&](const bf16_t* k, int rows, unsigned buf) {  // k: the tile's first key
    dma.issue(k, rows, ld, lds0 + buf, wave);
    dma.issue(k + d, rows, ld, lds0 + buf + 64 * NCH * 16, wave);
  };
  uint4 qf[NK], dof[NK], of[NK];
  float lse_in;
  auto load_rows = [&](int blk) {
    const int row0 = blk * 128 + wave * 32, left = a.S - row0;
    const __amdgpu_buffer_rsrc_t q_rows = rows_at<DH>(base + (size_t)row0 * ld, left, ld);
    const __amdgpu_buffer_rsrc_t do_rows = rows_at<DH>(dobase + (size_t)row0 * a.ld_o, left, a.ld_o);
    const bf16_t* const orow = obase + (size_t)min(row0 + li, a.S - 1) * a.ld_o + 8 * g;  // past the end: a row whose products nobody stores
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      qf[kk] = row_chunk(q_rows, lane_row<FAR>(li, a.S) * (unsigned)ld * 2u + 32u * kk + 16u * g);
      dof[kk] = row_chunk(do_rows, lane_row<FAR>(li, a.S) * (unsigned)a.ld_o * 2u + 32u * kk + 16u * g);
      of[kk] = *reinterpret_cast<const uint4*>(orow + 16 * kk);
    }
    const __amdgpu_buffer_rsrc_t lse_rows =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(lse + row0), 0, max(min(left, 32), 0) * 4, 0x00020000);
    lse_in = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(lse_rows, li * 4, 0, 0));
    asm volatile("" ::: "memory");
  };
  fetch(base + d, a.S, 0);
  load_rows(item.blk);
  const uint4* kr[NK];   // K rows l%32, chunk 2kk + g; V is 64 rows further on
  ColsBase kc_[NC];      // K columns c*32.., rows from 0
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) kr[kk] = rows_base<DH>(tK, li, 2 * kk + g);
#pragma unroll
  for (int c = 0; c < NC; ++c) kc_[c] = cols_base<DH>(tK, c * 32, lane);
  f32x16 acc[NC];
  float lse2, delta;
  int t = 0, n_tiles = 0;
  const bf16_t* ktile = base + d;
  loads_landed();
  auto tile = [&](auto buf_) {
    constexpr int B = decltype(buf_)::value * BUF;  // chunks to the tile's buffer
    __syncthreads();
    if (t == 0) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[c][r] = 0.f;
      n_tiles = (a.causal ? min(a.S, item.blk * 128 + 128) + 63 : a.S + 63) / 64;
      const float2 dh = wave_swap32(delta_part<NK>(dof, of));
      delta = dh.x + dh.y;
      lse2 = lse_in * LOG2E;
    }
    const int j0 = t * 64, row0 = item.blk * 128 + wave * 32, iq = row0 + li;
    const bool last = t + 1 == n_tiles, more = !last || (!ONE_ITEM && item.then >= 0);
    ktile = last ? base + d : ktile + (size_t)64 * ld;
    if (more) fetch(ktile, last ? a.S : a.S - j0 - 64, (unsigned)((BUF - B) * 16));
    const bool edge = j0 + 64 > a.S || (a.causal && j0 + 63 > row0);
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        s = mfma(kr[kk][B + sub * 32 * NCH], qf[kk], s);
        dp = mfma(kr[kk][B + (64 + sub * 32) * NCH], dof[kk], dp);
      }
      if (edge) {
        const int keys = (a.causal ? min(a.S, iq + 1) : a.S) - j0 - 4 * g;  // keys the query sees, from the lane's first on
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = sub * 32 + 8 * (r >> 2) + (r & 3) < keys ? s[r] : NEG_BIG;
      }
      if (sub == 1 && last && more) load_rows(item.then);
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = fast_exp2(fmaf(s[r], sc, -lse2)) * (dp[r] - delta);
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const uint4 df = pack_half(s, x);
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = mfma(read_cols_at<DH>(kc_[c], (unsigned)((B + (sub * 32 + 16 * x) * NCH) * 16)), df, acc[c]);
      }
    }
    loads_landed();
    ++t;
    if (!last) return true;
    const __amdgpu_buffer_rsrc_t dq_rows = rows_at<DH>(dqbase + (size_t)row0 * ld, a.S - row0, ld);
#pragma unroll
    for (int c = 0; c < NC; ++c) store_block(acc[c], a.scale, dq_rows, lane_row<FAR>(li, a.S) * (unsigned)ld * 2u + c * 64u, g);
    store_stat(delta, delta_out + row0, a.S - row0, li, g);
    item.blk = item.then, item.then = -1;
    t = 0;
    return more;
  };
  while (tile(std::integral_constant<int, 0>()) && tile(std::integral_constant<int, 1>())) {
  }
}

// ---- backward, dk and dv -----------------------------------------------------------------------------------
// Two waves per SIMD at DH = 128 (256 registers, no scratch: values that a tile needs once are worked out again from own_lane; 376, one wave, when tiles passed through registers and the
// accumulators moved between the two register files on every tile), three at DH = 64 (164; 200 before).  Together with
// the dq kernel, us before | now: 8 x 32 heads, 2048, 128, causal 1645 | 1250, 2 x [4 x 16, 1024, 128] 360 | 269,
// 4 x [32 x 12 heads, 512, 64] 527 | 480.  Held to one wave per SIMD at DH = 128: 1440; with its 16 LDS bases kept instead of
// bases128 (64 bytes of scratch, K and V fragments among them): 1362.
// OWN: the kernel works out delta itself instead of reading what the dq kernel left.
// The lane's number, worked out where it is used: kept in a register, or in scratch, it costs more than two instructions a tile
__device__ __forceinline__ unsigned own_lane() {
  unsigned l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}
template <int DH, bool OWN, bool ONE_ITEM = OWN, bool FAR = false>
__device__ __forceinline__ void dkv_body(const AttnBwdArgs& a, const AttnGrid& gr, int wg) {
  constexpr int NK = DH / 16, NC = DH / 32, NCH = DH / 8;
  extern __shared__ __attribute__((aligned(256))) uint4 lds[];
  // two buffers of Q [64][NCH], dO [64][NCH], then two of [2][64]: lse*log2e, delta
  uint4* tQ = lds;
  constexpr int BUF = 2 * 64 * NCH;  // chunks per buffer
  float* const st = reinterpret_cast<float*>(lds + 2 * BUF);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), li = lane & 31, g = lane >> 5;
  AttnItem item;
  if (!attn_item<false>(wg, gr, item)) return;
  const int d = a.H * DH, ld = a.ld_qkv, n_tiles = (a.S + 63) / 64;
  const float sc = a.scale * LOG2E;
  TileDma<DH, DH == 128, OWN, FAR> dma_q, dma_o;
  dma_q.init(ld, a.S, wave, lane);
  dma_o.init(a.ld_o, a.S, wave, lane);
  const unsigned lds0 = lds_byte_addr(lds), row_off = lane_row<FAR>(li, a.S) * (unsigned)ld * 2u + 16u * g;
  const size_t seq = (size_t)item.b * a.S;
  const bf16_t* const base = a.qkv[item.gi] + seq * ld + item.h * DH;
  const bf16_t* const dobase = a.dout[item.gi] + seq * a.ld_o + item.h * DH;
  const bf16_t* const obase = OWN ? a.o[item.gi] + seq * a.ld_o + item.h * DH : nullptr;
  const float* const stat = (wave == 0 ? a.lse[item.gi] : a.delta[item.gi]) + (size_t)item.bh * a.S;  // wave 1 reads delta
  bf16_t* const dkbase = a.dqkv[item.gi] + seq * ld + d + item.h * DH;
  auto first_tile = [&](int blk) { return a.causal ? blk * 2 : 0; };  // queries before the workgroup's first key see none of its keys
  float pst = 0.f;
  uint4 own_do[NK], own_o[NK];
  auto fetch = [&](int t, unsigned buf) {
    const int left = a.S - t * 64;
    // threads 0..63: lse*log2e, 64..127: delta of query 64 t + tid%64 (zero past the last query); the other waves read nothing
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(stat + t * 64), 0, wave < (OWN ? 1 : 2) ? min(left, 64) * 4 : 0, 0x00020000);
    pst = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, own_lane() * 4, 0, 0));
    dma_q.issue(base + (size_t)t * 64 * ld, left, ld, lds0 + buf, wave);
    dma_o.issue(dobase + (size_t)t * 64 * a.ld_o, left, a.ld_o, lds0 + buf + 64 * NCH * 16, wave);
    if (OWN && wave >= 2) {  // waves 2 and 3: 32 queries each, two lanes to a query as in the dq kernel
      const int i = t * 64 + (wave - 2) * 32 + li;
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        own_do[kk] = own_o[kk] = make_uint4(0, 0, 0, 0);
        if (i < a.S) {
          const size_t off = (size_t)i * a.ld_o + 16 * kk + 8 * g;
          own_do[kk] = *reinterpret_cast<const uint4*>(dobase + off);
          own_o[kk] = *reinterpret_cast<const uint4*>(obase + off);
        }
      }
    }
  };
  auto put_stats = [&](float* stb) {
    if (wave < (OWN ? 1 : 2)) stb[wave * 64 + own_lane()] = wave == 0 ? pst * LOG2E : pst;
    if (OWN && wave >= 2) {
      const float2 dh = wave_swap32(delta_part<NK>(own_do, own_o));
      if (g == 0) stb[64 + (wave - 2) * 32 + li] = dh.x + dh.y;
    }
  };
  uint4 kf[NK], vf[NK];
  auto load_kv = [&](int blk) {
    const int row0 = blk * 128 + wave * 32;
    const bf16_t* const k = base + (size_t)row0 * ld + d;
    const __amdgpu_buffer_rsrc_t k_rows = rows_at<DH>(k, a.S - row0, ld), v_rows = rows_at<DH>(k + d, a.S - row0, ld);
#pragma unroll
    for (int kk = 0; kk < NK; ++kk) {
      kf[kk] = row_chunk(k_rows, row_off + 32u * kk);
      vf[kk] = row_chunk(v_rows, row_off + 32u * kk);
    }
    asm volatile("" ::: "memory");
  };
  int t = first_tile(item.blk);
  fetch(t, 0);
  load_kv(item.blk);
  put_stats(st);
  f32x16 dk[NC], dv[NC];
  auto clear = [&] {
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) dk[c][r] = dv[c][r] = 0.f;
  };
  clear();
  const uint4* qr[NK];   // Q rows l%32, chunk 2kk + g; dO is 64 rows further on
  ColsBase qc[NC];       // Q columns c*32.., rows from 0
#pragma unroll
  for (int kk = 0; kk < NK; ++kk) qr[kk] = rows_base<DH>(tQ, li, 2 * kk + g);
#pragma unroll
  for (int c = 0; c < NC; ++c) qc[c] = cols_base<DH>(tQ, c * 32, lane);
  loads_landed();
  auto tile = [&](auto buf_) {
    constexpr int B = decltype(buf_)::value * BUF;  // chunks to the tile's buffer
    const float* const stb = st + decltype(buf_)::value * 128;
    const int i0 = t * 64, row0 = item.blk * 128 + wave * 32;  // the wave's first key
    const bool last = t + 1 == n_tiles, more = !last || (!ONE_ITEM && item.then >= 0);
    __syncthreads();
    if (more) fetch(last ? first_tile(item.then) : t + 1, (unsigned)((BUF - B) * 16));
    // queries past the end, or (causal) queries that precede some key of this wave, need the mask
    const bool edge = i0 + 64 > a.S || (a.causal && i0 < row0 + 31);
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      if constexpr (DH == 128) bases128(qr, qc);
      f32x16 s, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
#pragma unroll
      for (int kk = 0; kk < NK; ++kk) {
        s = mfma(qr[kk][B + sub * 32 * NCH], kf[kk], s);
        dp = mfma(qr[kk][B + (64 + sub * 32) * NCH], vf[kk], dp);
      }
      f32x16 ds;
      if (edge) {
        // queries that see the key: from `seen` on, `n` of them, both counted from the lane's first
        const int l = own_lane(), i1 = i0 + 4 * (l >> 5), seen = a.causal ? row0 + (l & 31) - i1 : -i1, n = max(a.S - i1 - seen, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = (unsigned)(sub * 32 + 8 * (r >> 2) + (r & 3) - seen) < (unsigned)n ? s[r] : NEG_BIG;
      }
      if (sub == 1 && last && more) load_kv(item.then);
      const float* const stl = stb + 4 * (DH == 128 ? (int)(own_lane() >> 5) : g);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int il = sub * 32 + 8 * (r >> 2) + (r & 3);
        const float p = fast_exp2(fmaf(s[r], sc, -stl[il]));
        s[r] = p;
        ds[r] = p * (dp[r] - stl[64 + il]);
      }
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        const uint4 pf = pack_half(s, x), df = pack_half(ds, x);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          dv[c] = mfma(read_cols_at<DH>(qc[c], (unsigned)((B + (64 + sub * 32 + 16 * x) * NCH) * 16)), pf, dv[c]);
          dk[c] = mfma(read_cols_at<DH>(qc[c], (unsigned)((B + (sub * 32 + 16 * x) * NCH) * 16)), df, dk[c]);
        }
      }
    }
    if (more) put_stats(st + (1 - decltype(buf_)::value) * 128);
    loads_landed();
    ++t;
    if (!last) return true;
    const bf16_t* const ok = dkbase + (size_t)row0 * ld;
    const __amdgpu_buffer_rsrc_t dk_rows = rows_at<DH>(ok, a.S - row0, ld), dv_rows = rows_at<DH>(ok + d, a.S - row0, ld);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      store_block(dk[c], a.scale, dk_rows, lane_row<FAR>(li, a.S) * (unsigned)ld * 2u + c * 64u, g);
      store_block(dv[c], 1.f, dv_rows, lane_row<FAR>(li, a.S) * (unsigned)ld * 2u + c * 64u, g);
    }
    item.blk = item.then, item.then = -1;
    t = first_tile(item.blk);
    clear();
    return more;
  };
  while (tile(std::integral_constant<int, 0>()) && tile(std::integral_constant<int, 1>())) {
  }
}

// Single row blocks need 128 registers at DH = 64, four waves per SIMD; pairs, with the rows of the next block on their way, 156 (us, all as
// pairs | apart, both halves of the pass: 4 x [32 x 12 heads, 512, 64] 433 | 422, 4 x [8 x 12, 2048, 64] 1358 | 1326).
template <int DH, bool PAIRS, bool FAR = false>
__global__ __launch_bounds__(256, DH == 64 ? (PAIRS ? 3 : 4) : 2) void attn_bwd_dq_kernel(const AttnBwdArgs a, const AttnGrid gr) {
  dq_body<DH, !PAIRS, false, FAR>(a, gr, blockIdx.x);
}
template <int DH, bool FAR = false>
__global__ __launch_bounds__(256, DH == 64 ? 3 : 2) void attn_bwd_dkv_kernel(const AttnBwdArgs a, const AttnGrid gr) {
  dkv_body<DH, false, false, FAR>(a, gr, blockIdx.x);
}
// Small launches: both halves of the backward pass side by side, dk/dv (the longer one) first.  They share nothing but delta,
// which the dk/dv workgroups then work out themselves from rows of dO and O (same bits): a few percent more work for
// one launch and one latency chain less.
// Backward pass, two launches | one, us: 4 x [8 x 4 heads, 128, 64] 17.0 | 10.5, 1 x [4 x 8, 100, 128] 25.5 | 16.1, 2 x [2 x 4, 512, 64]
// 31.6 | 20.6, 1 x [1 x 4, 2048, 128] causal 166 | 131, 4 x [8 x 4, 256, 64] (256 row blocks) 24.4 | 18.3.
template <int DH>
__global__ __launch_bounds__(256, DH == 64 ? 2 : 1) void attn_bwd_both_kernel(const AttnBwdArgs a, const AttnGrid gr) {
  const int half = gridDim.x / 2;
  if ((int)blockIdx.x < half) dkv_body<DH, true>(a, gr, blockIdx.x);
  else dq_body<DH, true>(a, gr, blockIdx.x - half);
}

template <int DH> constexpr size_t fwd_lds() { return (size_t)2 * 2 * 64 * (DH / 8) * 16; }
template <int DH> constexpr size_t dq_lds() { return (size_t)2 * 2 * 64 * (DH / 8) * 16; }
template <int DH> constexpr size_t dkv_lds() { return (size_t)2 * 2 * 64 * (DH / 8) * 16 + 2 * 128 * 4; }

bool attn_ok(int B, int S, int H, int DH, int ld_qkv, int ld_o, int G) {
  return G >= 1 && G <= MAXG && B >= 1 && S >= 1 && H >= 1 && (DH == 64 || DH == 128) && ld_qkv >= 3 * H * DH &&
         !(ld_qkv & 7) && ld_o >= H * DH && !(ld_o & 7) &&
         (long)std::min(S, 64) * std::max(ld_qkv, ld_o) * 2 <= 0x7fffffffL;  // the rows of a tile: 31 bits from the first
}
// Loads into LDS move 16 bytes of one row: the matrices whose tiles they bring have to start on such a boundary (their rows then do).
bool tiles_ok(const bf16_t* const* m, int G) {
  uintptr_t bits = 0;
  for (int g = 0; g < G; ++g) bits |= (uintptr_t)m[g];
  return (bits & 15) == 0;
}

// o of some problem inside the buffer that dqkv is written to.  The dq kernel alone reads o, a row before it stores that row of dq;
// side by side the dk/dv workgroups would read o while dq is stored.
bool o_in_dqkv(const AttnBwdArgs& a) {
  const uintptr_t rows = (uintptr_t)a.B * a.S;
  for (int g = 0; g < a.G; ++g) {
    const uintptr_t o = (uintptr_t)a.o[g], q = (uintptr_t)a.dqkv[g];
    if (o < q + rows * a.ld_qkv * 2 && q < o + rows * a.ld_o * 2) return true;
  }
  return false;
}

// Work items of a launch: 128-row blocks of every (batch, head) of every problem
dim3 attn_grid(int B, int S, int H, int G, AttnGrid& gr) {
  auto rcp = [](unsigned d) { return d == 1 ? 0xffffffffu : (unsigned)((1ull << 32) / d); };
  gr.n_blk = ((unsigned)S + 127) / 128;
  gr.n_bh = (unsigned)B * H;
  gr.n_h = H;
  gr.total = gr.n_blk * gr.n_bh * G;
  gr.per_xcd = (gr.total + 7) / 8;
  gr.last = -1;
  gr.r_blk = rcp(gr.n_blk);
  gr.r_bh = rcp(gr.n_bh);
  gr.r_h = rcp(gr.n_h);
  return dim3(gr.per_xcd * 8);
}

// The same with two row blocks to a workgroup where that is ahead
dim3 attn_grid_causal(int B, int S, int H, int G, int causal, int per_cu, AttnGrid& gr) {
  const dim3 grid = attn_grid(B, S, H, G, gr);
  if (!causal || !attn_pairs(gr.n_blk, gr.total, per_cu)) return grid;
  const int last = (int)gr.n_blk - 1;
  const dim3 pairs = attn_grid(B, ((S + 127) / 128) / 2 * 128, H, G, gr);  // n_blk is even
  gr.last = last;
  return pairs;
}

// Rows past the sequence whose offsets would pass 32 bits (lane_row)
bool rows_far(int ld_qkv, int ld_o) { return 64L * std::max(ld_qkv, ld_o) * 2 > 0xffffffffL; }
template <int DH>
void launch_bwd_far(const AttnBwdArgs& a, const AttnGrid& gr, dim3 grid, hipStream_t s) {
  hipLaunchKernelGGL((attn_bwd_dq_kernel<DH, false, true>), grid, dim3(256), dq_lds<DH>(), s, a, gr);
  hipLaunchKernelGGL((attn_bwd_dkv_kernel<DH, true>), grid, dim3(256), dkv_lds<DH>(), s, a, gr);
}

}  // namespace

hipError_t attn_init() {  // the other kernels stay within the default LDS limit
  const void* const kernels[] = {reinterpret_cast<const void*>(&attn_bwd_dkv_kernel<128>), reinterpret_cast<const void*>(&attn_bwd_dkv_kernel<128, true>),
                                 reinterpret_cast<const void*>(&attn_bwd_both_kernel<128>)};
  for (const void* k : kernels) {
    const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dkv_lds<128>());
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_attn_fwd(const AttnArgs& a, hipStream_t s) {
  if (!attn_ok(a.B, a.S, a.H, a.DH, a.ld_qkv, a.ld_o, a.G) || !tiles_ok(a.qkv, a.G)) return hipErrorInvalidValue;
  AttnGrid gr;
  const dim3 grid = attn_grid_causal(a.B, a.S, a.H, a.G, a.causal, a.DH == 64 ? 4 : 2, gr);
  if (rows_far(a.ld_qkv, a.ld_o)) {
    if (a.DH == 64) hipLaunchKernelGGL((attn_fwd_kernel<64, true>), grid, dim3(256), fwd_lds<64>(), s, a, gr);
    else hipLaunchKernelGGL((attn_fwd_kernel<128, true>), grid, dim3(256), fwd_lds<128>(), s, a, gr);
    return hipGetLastError();
  }
  if (a.DH == 64) hipLaunchKernelGGL(attn_fwd_kernel<64>, grid, dim3(256), fwd_lds<64>(), s, a, gr);
  else hipLaunchKernelGGL(attn_fwd_kernel<128>, grid, dim3(256), fwd_lds<128>(), s, a, gr);
  return hipGetLastError();
}

hipError_t launch_attn_bwd(const AttnBwdArgs& a, hipStream_t s) {
  if (!attn_ok(a.B, a.S, a.H, a.DH, a.ld_qkv, a.ld_o, a.G) || !tiles_ok(a.qkv, a.G) || !tiles_ok(a.dout, a.G))
    return hipErrorInvalidValue;
  AttnGrid gr;
  const dim3 grid = attn_grid(a.B, a.S, a.H, a.G, gr);
  if (rows_far(a.ld_qkv, a.ld_o)) {
    if (a.DH == 64) launch_bwd_far<64>(a, gr, grid, s);
    else launch_bwd_far<128>(a, gr, grid, s);
    return hipGetLastError();
  }
  // The halves' workgroups fit the chip together: two per CU at DH = 64, one at DH = 128 (476 registers), where a second round of
  // the shorter dq workgroups still pays a little past that.  us, two launches | one: DH = 64, 256 row blocks 53.4 | 43.0;
  // DH = 128, 128 blocks 89.1 | 72.9, 160 56.5 | 46.2, 192 57.7 | 63.5 and 94.9 | 109 (causal 163 | 138), 256 98.9 | 114.
  if (grid.x <= (a.DH == 64 ? 256 : 160) && !o_in_dqkv(a)) {
    const dim3 both(2 * grid.x);
    if (a.DH == 64) hipLaunchKernelGGL(attn_bwd_both_kernel<64>, both, dim3(256), dkv_lds<64>(), s, a, gr);
    else hipLaunchKernelGGL(attn_bwd_both_kernel<128>, both, dim3(256), dkv_lds<128>(), s, a, gr);
    return hipGetLastError();
  }
  const dim3 wgs = attn_grid_causal(a.B, a.S, a.H, a.G, a.causal, a.DH == 64 ? 3 : 2, gr);
  if (a.DH == 64) {
    if (gr.last >= 0) hipLaunchKernelGGL((attn_bwd_dq_kernel<64, true>), wgs, dim3(256), dq_lds<64>(), s, a, gr);
    else hipLaunchKernelGGL((attn_bwd_dq_kernel<64, false>), wgs, dim3(256), dq_lds<64>(), s, a, gr);
    hipLaunchKernelGGL(attn_bwd_dkv_kernel<64>, wgs, dim3(256), dkv_lds<64>(), s, a, gr);
  } else {
    if (gr.last >= 0) hipLaunchKernelGGL((attn_bwd_dq_kernel<128, true>), wgs, dim3(256), dq_lds<128>(), s, a, gr);
    else hipLaunchKernelGGL((attn_bwd_dq_kernel<128, false>), wgs, dim3(256), dq_lds<128>(), s, a, gr);
    hipLaunchKernelGGL(attn_bwd_dkv_kernel<128>, wgs, dim3(256), dkv_lds<128>(), s, a, gr);
  }
  return hipGetLastError();
}

}  // namespace hydra
