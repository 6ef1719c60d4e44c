// What the direct-to-LDS ring's loads of an operand with k as the slow index add to the start of their descriptor, which ends with the last
// of the operand's K k-rows: loads past it bring zeros and fetch nothing.  An offset is the sum of a part that the wave shares and a lane's own, each
// at most K rows, so that with K rows below 2 GiB the sum stays below 4 GiB.  Nothing here calls HIP.
#pragma once

namespace hydra {

// The operands that the ring takes: a page short of 2 GiB, which the bytes inside a k-row (less than 2 KB) may fill
constexpr bool ring_spans(long K, long ld, long sz) { return K * ld * sz < 0x7ffff000L; }

// Bytes of an operand with k as the slow index, from its first element to the end of the 16-byte chunk that holds the last element of its n columns
// in its last k-row: behind that the operand's buffer may end (columns of a wider matrix, where a tile's columns past n would be read
// behind the whole matrix).
constexpr long k_slow_bytes(long K, long ld, long n, long sz) { return ((K - 1) * ld + (n * sz + 15) / 16 * 16 / sz) * sz; }

// The shared part, of sub-tile t (bk k-rows of row_bytes).  k_end: where the sum, or the range of it that a workgroup takes, ends; sub-tiles from
// there on begin past the operand.  Most kernels' k_end is K, and this is one minimum of the scalar unit; a comparison and a selection per
// operand took 0.1 to 0.25 us in weight gradients of few tiles (4 x [256 x 1024] over 1024 rows 12.3 | 12.5).
// With the descriptor's end alone every range of a split sum but the last fetches up to three sub-tiles of the next one, which nobody
// uses.  us, that | now: 4 x [1024 x 1024] over 8192 rows with Adam (8 ranges) 114.2 | 112.5, over 16384 180 | 178, 2 x [1000 x 1000] over 8200
// 69.0 | 67.9, 2 x [2048 x 1024] over 4096 (4 ranges) 71.7 | 70.5, 4 x [768 x 3072] over 2048 (2) 109.1 | 107.9.
constexpr unsigned ring_sub_tile(int t, int bk, int k_end, int K, unsigned row_bytes) {
  return (unsigned)(t * bk < k_end ? t * bk : K) * row_bytes;
}

// A lane's part: k-row k of a sub-tile, `col` bytes into it.  k-rows past K count as K.  (Counted on, those of the last sub-tile come round to rows
// that are there where rows lie 2^32 / 32 to 2^32 / 128 bytes apart or more.)
constexpr unsigned ring_lane(int k, int K, unsigned row_bytes, unsigned col) { return (unsigned)(k < K ? k : K) * row_bytes + col; }

}  // namespace hydra
