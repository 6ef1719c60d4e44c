// What the direct-to-LDS ring's loads of an operand with k as the slow index add to the start of their descriptor, which ends with the
// operand's k-rows: loads past it bring zeros and fetch nothing.  Nothing here calls HIP.
#pragma once

namespace hydra {

// An offset past every descriptor (operands span less than 2 GiB: dma_eligible)
constexpr unsigned RING_PAST = 0x7fffffffu;

// The part of sub-tile t (bk k-rows of row_bytes): the same for the whole wave, so that the end of the sum, or of the range of it that a
// workgroup takes, costs the scalar unit a comparison and the vector unit nothing.  With the
// descriptor's end alone, which is the operand's, every range of a split sum but the last fetches up to three sub-tiles of the next one, which
// nobody uses.  us, that | now: 4 x [1024 x 1024] over 16384 rows with Adam (8 ranges) 183.5 | 181.7, 2 x [1000 x 1000] over 8200 69.3 | 68.3,
// 2 x [2048 x 1024] over 4096 (4 ranges) 72.5 | 71.5, 4 x [768 x 3072] over 2048 (2) 112 | 112.
constexpr unsigned ring_sub_tile(int t, int bk, int k_end, unsigned row_bytes) {
  return t * bk < k_end ? (unsigned)(t * bk) * row_bytes : RING_PAST;
}

}  // namespace hydra
