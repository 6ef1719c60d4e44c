// Which of two forms of a launch is ahead, by counts alone: the forms give the same bits, so a choice changes nothing but the time.  Nothing
// here calls HIP.
#pragma once

namespace hydra {

// ---- bf16 products: 256x256 tiles or 128x128 ones -------------------------------------------------------------------------------
// A launch of `big` 256x256 tiles runs in passes of one tile per CU (256), the same launch as `mid` 128x128 tiles with two workgroups per CU.
inline long tile_passes(long big) { return (big + 255) / 256; }
// percent of the passes of 256x256 tiles that hold a tile
inline long pass_fill(long big) { return big * 100 / (tile_passes(big) * 256); }
// How many 128x128 tiles the fullest CU has beyond three to a pass.  A pass of 256x256 tiles takes as long as three or four of them: three are
// ahead, a fourth is behind unless the epilogue is long against the sum.
inline long rounds_over(long big, long mid) { return (mid + 255) / 256 - 3 * tile_passes(big); }

// Products of two passes or more whose passes are a sixth (K <= 768) or a quarter empty.  wide: the epilogue reads a gate or stores the
// pre-activation beside the output.  us, 256x256 | 128x128, K = 768 and 3072:
//   three to a pass   288 tiles GeLU 61 | 46 and 153 | 133, 320 gate 61 | 50 and 161 | 139, 384 plain 50 | 45 and 147 | 143, 576 73 | 68 and 222 | 217
//   one more, 2 passes   390 GeLU 60 | 60 and 153 | 174, gate 63 | 64 and 160 | 178, bias 49 | 51 and 143 | 165, plain 47 | 50 and 143 | 166; 400,
//     K = 512 GeLU 49 | 47, gate 53 | 52, bias 37 | 39, plain 37 | 40
//   one more, 3 and 4 passes   640 GeLU 94 | 86 and 243 | 241, plain 75 | 74 and 227 | 236; 832 GeLU 124 | 110, plain 98 | 96
//   two more, 4 passes   860 GeLU 122 | 114, gate 128 | 125, plain 97 | 102
// One pass that is not full stays with 256x256 tiles (192 tiles: 30 | 31 and 76 | 84), and so do operands that the direct-to-LDS kernels
// do not reach (!direct): of the register-staged ones the smaller tile is behind (288 tiles plain, K = 131136, 7250 | 8371).
inline bool mid_tiles_for_product(long big, long mid, int K, bool wide, bool direct) {
  const long passes = tile_passes(big), over = rounds_over(big, mid);
  if (!direct || passes < 2 || pass_fill(big) > (K <= 768 ? 84 : 76)) return false;
  if (over <= 0) return true;
  if (wide) return K <= (passes >= 3 ? 768 : 512);
  return passes >= 3 && over == 1 && K <= 768;
}

// Updates over K >= 2048, whose thin passes cost the state's part of the epilogue, too.  us, 256x256 | 128x128, Adam, K = 2048, 8192, 16384:
//   one pass, three to it   144 tiles 105 | 95, 255 | 231, 442 | 490; 192 125 | 108, 284 | 253 (rows 8 KB apart 115 | 112, 278 | 259; SGD 80 | 72,
//     241 | 224); 12 x [1024 x 1024] 126 | 104, 291 | 266, at K = 12288 401 | 396 and SGD 360 | 365
//   one pass, a fourth   195 120 | 120, 277 | 295; 198 117 | 119, 273 | 291; SGD 195 82 | 84, 237 | 262
//   more passes, three to each   288 215 | 170, 526 | 394, 916 | 750; 384 238 | 204, 561 | 497, 977 | 917; 576 364 | 283, 827 | 742, 1465 | 1447
//   more passes, a fourth to each   390 242 | 206, 563 | 537, 968 | 1014; 585 367 | 294, 839 | 783, 1462 | 1486; SGD 390 160 | 144, 475 | 474, 898 | 943
// In full passes the 128x128 tile gains 2 to 6 % on one update repeated (256 tiles, Adam, K = 2048 to 4096) and nothing, or 1 % less, behind the
// input gradient that it follows in a layer's backward pass; SGD's is 2 to 11 % slower.
inline bool mid_tiles_for_long_update(long big, long mid, int K) {
  if (pass_fill(big) > 76) return false;
  if (rounds_over(big, mid) <= 0) return tile_passes(big) > 1 || K <= 8192;
  return tile_passes(big) > 1 && K <= 8192;
}

// ---- fp32 weight gradients with an update over fewer than 64 rows: 32x32 tiles in one stage or 32x128 ones -------------------------------
// Rows of the state that are no whole number of 128-byte lines: neighbours along a row share the lines at their seam, through one L2 only if they run
// on one XCD, ids a multiple of 8 apart.  32x32 tiles are numbered down the columns, so their grid is made that high (workgroups past the
// matrix end at once), if these are half as many as the others at most, for SGD, which moves a third of Adam's bytes, fewer than a third
// (2 x [547 x 2128] of 18 tile rows 9.5 | 9.9 and 16.4 | 15.2, 10 x [320 x 496] of 10 Adam 13.1 | 13.8).  us, SGD and Adam, as it is | so: 1 x [1742 x 792], K = 32 8.3 | 5.9 and 13.7 | 9.6; 2 x [1616 x 712], 32
// 11.1 | 8.6 and 19.5 | 13.2; 3 x [800 x 1000], 16 11.2 | 9.1 and 19.8 | 14.3; of 3 and 4 tile rows 12.2 | 22.1 and 9.8 | 11.1.  Whole lines gain nothing and
// pay for the empty workgroups (4 x [784 x 768], 8 8.8 | 9.5 and 14.1 | 15.8).
inline long f32_update_tile_rows(long rows, int ldo, bool adam) {
  const long high = (rows + 7) / 8 * 8;
  return ldo % 32 && rows > 8 && (adam ? 2 * high <= 3 * rows : 3 * high < 4 * rows) ? high : rows;
}
// tiles: of 32x32; rows: tile rows of a problem; wide: tiles of 32x128.  Up to 1600 small tiles
// hide the state's way behind one another; Adam's three matrices and sums over more than 32 rows keep them ahead beyond.  SGD over few rows is ahead
// with 32x128 tiles, unless two in seven of their columns lie past the matrix or the seams above are taken care of.  us, 32x128 | 32x32, four sets of
// buffers in turn:  1 x [2300 x 480] over 25 rows, SGD 6.6 | 5.3;  9 x [1229 x 352] over 41, SGD 16.1 | 12.7;  9 x [830 x 544] over 42, Adam 28.5 | 22.5;
//   SGD, 10 x [522 x 376] over 30 rows 8.5 | 10.8, 14 x [203 x 736] over 28 8.3 | 9.4, 12 x [2073 x 160] over 20 15.1 | 12.2;  of 72 tile rows with seams
//   5 x [2283 x 168] over 31 9.3 | 8.0.  640 random shapes over 1 to 63 rows, this rule against 32x128 tiles throughout: 1.11 (SGD) and 1.18 (Adam) times as
//   fast, 0.87 at worst (few tile rows with seams, 16 x [75 x 1032] over 12 7.4 | 8.5).
inline bool f32_update_few(long tiles, long rows, long wide, int ldo, int K, bool adam) {
  if (tiles <= 1600 || tiles > 4096) return tiles <= 1600;
  if (adam || K > 32) return true;
  return (ldo % 32 && f32_update_tile_rows(rows, ldo, adam) % 8 == 0) || 20 * wide >= 7 * tiles;
}

// ---- launches that two products share ---------------------------------------------------------------------------------------------
// A weight gradient with its update, n_w tiles of 64x64 over k_w rows, and an input gradient, n_d such tiles over k_d, as one launch of them.
// 512 tiles run at a time.  d_small: the input gradient takes 64x64 tiles alone, too; then the launch is never slower (2531 measured pairs of up
// to 1280 tiles, 0.976 of the two launches at worst).  Otherwise its 64x64 tiles cost more than the 128x128 ones that it gives up: little
// over a short sum, and nothing where all tiles run at once or the update takes the longer.  Together against apart, n pairs, mean and worst, and
// examples in us, apart | together (n_d + n_w, k_d and k_w):
//   k_d <= 384: 1013, 0.74, 1.07 (eight slower, the next worst 1.04)   1024 + 192, 256 and 1024 25 | 20;  756 + 144, 384 and 1328 18.5 | 19.8
//   all tiles at once: 279, 0.68, 0.87
//   n_d <= 512, k_w >= 1.5 k_d: 173, 0.77, 1.02   512 + 256, 1024 and 2048 30 | 26
//   k_d <= 512, a last pass of 160 tiles or more: 78, 0.82, 1.00   512 + 384, 512 and 1024 23 | 17;  696 + 144, 472 and 1841 27.7 | 26.6
//   the rest: 268, 0.94, 1.29 (76 slower)   675 + 450, 952 and 572 30 | 38;  576 + 512, 1024 and 1100 34 | 40;  576 + 128, 768 and 1100 19 | 21
// More than 1280 tiles: 1536 46 | 44 to 47 | 49, 2240 30 | 31, 2560 79 | 89, 6576 91 | 106.  k_d > 1024: together is ahead up to some 1000 tiles (768 44 |
// 34) and behind from there (1536 60 | 65, 2560 93 | 123); not taken.
inline bool pair_ahead(long n_d, long n_w, bool d_small, int k_d, int k_w) {
  const long all = n_d + n_w, last = (all - 1) % 512 + 1;
  if (all > 1280 || k_d > 1024) return false;
  if (d_small || k_d <= 384 || all <= 512) return true;
  return (k_d <= 512 && last >= 160) || (n_d <= 512 && 2L * k_w >= 3L * k_d);
}

// ---- LayerNorm backward of bf16 rows wider than 512: four workgroups to a CU or three ------------------------------------------------
// Four take the blocks in one pass where three would begin a second one.  us, three | four: 768 blocks 69.6 | 70.0, 826 64.8 | 58.2, 924 95.2 |
// 87.4, 959 119 | 110, 1024 95.7 | 91.1;  beyond that the passes run into one another and four are behind: 1115 82.2 | 84.1, 1444 138 | 141, 1965
// 205 | 208, 2340 level.
inline bool ln_four_to_a_cu(long blocks) { return blocks > 768 && blocks <= 1024; }

// fp32 rows of 1024 to 2048 elements, 32 to a workgroup: the next row asked for ahead (ln_bwd_wide_kernel), or not (ln_bwd_wide_f32_kernel).  Up to
// two workgroups to a CU are ahead with it.  From there to two and a half, where few CUs hold a third one, those few are waited for (two
// that ask ahead fill a CU's share of the memory, it seems: 512 to 514 blocks 110 -> 134 us at d = 2048); without it a workgroup goes at the pace of its own
// waits, whatever stands beside it.  us, not | ahead, backward pass of two problems, 512, 514, 564, 596, 626 and 656 blocks:
//   d = 2048  119 | 110, 122 | 134, 133 | 141, 134 | 141, 139 | 147, 146 | 147;  712 158 | 153
//        1792  106 | 100, 109 | 118, 119 | 124, 121 | 125, 124 | 127, 132 | 131
//        1536  92 | 86, 98 | 103, 105 | 108, 107 | 109, level, 114 | 112, and with the forward pass 564 151 | 147: the line lies here
//        1288  14, 2, 4, 5, 6 and 7 % behind without;  1032  20 to 30 % behind
inline bool ln_wide_ahead(long blocks, int d) { return d <= 1536 || blocks <= 512 || blocks > 640; }

// ---- attention under a causal mask: two row blocks of a head to a workgroup, or one --------------------------------------------------
// `blocks` 128-row blocks in all, n_blk to a head; per_cu: workgroups that fit a CU.  One to a workgroup suffers most where the blocks of a
// CU, 32 apart in an XCD's run, are blocks of the same number: n_blk a multiple of 8; then pairs are ahead as soon as there is more than one
// block to a CU.  Otherwise they are from the point where single blocks need a second pass.  An odd block left over spoils the balance.
// us, one | two, forward and backward, n_blk and blocks:
//   8 and 16   dh 64: 768 34.8 | 31.9, 90 | 85; 1024 42.7 | 33.4, 113 | 94; 2048 70 | 59, 198 | 178;  dh 128: 320 35 | 31, 101 | 95; 512 38 | 32, 113 | 104;
//     16 blocks, dh 64: 288 42 | 35, 110 | 97; 1024 78 | 56, 191 | 158; dh 128: 256 47.2 | 51.7, 142 | 158; 512 65 | 53, 187 | 163
//   4   dh 64: 640 20.1 | 19.6, 54.8 | 56.3; 1280 31.4 | 28.9, 88 | 84; 4096 82 | 70, 261 | 237;  dh 128: 320 22.1 | 20.6, 63.7 | 64.8; 640 33 | 30, 106 | 95
//   6   dh 64: 288 16.2 | 17.7, 42 | 47; 768 22.0 | 24.9, 62 | 68; 3072 70 | 65, 203 | 194;  dh 128: 384 25.1 | 26.4, 72 | 76; 1536 66 | 61, 205 | 200
//   2   dh 128: 2048 52.3 | 53.8, 199 | 206
//   3, 5, 7, 9, 11   dh 64: 3072 48 | 53, 154 | 188; 5120 105 | 104, 330 | 338; 7168 186 | 192, 552 | 586; 6912 211 | 208, 628 | 634; 4224 156 | 154, 454 | 459
inline bool attn_pairs(unsigned n_blk, unsigned blocks, int per_cu) {
  return n_blk >= 4 && n_blk % 2 == 0 && blocks > 256u * (n_blk % 8 == 0 ? 1 : per_cu);
}

}  // namespace hydra
