// Which of its kernels a product of fp32 operands takes (gemm_f32.hip): arithmetic on the sizes, no device code.
#pragma once
#include <cstdint>

namespace tmk {

struct F32Form {
  int tile;      // edge of a block's tile: 128, 64, 32 or 16
  int split;     // waves of a tile that split every stage's reduction elements
  bool patches;  // an XCD walks its tiles in patches
};

// C[M,N] over K; wgrad: both operands strided along K, result fp32 in place.  reach16: the 16x16 form's offsets fit 32 bits.
//
// A block's time is its share of the MFMA rate, tile^2 per step, and a unit works through ceil(blocks / 256) of them; the
// smaller tiles read LDS and synchronise more per MFMA (factors).  The lines below are drawn from every form's time, in plain
// order and in patches, on 1800 products of each kind with 16 to 8192 rows, columns and reduction elements.  On 6700 others
// the pick is 0.4 % (weight gradients 0.9 %) slower than the fastest form, 5 to 16 % faster than the best of 128x128, 64x64 and
// four-way 32x32 tiles by area alone, and on none of them more than 4 % slower.
//  * 16x16 tiles for up to two a unit: 232 x 256 over 512 3.4 us, 5.1 on 32x32; 135 x 768 over 512, two a unit, 4.3 and 5.2;
//    350 x 512 over 512, three, 5.9 and 5.3.  Weight gradients, which fetch 64-byte pieces of both operands, for one a unit:
//    256 x 256 over 319 3.2 and 4.0; 152 x 664 over 226, two a unit, 4.4 and 4.1; 296 x 960 over 91, five, 7.2 and 4.2.
//  * Four waves that split a 64x64 tile's reduction have to meet at the end: from 512 elements on and for at most one block a
//    unit (1024 x 1024 over 1024 23.7 -> 21.9 us, over 4096 86 -> 77).  With several, which cover each other's waits, 3072 x
//    1024 over 1024 56 -> 61, and two waves in place of one 56 -> 57.
//  * Eight waves instead of four on a 32x32 tile for weight gradients of 256 elements and more (2 to 9 % faster; other
//    products -2 to 4 % slower, shorter weight gradients up to 4 %).
//  * Patches for small tiles whose operands exceed an XCD's L2 (4 MiB), several of which would otherwise fetch all of them:
//    16x16 (64 x 2048 over 2048 with strided weights, pieces of 64 bytes, 23.8 -> 10.8 us; 78 x 1536 over 896 9.4 -> 6.8)
//    and, from 6 MiB on, 32x32 (1 to 5 % faster).  Below, patches are 1 to 3 % slower; larger tiles gain nothing (within 0.5 %).
inline F32Form f32_form(int64_t M, int64_t N, int64_t K, bool wgrad, bool reach16) {
  constexpr int64_t units = 256;
  auto tiles = [&](int64_t b) { return ((M + b - 1) / b) * ((N + b - 1) / b); };
  auto cost = [&](int64_t b, double factor) { return (double)((tiles(b) + units - 1) / units) * (double)(b * b) * factor; };
  auto patches = [&](int64_t b, int64_t mib) { return tiles(b) > units && K * (M + N) * 4 > mib << 20; };
  if (reach16 && tiles(16) <= (wgrad ? 1 : 2) * units) return {16, 4, patches(16, 4)};
  const double c128 = cost(128, 1.0), c64 = cost(64, 1.1), c32 = cost(32, K >= 512 ? 1.4 : 1.5);
  if (c128 <= c64 && c128 <= c32) return {128, 1, false};
  if (c64 <= c32) return {64, tiles(64) <= units && K >= 512 ? 4 : 1, false};
  if (wgrad && K < 256) return {32, 4, false};
  return {32, wgrad ? 8 : 4, patches(32, 6)};
}

}  // namespace tmk
