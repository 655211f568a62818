// Which of its kernels a product of fp32 operands takes (gemm_f32.hip, gemm_f32_split.hip): arithmetic on the sizes, no device
// code.
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

// Whether the kernel on bf16 terms (gemm_f32_split.hip, 128x128 tiles) is the faster one.
//
// Times in us from the passes over the chip (r; one block a unit on bf16 terms), the tiles a unit has on average (u) and the
// reduction length, fitted by non-negative least squares to every form's time on 300 to 600 products of each kind with 96 to 8192
// rows and columns over 256 to 8192 elements; they meet them to 3 to 6 %.  It has to win by 5 %.  Single products from a warm
// cache then take 0.84 of their time (247 of 900, at most 1.00; 128x128 tiles 0.79, 64x64 ones that a unit has several of 0.86).
//
// In whole passes less is left, for the card's matrix rate on random data falls under a lasting load; and short reductions over
// more than one round of blocks, whose results leave a unit with nothing beside them and meet a cold cache, lose: 2026 x 5888 over
// 384 in a step of 676 us 0.968 of the speed, 1594 x 5504 over 768 in one of 885 us 0.967.  Without those, 90 layers and linear
// maps that use it are 2.5 % faster (geometric mean; 0.98 to 1.24), a layer of hidden 1024 on 1024 tokens 3 to 8 %.
//
// Never at the price of precision: its error on N(0,1) data, 1.9e-7 of the result over 1024 elements, is below that of the whole
// walks (5.7e-7) and the four-way ones (2.9e-7) that it replaces; weight gradients that eight waves split (2.0e-7) stay.
inline bool f32_split(int64_t M, int64_t N, int64_t K, bool wgrad, bool reach16) {
  const F32Form f = f32_form(M, N, K, wgrad, reach16);
  if (K < 256 || f.tile == 16 || f.split != (f.tile == 32 ? 4 : 1)) return false;
  if (K < 1024 && ((M + 127) / 128) * ((N + 127) / 128) > 256) return false;
  struct Grid {
    double r, u;
  };
  auto grid = [&](int64_t b) {
    const int64_t n = ((M + b - 1) / b) * ((N + b - 1) / b);
    return Grid{(double)((n + 255) / 256), (double)n / 256};
  };
  const double k = (double)K / 1024;
  const Grid g = grid(f.tile), t = grid(128);
  const double now = f.tile == 128  ? 4.0 + g.r * (3.0 + 61 * k)
                     : f.tile == 64 ? 2.9 + g.r * (0.4 + 16.8 * k) + g.u * 0.5
                                    : 2.7 + g.r * (0.3 + 5.1 * k) + g.u * 0.4;
  return 1.05 * (1.0 + t.r * (6.0 + 33.9 * k) + t.u * (1.2 + 11.9 * k)) < now;
}

}  // namespace tmk
