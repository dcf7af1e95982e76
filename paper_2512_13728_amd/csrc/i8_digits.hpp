// The fixed-point arithmetic of the digit products (k_gemm_i8.hip), in plain
// C++ so that the CPU tests compile the very code that the kernels run.
//
// x = v 2^(e-46) with |x| < 2^e and v an integer in I8_NS signed base-256
// digits, v = sum_a s_a 256^(5-a).  Digit products s_a t_b of one weight,
// a + b = T, add up exactly in int32: at most six of at most 2^14 each over at
// most I8_KMAX rows.  A digit product of weight T is at most 2^(14 + 8 (10 - T)),
// against 2^92 for the whole product: 2^-38 at T = 5, 2^-46 at T = 6, 2^-54 at
// T = 7.
#pragma once

namespace cd {

constexpr int I8_NS = 6;           // digits per operand
constexpr int I8_KMAX = 16384;     // rows of one exact int32 sum: 6 * 2^14 * 2^14 < 2^31
// The largest weight kept.  Products of two different operands drop T > 5: 21
// digit products; what is dropped has either sign and averages over K (about
// 2^-46.4 sqrt(K) of the largest product).  A Gram matrix also keeps T = 6, 26
// in all: on its diagonal that weight holds the square s_3^2, which never
// averages: without it W_ii is low by K 2^-47.6 of the column's largest square,
// and where one row dominates the columns that passes the pivot floor of 1e-13
// (2048 x 512, r = 256, a row 1e5 above the others, kappa(P~) 3.3e6: 16 pivots
// floored where none is weak).  What T = 7 drops has either sign and T = 8's
// squares are 2^-63.6 a row.
constexpr int I8_TOP = 5;
constexpr int I8_TOP_GRAM = 6;

// x 2^(46-e) is rounded to an integer v by adding 1.5 2^52; the added
// 0x808080808080 turns the digits of v into the bytes of the sum, each 128
// more than the digit (|v| <= 2^46, so the sum stays inside its 48 bits):
// fma(x, 2^(46-e), I8_BIAS)'s byte 5 - a, exclusive-or 0x80, is digit a.
constexpr double I8_BIAS = 6755399441055744.0 + 141289400074368.0;

}  // namespace cd
