// lf2_lengths.hpp -- line lengths with compiled kernels.
// LF2_LENGTHS: 2^a, 3 * 2^a and 5 * 2^a, with every tile variant.
// LF2_RAGGED_LENGTHS: the other 2^a 3^b 5^c up to 1024 points.  An axis of
// such a length takes a radix schedule at run time when one is set; until
// then it runs the compiled narrow tiles of these lengths, whose divisions,
// twiddle strides and unrolled stages are constants and whose first and last
// stages load and store memory from registers.  A 360 x 300 x 216 Poisson
// solve: 671 us with run-time schedules, 238 us compiled; the r2c pair of a
// 240 x 180 x 150 x 3 field with halo 1: 580 and 219 us; cubes of 30 to 480
// points 1.5 to 3.4 times faster, none slower.  Two lists of about equal
// compile time.
#pragma once
#define LF2_LENGTHS(X)                                                                       \
    X(1) X(2) X(3) X(4) X(5) X(6) X(8) X(10) X(12) X(16) X(20) X(24) X(32) X(40) X(48)      \
    X(64) X(80) X(96) X(128) X(160) X(192) X(256) X(320) X(384) X(512) X(640) X(768) X(1024)
// Strided (y / z) passes also take 2048-point lines (2048^3 lattices).
#define LF2_S_LENGTHS(X) LF2_LENGTHS(X) X(2048)
#define LF2_RAGGED_LENGTHS_A(X) X(9) X(15) X(18) X(25) X(27) X(30) X(36) X(45) X(50)        \
    X(54) X(60) X(72) X(75) X(81) X(90) X(100) X(108) X(120) X(125) X(135) X(144) X(150)    \
    X(162) X(180) X(200) X(216) X(225) X(240) X(243) X(250) X(270)
#define LF2_RAGGED_LENGTHS_B(X) X(288) X(300) X(324) X(360) X(375) X(400) X(405) X(432)     \
    X(450) X(480) X(486) X(500) X(540) X(576) X(600) X(625) X(648) X(675) X(720) X(729)     \
    X(750) X(800) X(810) X(864) X(900) X(960) X(972) X(1000)
#define LF2_RAGGED_LENGTHS(X) LF2_RAGGED_LENGTHS_A(X) LF2_RAGGED_LENGTHS_B(X)
