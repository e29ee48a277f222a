// Line lengths the fast transforms (k_fft.h) are built for, as (N, R1, R2):
// N = R1 R2, R1 points of real data in stage A, R2 complex ones in stage B.
// Every multiple of 16 up to 512 without a prime factor above 13 (272, 304, 368,
// 464 and 496 have one and take the dense products: such a stage is summed
// directly), so that both stages stay within 32 real or 20 complex values per
// thread.  Stage A takes the larger factor: real data hold half as many
// registers per point.
#pragma once

#define IBS_FFT_SIZES_32(X)                                                                              \
    X(32, 8, 4) X(64, 8, 8) X(96, 12, 8) X(128, 16, 8) X(160, 16, 10) X(192, 16, 12) X(224, 16, 14)       \
    X(256, 16, 16) X(288, 24, 12) X(320, 20, 16) X(352, 22, 16) X(384, 24, 16) X(416, 26, 16)             \
    X(448, 28, 16) X(480, 30, 16) X(512, 32, 16)
#define IBS_FFT_SIZES_16(X)                                                                              \
    X(16, 4, 4) X(48, 8, 6) X(80, 10, 8) X(112, 14, 8) X(144, 16, 9) X(176, 16, 11) X(208, 16, 13)        \
    X(240, 16, 15) X(336, 24, 14) X(400, 20, 20) X(432, 24, 18)

// Those the fused x-z transforms (k_plane.h) are built for.
#define IBS_PLANE_SIZES(X) X(16, 4, 4) X(32, 8, 4) X(48, 8, 6) X(64, 8, 8)

// FP32 fields (refined path): lines of up to FFT_F64_ARITH_MAX points take FP64
// arithmetic, longer ones FP32; in forward transforms longer ones take FP64
// too where the solve amplifies what they leave on the lowest modes (a
// pressure solve; Helmholtz pencils of a condition bound beyond FP32's), and
// where both axes together have at most FFT_F64_FORWARD_SUM points.
// The three-term bfloat16 products these transforms replace carried a line's
// result to within a few roundings whatever its length.  FP32 butterflies
// forward spread eps of the whole line over every mode, and the pressure
// solve multiplies what falls on the lowest by 1 / lambda: refined Poisson
// solves ended up to 2.7 times further from the FP64 solution than with the
// products (416x32x64), with walls in x up to 6 times (512x32x64); with FP64
// they end as near or up to 20 times nearer.  A Helmholtz solve multiplies by
// 1 / (1 + c lambda), at most 1, but at c lambda beyond FP32's bound all that is
// left of its solution are those modes: up to 4.3 times further (512x48x64,
// walls in x, c = 1) in FP32, in FP64 at 0.03 to 0.4 of the products' error.
// At small c longer lines end 1.05 to 6 times nearer in FP32 already, short ones
// further (96^3 1.45 times, 128^3 1.37, 192x160x96 1.06; in FP64 0.75, 0.77,
// 0.5), hence FFT_F64_FORWARD_SUM.  Inverse transforms do not amplify.
// Cost: up to 64 points nothing (the pass is bound by memory), a 256^3 pressure
// z transform 28 us instead of 24 and x 26 instead of 22, three Helmholtz
// solves 104 -> 107 us at 96^3, 151 -> 158 at 128^3.
namespace ibs {
constexpr int FFT_F64_ARITH_MAX = 64;
constexpr int FFT_F64_FORWARD_SUM = 288;
constexpr int PLANE_MAX = 64;   // longest line of the fused x-z transforms
}
