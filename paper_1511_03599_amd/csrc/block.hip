// Blocked FIR + FFT: which shapes take it, and the launcher for each input
// type (the kernel is in block_launch.h).
#include "launch.h"

namespace pfb {

// Up to 128 channels every window, 256 to 1024 channels the windows beyond
// the register-window kernel, above that windows of up to 32 taps (16 at
// 8192 channels). Longer ones gain little or lose: 2^26 samples, split ->
// blocked, complex64: 2048 channels, 64 taps 0.51 -> 0.41 ms, 4096 channels,
// 64 taps 0.52 -> 0.54, 8192 channels, 32 taps 0.44 -> 0.56 (most of a
// block's raw rows are then history); their unrolled kernels also take the
// longest to compile.
bool block_supported(int dtype, int tp, int log2c, bool pol)
{
    if (dtype < 0 || dtype > 3 || tp < 4)
        return false;
    if (pol)
        return log2c >= 9 && log2c <= 12 && tp <= 32;
    if (log2c < 5 || log2c > 13)
        return false;
    if (log2c <= 7)
        return tp <= 64;
    if (log2c <= 10)
        return tp == 32 || tp == 64;
    return tp <= (log2c == 13 ? 16 : 32);
}

// Filtered spectra per block (BlockShape::R2).
int block_rows(int log2c, bool pol)
{
    return (16384 >> log2c) * (log2c >= 10 ? 2 : 1) / (pol ? 2 : 1);
}

// Whether the blocked kernel is the faster one for `units` streams (or
// sub-bands) of S spectra. A block takes one CU 9 us (128 channels) to 40 us
// (4096 channels, 32 taps), and a launch of few blocks leaves the other CUs
// idle, where the FIR and FFT launches spread over more of them. Split over
// blocked time, on 256 CUs, at 64 and 128 blocks and where noted 32 or 256;
// a line between two measured counts is where the time interpolates to equal,
// and it is in blocks per CU (a partition of the card has fewer):
//   2048 channels, 16 taps        complex64 0.90, 1.25; int8 0.95, 1.46
//   4096 channels, 8 taps         0.97, 1.23
//   1024 channels, 32 taps        0.83, 1.35
//   1024 channels, 64 taps        complex64 1.00, 1.17; int8 0.99, 0.93 (256: 1.44)
//   4096 channels, 32 taps        128: 0.80; 256: 1.35
//   2048 channels, 32 taps        128: 1.03
//   8192 channels, 16 taps        0.84 and 1.38
//   512 channels, 32 taps         64: 1.04
//   256 channels, 64 taps         0.90, 1.17; 40 taps int8 0.72, 0.88 (256: 1.40)
//   sub-bands of 4096 channels    32: 0.84; 128: 1.52
// Otherwise up to 512 channels one launch is the faster from one block on
// (256 channels, 32 taps, 16 blocks 15.2 -> 13.7 us, 128 channels, 8 taps, 4
// blocks 11.8 -> 9.4), but for part of a block at 17 to 32 taps, which still
// takes the time of a whole one. Split and blocked, in us: 128 channels
// complex64 1 spectrum 8.5, 13.9, 20 spectra 12.8, 14.0, 64 spectra 13.0,
// 14.0; int8 5 spectra 10.7, 14.2, 20 spectra 15.7, 14.2 (its FIR tests the
// rows of a ragged tile); 256 channels 5 spectra 9.5, 12.9, 16 spectra 13.3,
// 12.9; 32 channels 32 spectra 15.7, 12.2. (With FIR tiles of 128 rows the
// split path took 12.2 at 1 spectrum and 13.0 at 20, complex64.)
bool block_pays(int dtype, int tp, int log2c, bool pol, int64_t units, int64_t S, int cus)
{
    if (!block_supported(dtype, tp, log2c, pol))
        return false;
    const bool ints = dtype == 1 || dtype == 2;
    if (!pol && tp == 32 && log2c >= 6 && log2c <= 8 && units * S < (log2c == 7 && !ints ? 48 : 16))
        return false;
    const int64_t rows = block_rows(log2c, pol);
    const int64_t blocks = units * ((S + rows - 1) / rows);
    int from = 1;
    if (pol)
        from = log2c <= 9 ? 1 : tp >= 32 ? 112 : 72;
    else if (tp == 64)
        from = log2c >= 10 && dtype != 0 ? 192 : 128;
    else if (log2c == 9)
        from = tp == 32 ? 60 : 1;
    else if (log2c >= 10)
        from = log2c >= 11 && (tp >= 32 || (log2c == 13 && tp == 16)) ? 160 : 84;
    return 256 * blocks >= (int64_t)from * cus;
}

hipError_t launch_block(const BlockArgs &a, int dtype, int tp, int log2c, bool pol, hipStream_t st)
{
    if (!block_supported(dtype, tp, log2c, pol))
        return hipErrorInvalidValue;
#define PFB_BLOCK_DT(DT, NAME)                                                                               \
    case DT:                                                                                                 \
        return pol           ? launch_block_##NAME##_pol(a, tp, log2c, st)                                   \
               : log2c >= 11 ? launch_block_##NAME##_large(a, tp, log2c, st)                                 \
                             : launch_block_##NAME##_small(a, tp, log2c, st);
    switch (dtype) {
        PFB_BLOCK_DT(0, c64)
        PFB_BLOCK_DT(1, ci16)
        PFB_BLOCK_DT(2, ci8)
        PFB_BLOCK_DT(3, cf16)
    default:
        return hipErrorInvalidValue;
    }
#undef PFB_BLOCK_DT
}

} // namespace pfb
