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
// idle, where the FIR and FFT launches spread over more of them; likewise the
// launch whose second round of blocks is nearly empty. Split over blocked
// time on 256 CUs, in blocks (the lines scale with the CUs, for partitions of
// the card); ints are int8 and int16:
//   2048, 16 taps        64: 0.86-0.96; 84: 0.99-1.05; 128: over 1.2
//   2048, 32 taps        100: 0.90-1.03; 128: 0.97-1.05; 280: 1.02-1.05,
//                        float16 0.95
//   4096, 8 taps         64: 0.96-1.02; 84: 1.04-1.2
//   4096, 16 taps        84: 0.98-1.03, complex64 0.86; 100: 1.02-1.1
//   4096, 32 taps        128: 0.78-0.99; 165: over 1.1; 280: 0.82-0.94; 350:
//                        complex64 0.95, others 1.1
//   8192, 8 taps         84: over 1.06, complex64 0.94; 100: complex64 1.00
//   8192, 16 taps        128: 0.86-0.99; 165: over 1.1; 257: ints 0.95; 280:
//                        1.00-1.03, complex64 0.92; 320: complex64 0.94
//   1024, 32 taps        84: 0.97-1.06, float16 0.90; 128: float16 1.01
//   512, 32 taps         64: 1.01-1.05, float16 0.96
//   64 to 1024, 33 to 64 92: complex64 0.86-1.03; 128: 0.96-1.2, others 0.81-0.98;
//                        150: 0.96-1.2; 280: complex64 over 1.04, ints 0.84-1.0;
//                        float16 0.79-0.95, 350: 0.93-1.04
//   sub-bands of 4096    32: 0.84; 128: 1.52
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
    const bool c64 = dtype == 0, ints = dtype == 1 || dtype == 2, cf16 = dtype == 3;
    if (!pol && tp == 32 && log2c >= 6 && log2c <= 8 && units * S < (log2c == 7 && !ints ? 48 : 16))
        return false;
    const int64_t rows = block_rows(log2c, pol);
    const int64_t blocks = units * ((S + rows - 1) / rows);
    int from = 1, again = 0; // again: the end of the nearly empty second round, 0 if it pays too
    if (pol) {
        from = log2c <= 9 ? 1 : tp >= 32 ? 112 : 72;
    } else if (tp == 64) {
        from = c64 ? 128 : 160;
        again = c64 || log2c == 5 ? 0 : cf16 ? 384 : log2c >= 10 ? 352 : 320;
    } else if (log2c == 9) {
        from = tp == 32 ? (cf16 ? 72 : 60) : 1;
    } else if (log2c == 10) {
        from = cf16 ? 128 : 84;
    } else if (log2c >= 11) {
        const bool late = tp == 32 || (log2c == 13 && tp == 16);
        from = late ? 160 : c64 && ((log2c == 12 && tp == 16) || (log2c == 13 && tp == 8)) ? 100 : 84;
        if (tp == 32 && log2c == 12)
            again = c64 ? 400 : 320;
        else if (tp == 32 && cf16)
            again = 320;
        else if (tp == 16 && log2c == 13)
            again = c64 ? 344 : 272;
    }
    if (256 * blocks < (int64_t)from * cus)
        return false;
    return blocks <= cus || 256 * blocks >= (int64_t)again * cus;
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
