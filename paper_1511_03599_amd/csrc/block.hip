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
// sub-bands) of S spectra. A block takes one CU 9 us (up to 512 channels) to
// 30 us, and a launch of few blocks leaves the other CUs idle, where the FIR
// and FFT launches spread over more of them. Measured, split -> blocked:
// 2048 channels, 16 taps, complex64, 32 blocks 14.6 -> 23.1 us, 128 blocks
// 30.3 -> 23.7; 4096 channels int8, 32 blocks 15.8 -> 25.0, 128 blocks
// 30.5 -> 25.3; sub-bands of 4096 channels, 32 blocks 22.8 -> 27.2, 128
// blocks 44.3 -> 29.1. At 32 taps the split path's FIR of integer samples is
// slow (4096 channels int8: 2 blocks 35.9 -> 34.5), and at 1024 channels the
// lines cross at 8 blocks (complex64, 32 taps 28.3 -> 28.6). Up to 512
// channels one launch is always faster than two (128 channels, 4 blocks 11.8
// -> 9.4).
bool block_pays(int dtype, int tp, int log2c, bool pol, int64_t units, int64_t S)
{
    if (!block_supported(dtype, tp, log2c, pol))
        return false;
    const int64_t rows = block_rows(log2c, pol);
    const int64_t blocks = units * ((S + rows - 1) / rows);
    if (log2c <= 9)
        return true;
    if (!pol && tp >= 32 && (log2c == 10 || dtype == 1 || dtype == 2))
        return blocks >= 8;
    return blocks >= (pol ? 64 : 96);
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
