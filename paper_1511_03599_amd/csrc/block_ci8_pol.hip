// Blocked FIR + FFT (block_launch.h) for ci8 input, polarisation-interleaved sub-bands.
#include "block_launch.h"

namespace pfb {

hipError_t launch_block_ci8_pol(const BlockArgs &a, int tp, int log2c, hipStream_t st)
{
    return launch_block_pol<DT_CI8>(a, tp, log2c, st);
}

} // namespace pfb
