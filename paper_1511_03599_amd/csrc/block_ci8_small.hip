// Blocked FIR + FFT (block_launch.h) for ci8 input, up to 1024 channels.
#include "block_launch.h"

namespace pfb {

hipError_t launch_block_ci8_small(const BlockArgs &a, int tp, int log2c, hipStream_t st)
{
    return launch_block_small<DT_CI8>(a, tp, log2c, st);
}

} // namespace pfb
