// Blocked FIR + FFT (block_launch.h) for ci16 input, 2048 to 8192 channels.
#include "block_launch.h"

namespace pfb {

hipError_t launch_block_ci16_large(const BlockArgs &a, int tp, int log2c, hipStream_t st)
{
    return launch_block_large<DT_CI16>(a, tp, log2c, st);
}

} // namespace pfb
