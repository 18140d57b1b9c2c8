// Blocked FIR + FFT (block_launch.h) for c64 input, up to 1024 channels.
#include "block_launch.h"

namespace pfb {

hipError_t launch_block_c64_small(const BlockArgs &a, int tp, int log2c, hipStream_t st)
{
    return launch_block_small<DT_C64>(a, tp, log2c, st);
}

} // namespace pfb
