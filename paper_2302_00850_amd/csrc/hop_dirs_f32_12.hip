// Instantiations of the hop for small launches: F32 spinors, F32_12 links.
#include "hop_dirs.h"

namespace cola {

hipError_t hop_dirs_launch_f32_12(const HopArgs &a, int grid, hipStream_t st) {
    return hop_dirs_launch<SpinorFmt::F32, LinkFmt::F32_12, float>(a, grid, st);
}

}  // namespace cola
