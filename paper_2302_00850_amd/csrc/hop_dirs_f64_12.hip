// Instantiations of the hop for small launches: F64 spinors, F64_12 links.
#include "hop_dirs.h"

namespace cola {

hipError_t hop_dirs_launch_f64_12(const HopArgs &a, int grid, hipStream_t st) {
    return hop_dirs_launch<SpinorFmt::F64, LinkFmt::F64_12, double>(a, grid, st);
}

}  // namespace cola
