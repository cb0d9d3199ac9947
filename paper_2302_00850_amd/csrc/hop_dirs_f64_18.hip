// Instantiations of the hop for small launches: F64 spinors, F64_18 links.
#include "hop_dirs.h"

namespace cola {

hipError_t hop_dirs_launch_f64_18(const HopArgs &a, int grid, hipStream_t st) {
    return hop_dirs_launch<SpinorFmt::F64, LinkFmt::F64_18, double>(a, grid, st);
}

}  // namespace cola
