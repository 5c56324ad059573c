// Delay-and-sum kernels for blocks of 8 frames.
#include "das_kernel.hpp"

namespace fq {
DasFn das_fn8(int at, int interp, bool wide, int groups) { return das_pick<8>(at, interp, wide, groups); }
}  // namespace fq
