// Delay-and-sum kernels for blocks of 6 frames.
#include "das_kernel.hpp"

namespace fq {
DasFn das_fn6(int at, int interp, bool wide, int groups) { return das_pick<6>(at, interp, wide, groups); }
}  // namespace fq
