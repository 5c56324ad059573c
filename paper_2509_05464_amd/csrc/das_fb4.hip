// Delay-and-sum kernels for blocks of 4 frames.
#include "das_kernel.hpp"

namespace fq {
DasFn das_fn4(int at, int interp, bool wide, int groups) { return das_pick<4>(at, interp, wide, groups); }
}  // namespace fq
