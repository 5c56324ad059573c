// Delay-and-sum kernels for blocks of 2 frames.
#include "das_kernel.hpp"

namespace fq {
DasFn das_fn2(int at, int interp, bool wide, int groups) { return das_pick<2>(at, interp, wide, groups); }
}  // namespace fq
