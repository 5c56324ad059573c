// Delay-and-sum kernels for blocks of 3 frames.
#include "das_kernel.hpp"

namespace fq {
DasFn das_fn3(int at, int interp, bool wide, int groups) { return das_pick<3>(at, interp, wide, groups); }
}  // namespace fq
