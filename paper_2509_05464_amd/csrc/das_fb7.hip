// Delay-and-sum kernels for blocks of 7 frames.
#include "das_kernel.hpp"

namespace fq {
DasFn das_fn7(int at, int interp, bool wide, int groups) { return das_pick<7>(at, interp, wide, groups); }
}  // namespace fq
