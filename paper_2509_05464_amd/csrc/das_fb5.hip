// Delay-and-sum kernels for blocks of 5 frames.
#include "das_kernel.hpp"

namespace fq {
DasFn das_fn5(int at, int interp, bool wide, int groups) { return das_pick<5>(at, interp, wide, groups); }
}  // namespace fq
