// Delay-and-sum kernels for blocks of 1 frame.
#include "das_kernel.hpp"

namespace fq {
DasFn das_fn1(int at, int interp, bool wide, int groups) { return das_pick<1>(at, interp, wide, groups); }
}  // namespace fq
