// Variants of the step kernel: a head's blocks on one XCD.  (In files of their own so that they are compiled side by side.)
#include "fkv_step_dev.h"

#pragma clang fp contract(off)

namespace fkv {
bool launch_step_kernel_home(const StepArgs& a, int dtype, int G, bool past, int rows, size_t lds, hipStream_t st) {
  return launch_step_kernel_variant<true, true>(a, dtype, G, past, rows, lds, st);
}
}  // namespace fkv
