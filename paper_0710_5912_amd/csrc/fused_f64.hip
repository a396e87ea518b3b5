// Four-pass row kernels in FP64.
#include "fused_impl.hpp"

namespace le {
void set_fused_f64(int nx, Ops* ops) { set_fused<double>(nx, ops); }
}  // namespace le
