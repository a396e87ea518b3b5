// Four-pass row kernels in FP32.
#include "fused_impl.hpp"

namespace le {
void set_fused_f32(int nx, Ops* ops) { set_fused<float>(nx, ops); }
}  // namespace le
