// Pipelined and coloured forms of the quadratic EBE product, FP32, 5 to 8
// cases (the kernel is in fan_kernel.h; the files compile in parallel).
#include "fan_kernel.h"

namespace ebe {

#define EBE_INST(n)                                                                                             \
  template hipError_t launch_fan<float, n>(const ebe_mesh*, const void*, void*, bool, bool, bool, const int*,      \
                                        hipStream_t, double*, bool);
EBE_INST(5) EBE_INST(6) EBE_INST(7) EBE_INST(8)
#undef EBE_INST

}  // namespace ebe
