// Pipelined and coloured forms of the quadratic EBE product by single
// elements, FP64, 1 to 8 cases (the kernel is in pipe_kernel.h; the files
// compile in parallel).
#include "pipe_kernel.h"

namespace ebe {

#define EBE_INST(n)                                                                                             \
  template hipError_t launch_pipe<double, n, 2, false>(const ebe_mesh*, const void*, void*, bool, bool, bool, \
                                                       const int*, hipStream_t, double*, bool);                 \
  template hipError_t launch_pipe_lds<double, n>(const ebe_mesh*, const void*, void*, bool, bool, bool,       \
                                                 const int*, hipStream_t, double*, bool);
EBE_INST(1) EBE_INST(2) EBE_INST(3) EBE_INST(4) EBE_INST(5) EBE_INST(6) EBE_INST(7) EBE_INST(8)
#undef EBE_INST

}  // namespace ebe
