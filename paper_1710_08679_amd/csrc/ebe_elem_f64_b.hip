// Pipelined and coloured forms of the quadratic EBE product by single
// elements, FP64, 9 to 16 cases (the kernel is in pipe_kernel.h; the files
// compile in parallel).
#include "pipe_kernel.h"

namespace ebe {

#define EBE_INST(n)                                                                                             \
  template hipError_t launch_pipe<double, n, 2, false>(const ebe_mesh*, const void*, void*, bool, bool, bool, \
                                                       const int*, hipStream_t, double*, bool);                 \
  template hipError_t launch_pipe_lds<double, n>(const ebe_mesh*, const void*, void*, bool, bool, bool,       \
                                                 const int*, hipStream_t, double*, bool);
EBE_INST(9) EBE_INST(10) EBE_INST(11) EBE_INST(12) EBE_INST(13) EBE_INST(14) EBE_INST(15) EBE_INST(16)
#undef EBE_INST

}  // namespace ebe
