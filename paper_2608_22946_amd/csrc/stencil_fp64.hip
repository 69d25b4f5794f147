// Level-operator kernels with FP64 arithmetic: the FP64 mode's operands and the outer residual
// of the other modes (FP64 operands, FP32 result).
#include "stencil_impl.h"

namespace helm {

template hipError_t launch_stencil<double, c64, c64, c64>(const LevelArgs<double> &, const StencilCall &,
                                                          const RedBuf &, hipStream_t);
template hipError_t launch_stencil<double, c64, c64, c32>(const LevelArgs<double> &, const StencilCall &,
                                                          const RedBuf &, hipStream_t);

}  // namespace helm
