// fd_step3d_f16_cached.hip -- the 3D step kernels with IEEE half wavefields that
// read float32 p with ordinary loads (kPCached), for the forms that have
// kernels of their own for it.
// A translation unit of its own, so that the storage forms'
// instantiations compile in parallel.
#include "fd_step3d.h"

namespace fd {

StepFn step3d_kernel_f16_cached(int r, int mode, int shape) { return step3d_get_cached<Store::F16>(r, mode, shape); }

}  // namespace fd
