// The scoring and residual kernels for fp32 keys of 128 dims (a file of their own: they compile in parallel).
#define VEC_DEFINE_PASSES
#include "score_stream.hpp"

namespace vec {

template int launch_passes<float, 128, false>(const KernelArgs<PassParams, false>&, const PassLaunch&, dim3, dim3, hipStream_t);
template int launch_passes<float, 128, true>(const KernelArgs<PassParams, true>&, const PassLaunch&, dim3, dim3, hipStream_t);

}  // namespace vec
