// The scoring and residual kernels for fp32 keys of 64 dims (a file of their own: they compile in parallel).
#define VEC_DEFINE_PASSES
#include "score_stream.hpp"

namespace vec {

template int launch_passes<float, 64, false>(PassArgs<false>&, const PassLaunch&, hipStream_t);
template int launch_passes<float, 64, true>(PassArgs<true>&, const PassLaunch&, hipStream_t);

}  // namespace vec
