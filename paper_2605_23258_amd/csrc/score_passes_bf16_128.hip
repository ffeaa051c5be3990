// The scoring and residual kernels for bf16 keys of 128 dims (a file of their own: they compile in parallel).
#define VEC_DEFINE_PASSES
#include "score_stream.hpp"

namespace vec {

template int launch_passes<bf16_t, 128, false>(PassArgs<false>&, const PassLaunch&, hipStream_t);
template int launch_passes<bf16_t, 128, true>(PassArgs<true>&, const PassLaunch&, hipStream_t);
template int launch_probe<bf16_t, 128>(const PassLaunch&, hipStream_t);

}  // namespace vec
