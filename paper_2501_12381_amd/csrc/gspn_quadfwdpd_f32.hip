// Generic resident forward, unmerged outputs, fp32.
#include "gspn_quadfwd_impl.hpp"

namespace gspn {
template hipError_t launch_quad_fwd_pd<float, false>(QFwdParams p, hipStream_t st);
template hipError_t launch_quad_fwd_pd<float, true>(QFwdParams p, hipStream_t st);
}  // namespace gspn
