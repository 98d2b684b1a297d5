// Generic resident forward, unmerged outputs, bf16 storage (fp32 arithmetic).
#include "gspn_quadfwd_impl.hpp"

namespace gspn {
template hipError_t launch_quad_fwd_pd<bf16, false>(QFwdParams p, hipStream_t st);
template hipError_t launch_quad_fwd_pd<bf16, true>(QFwdParams p, hipStream_t st);
}  // namespace gspn
