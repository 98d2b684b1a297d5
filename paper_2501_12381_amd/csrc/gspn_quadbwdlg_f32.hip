// Generic resident backward, Eq. 6 logits, fp32.
#include "gspn_quadbwd_impl.hpp"

namespace gspn {
template hipError_t launch_quad_bwd<float, true>(QBwdParams p, hipStream_t st);
}  // namespace gspn
