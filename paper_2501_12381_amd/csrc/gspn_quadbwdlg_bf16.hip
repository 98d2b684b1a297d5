// Generic resident backward, Eq. 6 logits, bf16 storage (fp32 arithmetic).
#include "gspn_quadbwd_impl.hpp"

namespace gspn {
template hipError_t launch_quad_bwd<bf16, true>(QBwdParams p, hipStream_t st);
}  // namespace gspn
