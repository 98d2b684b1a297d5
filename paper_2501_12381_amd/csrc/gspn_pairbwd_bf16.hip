// Generic backward of planes whose states fit LDS one axis at a time, bf16 storage (fp32 arithmetic).
#include "gspn_quadbwd_impl.hpp"

namespace gspn {
hipError_t pair_bwd_bf16(const ResidentBwdArgs& a, float* hsum, float* gsum) {
  QBwdParams p = quad_bwd_params(a);
  p.hsum = hsum;
  p.gsum = gsum;
  return a.logits ? launch_pair_bwd<bf16, true>(p, (hipStream_t)a.stream)
                  : launch_pair_bwd<bf16, false>(p, (hipStream_t)a.stream);
}
}  // namespace gspn
