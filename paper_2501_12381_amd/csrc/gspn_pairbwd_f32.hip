// Generic backward of planes whose states fit LDS one axis at a time, fp32.
#include "gspn_quadbwd_impl.hpp"

namespace gspn {
hipError_t pair_bwd_f32(const ResidentBwdArgs& a, float* hsum, float* gsum) {
  QBwdParams p = quad_bwd_params(a);
  p.hsum = hsum;
  p.gsum = gsum;
  return a.logits ? launch_pair_bwd<float, true>(p, (hipStream_t)a.stream)
                  : launch_pair_bwd<float, false>(p, (hipStream_t)a.stream);
}
bool pair_bwd_fits(int H, int W) { return pair_bwd_size_fits(H, W); }
}  // namespace gspn
