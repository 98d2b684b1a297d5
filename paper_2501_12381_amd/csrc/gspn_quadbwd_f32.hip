// Generic resident backward, plain weights, fp32; dispatch
// of the logits ones (gspn_quadbwdlg_*).
#include "gspn_quadbwd_impl.hpp"

namespace gspn {
extern template hipError_t launch_quad_bwd<float, true>(QBwdParams p, hipStream_t st);
hipError_t quad_bwd_f32(const ResidentBwdArgs& a) {
  const QBwdParams p = quad_bwd_params(a);
  return a.logits ? launch_quad_bwd<float, true>(p, (hipStream_t)a.stream)
                  : launch_quad_bwd<float, false>(p, (hipStream_t)a.stream);
}
bool quad_bwd_fits(int H, int W) { return quad_bwd_size_fits(H, W); }
}  // namespace gspn
