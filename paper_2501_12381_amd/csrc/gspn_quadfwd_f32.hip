// Generic resident forward, merged outputs, fp32; dispatch
// of the unmerged ones (gspn_quadfwdpd_*).
#include "gspn_quadfwd_impl.hpp"

namespace gspn {
extern template hipError_t launch_quad_fwd_pd<float, false>(QFwdParams p, hipStream_t st);
extern template hipError_t launch_quad_fwd_pd<float, true>(QFwdParams p, hipStream_t st);
hipError_t quad_fwd_f32(const ResidentFwdArgs& a) {
  if (a.u_pd && !a.y_pd) return hipErrorInvalidValue;  // a merged y with per-direction u: streaming family
  const QFwdParams p = quad_fwd_params(a);
  hipStream_t st = (hipStream_t)a.stream;
  if (a.y_pd) return a.logits ? launch_quad_fwd_pd<float, true>(p, st) : launch_quad_fwd_pd<float, false>(p, st);
  return a.logits ? launch_quad_fwd<float, true>(p, st) : launch_quad_fwd<float, false>(p, st);
}
bool quad_fwd_fits(int H, int W, bool unmerged) { return quad_fwd_size_fits(H, W, unmerged); }
}  // namespace gspn
