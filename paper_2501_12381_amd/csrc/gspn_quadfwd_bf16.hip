// Generic resident forward, merged outputs, bf16 storage (fp32 arithmetic); dispatch
// of the unmerged ones (gspn_quadfwdpd_*).
#include "gspn_quadfwd_impl.hpp"

namespace gspn {
extern template hipError_t launch_quad_fwd_pd<bf16, false>(QFwdParams p, hipStream_t st);
extern template hipError_t launch_quad_fwd_pd<bf16, true>(QFwdParams p, hipStream_t st);
hipError_t quad_fwd_bf16(const ResidentFwdArgs& a) {
  if (a.u_pd && !a.y_pd) return hipErrorInvalidValue;  // a merged y with per-direction u: streaming family
  const QFwdParams p = quad_fwd_params(a);
  hipStream_t st = (hipStream_t)a.stream;
  if (a.y_pd) return a.logits ? launch_quad_fwd_pd<bf16, true>(p, st) : launch_quad_fwd_pd<bf16, false>(p, st);
  return a.logits ? launch_quad_fwd<bf16, true>(p, st) : launch_quad_fwd<bf16, false>(p, st);
}
}  // namespace gspn
