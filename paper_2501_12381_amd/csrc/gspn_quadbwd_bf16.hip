// Generic resident backward, plain weights, bf16 storage (fp32 arithmetic); dispatch
// of the logits ones (gspn_quadbwdlg_*).
#include "gspn_quadbwd_impl.hpp"

namespace gspn {
extern template hipError_t launch_quad_bwd<bf16, true>(QBwdParams p, hipStream_t st);
hipError_t quad_bwd_bf16(const ResidentBwdArgs& a) {
  const QBwdParams p = quad_bwd_params(a);
  return a.logits ? launch_quad_bwd<bf16, true>(p, (hipStream_t)a.stream)
                  : launch_quad_bwd<bf16, false>(p, (hipStream_t)a.stream);
}
}  // namespace gspn
