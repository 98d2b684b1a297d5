// Two-pass forward kernels, fp32.
#include "gspn_large_impl.hpp"

namespace gspn {
extern template hipError_t launch_vscan<float>(VScanParams p, int out, bool lg, hipStream_t st);
hipError_t large_fwd_f32(const LargeFwdArgs& a) { return large_fwd_t<float>(a); }
bool large_fwd_fits(int H, int W, int dtype) {
  return dtype == 0 ? large_fwd_supported<float>(H, W) : large_fwd_supported<bf16>(H, W);
}
// the horizontal pass is also the backward's recompute: instantiated here once
template hipError_t launch_large_h<float>(const LargeHParams& p, int nw, int64_t grid, size_t lds, bool lg,
                                        hipStream_t st);
}  // namespace gspn
