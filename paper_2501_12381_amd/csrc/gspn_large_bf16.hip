// Two-pass forward kernels, bf16 storage with fp32 arithmetic.
#include "gspn_large_impl.hpp"

namespace gspn {
extern template hipError_t launch_vscan<bf16>(VScanParams p, int out, bool lg, hipStream_t st);
hipError_t large_fwd_bf16(const LargeFwdArgs& a) { return large_fwd_t<bf16>(a); }
// the horizontal pass is also the backward's recompute: instantiated here once
template hipError_t launch_large_h<bf16>(const LargeHParams& p, int nw, int64_t grid, size_t lds, bool lg,
                                        hipStream_t st);
}  // namespace gspn
