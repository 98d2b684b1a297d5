// Vertical passes of the two-pass family (scan and adjoint), bf16 storage with fp32 arithmetic.
#include "gspn_vpass_impl.hpp"

namespace gspn {
extern template hipError_t launch_vband<bf16>(const VScanParams& p, const VBandGeom& g, bool lg, hipStream_t st);
template hipError_t launch_vscan<bf16>(VScanParams p, int out, bool lg, hipStream_t st);
template hipError_t launch_vadj<bf16>(VAdjParams p, bool lg, hipStream_t st);
}  // namespace gspn
