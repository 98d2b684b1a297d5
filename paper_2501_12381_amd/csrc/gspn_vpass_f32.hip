// Vertical passes of the two-pass family (scan and adjoint), fp32.
#include "gspn_vpass_impl.hpp"

namespace gspn {
extern template hipError_t launch_vband<float>(const VScanParams& p, const VBandGeom& g, bool lg, hipStream_t st);
template hipError_t launch_vscan<float>(VScanParams p, int out, bool lg, hipStream_t st);
template hipError_t launch_vadj<float>(VAdjParams p, bool lg, hipStream_t st);
}  // namespace gspn
