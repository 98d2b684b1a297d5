// Vertical scan in column bands (few planes), fp32 storage and arithmetic.
#include "gspn_vband_impl.hpp"

namespace gspn {
template hipError_t launch_vband<float>(const VScanParams& p, const VBandGeom& g, bool lg, hipStream_t st);
}  // namespace gspn
