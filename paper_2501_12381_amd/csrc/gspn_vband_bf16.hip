// Vertical scan in column bands (few planes), bf16 storage with fp32 arithmetic.
#include "gspn_vband_impl.hpp"

namespace gspn {
template hipError_t launch_vband<bf16>(const VScanParams& p, const VBandGeom& g, bool lg, hipStream_t st);
}  // namespace gspn
