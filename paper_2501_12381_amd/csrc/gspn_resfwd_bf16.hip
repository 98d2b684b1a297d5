// Resident-family forward dispatch, bf16 storage (fp32 arithmetic).
// The kernels are instantiated in their own translation units (gspn_fixed_*,
// gspn_widefwd_*, gspn_quadfwd*).
#include "gspn_resident_impl.hpp"

namespace gspn {
hipError_t resident_fwd_bf16(const ResidentFwdArgs& a) { return resident_fwd_t<bf16>(a); }
}  // namespace gspn
