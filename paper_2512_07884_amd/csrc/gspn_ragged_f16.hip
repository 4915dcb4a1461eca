// Scan kernel for maps of any size (gspn_ragged_impl.hpp): f16 storage.
#include "gspn_ragged_impl.hpp"

namespace gspn {
hipError_t launch_ragged_f16(const FwdParams& p, bool reverse, void* e_lo, hipStream_t s) {
    return launch_ragged_type<f16_t>(p, 2, reverse, e_lo, s);
}
}  // namespace gspn
