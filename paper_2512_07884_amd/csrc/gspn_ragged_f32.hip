// Scan kernel for maps of any size (gspn_ragged_impl.hpp): f32 storage.
#include "gspn_ragged_impl.hpp"

namespace gspn {
hipError_t launch_ragged_f32(const FwdParams& p, bool reverse, void* e_lo, hipStream_t s) {
    return launch_ragged_type<float>(p, 0, reverse, e_lo, s);
}
}  // namespace gspn
