// Scan kernel for maps of any size (gspn_ragged_impl.hpp): bf16 storage.
#include "gspn_ragged_impl.hpp"

namespace gspn {
hipError_t launch_ragged_bf16(const FwdParams& p, bool reverse, void* e_lo, hipStream_t s) {
    return launch_ragged_type<bf16_t>(p, 1, reverse, e_lo, s);
}
}  // namespace gspn
