// Scan kernel for maps of any size (gspn_ragged_impl.hpp): bf16 storage, merged output in an LDS tile.
#include "gspn_ragged_impl.hpp"

namespace gspn {
hipError_t launch_ragged_bf16_tile(const RaggedArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s) {
    return launch_ragged_type<bf16_t, true>(a, reverse, threads, nv, lds, s);
}
}  // namespace gspn
