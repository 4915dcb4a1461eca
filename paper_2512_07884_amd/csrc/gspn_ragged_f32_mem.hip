// Scan kernel for maps of any size (gspn_ragged_impl.hpp): f32 storage, merged output in global memory.
#include "gspn_ragged_impl.hpp"

namespace gspn {
hipError_t launch_ragged_f32_mem(const RaggedArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s) {
    return launch_ragged_type<float, false>(a, reverse, threads, nv, lds, s);
}
}  // namespace gspn
