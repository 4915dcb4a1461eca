// Scan kernel of a wave per line (gspn_lines_impl.hpp): f16 storage.
#include "gspn_lines_impl.hpp"

namespace gspn {
hipError_t launch_lines_f16(const LinesArgs& a, bool reverse, int nv, int threads, size_t lds, hipStream_t s) {
    return launch_lines_type<f16_t>(a, reverse, nv, threads, lds, s);
}
}  // namespace gspn
