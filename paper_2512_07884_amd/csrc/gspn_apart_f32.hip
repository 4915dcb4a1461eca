// Scan kernel for calls of few planes (gspn_apart_impl.hpp): fp32 storage.
#include "gspn_apart_impl.hpp"

namespace gspn {
hipError_t launch_apart_f32(const ApartArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s) {
    return launch_apart_type<float>(a, reverse, threads, nv, lds, s);
}
}  // namespace gspn
