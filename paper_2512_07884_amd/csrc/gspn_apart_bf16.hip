// Scan kernel for calls of few planes (gspn_apart_impl.hpp): bf16 storage.
#include "gspn_apart_impl.hpp"

namespace gspn {
hipError_t launch_apart_bf16(const ApartArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s) {
    return launch_apart_type<bf16_t>(a, reverse, threads, nv, lds, s);
}
}  // namespace gspn
