// Maps beyond 512 rows, the global scan with normalised weights (see gspn_fwd_stream_big.hip).
#include "gspn_fwd_stream_big_impl.hpp"

namespace gspn {

hipError_t launch_stream_big_global(const FwdParams& p, int dtype, bool reverse, hipStream_t s) {
    return launch_big_family<false, false>(p, dtype, reverse, s);
}

hipError_t launch_stream_big_halves(const FwdParams& p, int dtype, float* carry, hipStream_t s) {
    const BigPlan t = plan_big(p, dtype);
    if (!t.ok || t.two_rows || p.mask != 15 || p.kchunk > 0 || p.logits) return hipErrorInvalidValue;
    if (dtype == 0) return p.hs ? launch_big_halves_role<float, true>(p, t, carry, s) : launch_big_halves_role<float, false>(p, t, carry, s);
    if (dtype == 2) return p.hs ? launch_big_halves_role<f16_t, true>(p, t, carry, s) : launch_big_halves_role<f16_t, false>(p, t, carry, s);
    return p.hs ? launch_big_halves_role<bf16_t, true>(p, t, carry, s) : launch_big_halves_role<bf16_t, false>(p, t, carry, s);
}

}  // namespace gspn
