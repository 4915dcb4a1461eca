// Scan kernel of a wave per line (gspn_lines_impl.hpp): its launch shape.
#include "gspn_lines_impl.hpp"

namespace gspn {

hipError_t launch_lines_f32(const LinesArgs& a, bool reverse, int nv, int threads, size_t lds, hipStream_t s);
hipError_t launch_lines_bf16(const LinesArgs& a, bool reverse, int nv, int threads, size_t lds, hipStream_t s);
hipError_t launch_lines_f16(const LinesArgs& a, bool reverse, int nv, int threads, size_t lds, hipStream_t s);

// The launch shape of a call, or false where none fits.
static bool lines_plan(const FwdParams& p, int dtype, LinesArgs* out, int* nv, int* threads, size_t* lds) {
    const int H = p.H, W = p.W, longest = H > W ? H : W;
    if (p.mask != 15 || p.xt || p.kchunk > 0 || W < (dtype == 0 ? 4 : 8) || ln_parts(longest) > 4) return false;
    if ((unsigned long long)p.B * p.C * 512 >= (1ull << 32)) return false;       // a launch counts its threads in 32 bits
    LinesArgs a = {};
    a.p = p;
    *nv = longest > 112 && longest <= 128 ? 2 : 1;
    a.parts[0] = *nv == 1 ? ln_parts(W) : 1;
    a.parts[1] = *nv == 1 ? ln_parts(H) : 1;
    const int waves = 2 * (a.parts[0] > a.parts[1] ? a.parts[0] : a.parts[1]);
    a.pitch = (W + 7) / 8 * 8 + 4;                         // (16 bytes from row to row modulo 32: banks)
    size_t at = (size_t)(H + 7) / 8 * 8 * a.pitch * 4;     // whole units of rows
    a.blk_off = (int)at;
    at += (size_t)waves * LN_BLOCK * *nv;
    a.tail_off = (int)at;
    at += 24 * 16;
    a.edge_off = (int)at;
    a.edge_len = (longest + 7) / 8 * 8;
    if (waves > 2) at += (size_t)4 * a.edge_len * 4;
    if (at > 160 * 1024) return false;
    *threads = waves * 64;
    *lds = at;
    *out = a;
    return true;
}
bool lines_applicable(const FwdParams& p, int dtype) {
    LinesArgs a;
    int nv, threads;
    size_t lds;
    return lines_plan(p, dtype, &a, &nv, &threads, &lds);
}
hipError_t launch_lines(const FwdParams& p, int dtype, bool reverse, void* e_lo, hipStream_t s) {
    LinesArgs a;
    int nv, threads;
    size_t lds;
    if (!lines_plan(p, dtype, &a, &nv, &threads, &lds)) return hipErrorInvalidValue;
    a.hs_lo = e_lo;
    return (dtype == 0 ? launch_lines_f32 : dtype == 1 ? launch_lines_bf16 : launch_lines_f16)(a, reverse, nv, threads, lds, s);
}

}  // namespace gspn
