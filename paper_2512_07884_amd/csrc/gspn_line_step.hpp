// One line of the scan on a wave whose lanes hold NV adjacent positions each.
#pragma once
#include "gspn_tile_common.hpp"

namespace gspn {

// r <- a + w1 h + wb h(before) + wa h(after), one chain of FMAs per position in the line-by-line kernels'
// order, so that the states are theirs bit for bit (products of the reverse sweep summed in pairs instead: glam of fp32 maps
// 9 % further from 64 bits in the mean, up to 2.4 times).  The neighbours' states across lanes are operands of the FMAs themselves
// (DPP), which read 0 from beyond the wave and from lanes that are switched off.  In one block of assembly, because a DPP operand
// has to be two instructions old and nothing but the order here sees to that: the own taps come first.
template <int NV>
__device__ __forceinline__ void line_step(float (&r)[NV], const float (&a)[NV], const float (&h)[NV], const float (&wb)[NV], const float (&w1)[NV], const float (&wa)[NV]) {
#define RG_BEFORE " wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
#define RG_AFTER " wave_shl:1 row_mask:0xf bank_mask:0xf bound_ctrl:1\n"
    static_assert(NV == 1 || NV == 2 || NV == 4, "positions per lane");
    if constexpr (NV == 1)
        asm("v_fma_f32 %0, %4, %2, %1\n"
            "s_nop 0\n"
            "v_fmac_f32_dpp %0, %2, %3" RG_BEFORE
            "v_fmac_f32_dpp %0, %2, %5" RG_AFTER
            : "=&v"(r[0]) : "v"(a[0]), "v"(h[0]), "v"(wb[0]), "v"(w1[0]), "v"(wa[0]));
    else if constexpr (NV == 2)
        asm("v_fma_f32 %0, %8, %4, %2\n"
            "v_fma_f32 %1, %9, %5, %3\n"
            "v_fmac_f32_dpp %0, %5, %6" RG_BEFORE
            "v_fmac_f32_e32 %1, %7, %4\n"
            "v_fmac_f32_e32 %0, %10, %5\n"
            "v_fmac_f32_dpp %1, %4, %11" RG_AFTER
            : "=&v"(r[0]), "=&v"(r[1]) : "v"(a[0]), "v"(a[1]), "v"(h[0]), "v"(h[1]), "v"(wb[0]), "v"(wb[1]), "v"(w1[0]), "v"(w1[1]), "v"(wa[0]), "v"(wa[1]));
    else
        asm("v_fma_f32 %0, %16, %8, %4\n"
            "v_fma_f32 %1, %17, %9, %5\n"
            "v_fma_f32 %2, %18, %10, %6\n"
            "v_fma_f32 %3, %19, %11, %7\n"
            "v_fmac_f32_dpp %0, %11, %12" RG_BEFORE
            "v_fmac_f32_e32 %1, %13, %8\n"
            "v_fmac_f32_e32 %2, %14, %9\n"
            "v_fmac_f32_e32 %3, %15, %10\n"
            "v_fmac_f32_e32 %0, %20, %9\n"
            "v_fmac_f32_e32 %1, %21, %10\n"
            "v_fmac_f32_e32 %2, %22, %11\n"
            "v_fmac_f32_dpp %3, %8, %23" RG_AFTER
            : "=&v"(r[0]), "=&v"(r[1]), "=&v"(r[2]), "=&v"(r[3])
            : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(h[0]), "v"(h[1]), "v"(h[2]), "v"(h[3]), "v"(wb[0]), "v"(wb[1]), "v"(wb[2]), "v"(wb[3]),
              "v"(w1[0]), "v"(w1[1]), "v"(w1[2]), "v"(w1[3]), "v"(wa[0]), "v"(wa[1]), "v"(wa[2]), "v"(wa[3]));
#undef RG_BEFORE
#undef RG_AFTER
}

}  // namespace gspn
