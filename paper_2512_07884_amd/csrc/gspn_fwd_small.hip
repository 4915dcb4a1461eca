// Forward scan of few planes of at most 32x32 (serving one image: 384 channels of 14x14), all four directions.
//
// What bounds such a call is one chain of latencies: the kernels that hold a plane per wave walk its directions one after the other,
// each a round of requests, LDS and lines (384 planes 14x14 bf16: 16 us in sixteen workgroups).  Here the four waves of a workgroup take a
// direction each, of the same 64 / G planes (G lanes to a line: 8, 16 or 32), and there is one round only: every lane requests its
// position of all lines of x, lambda, u and the weights at once, element by element (at most 6 * 32 registers; nothing passes
// through LDS on the way in, so no order or alignment of a row matters), walks the lines with its neighbours' states from DPP, and leaves
// u * h in LDS, where the four directions meet and are added in their order: 16.2 -> 6.9 us back
// to back (a call by itself, its host path included, 15.3 -> 8.1), 768 planes of 7x7 12.5 -> 4.7, 3072 of 14x14 18.0 -> 12.6.  Element requests are an eighth as wide as the plane
// kernels': beyond a few thousand planes those are faster (gspn_dispatch.hip has the lines).
#include "gspn_tile_common.hpp"

namespace gspn {

namespace {

struct SmallArgs { FwdParams p; uint32_t starts[4]; };       // starts: bit t = scan step t of direction d starts a stretch

template <typename T> struct Raw { using type = uint16_t; };
template <> struct Raw<float> { using type = uint32_t; };

template <typename T, int G, bool SAVE, bool LOGITS>
__global__ void __launch_bounds__(256) fwd_small_kernel(SmallArgs a) {
    constexpr int NP = 64 / G, ES = (int)sizeof(T);
    __shared__ float part[4][NP][G][G + 1];
    const FwdParams& p = a.p;
    const int lane = threadIdx.x & 63, d = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int H = p.H, W = p.W, HW = H * W, planes = p.B * p.C;
    const int first = (int)xcd_contiguous_item(blockIdx.x, gridDim.x) * NP;
    const int q = lane / G, j = lane % G;
    const int plane = min(first + q, planes - 1);             // (spare lanes: the last plane once more, not stored)
    const bool vertical = d < 2, reversed = d & 1;
    const int S = vertical ? H : W, L = vertical ? W : H, ss = vertical ? W : 1, sj = vertical ? 1 : W;
    const int jc = min(j, L - 1);
    const bool head = j == 0, tail = j >= L - 1, mine = first + q < planes && j < L;
    const uint32_t starts = a.starts[d];

    const int b = plane / p.C, b0 = first / p.C;
    const int group = b * p.G + (plane - b * p.C) / p.cpg, group0 = b0 * p.G + (first - b0 * p.C) / p.cpg;
    const size_t slot_c = p.shared ? 0 : (size_t)d * planes * HW, slot_w = p.shared ? 0 : (size_t)d * p.B * p.G * 3 * HW;
    const rsrc_t xb = make_rsrc((const T*)p.x + (size_t)first * HW), lb = make_rsrc((const T*)p.lam + slot_c + (size_t)first * HW);
    const rsrc_t ub = make_rsrc((const T*)p.u + slot_c + (size_t)first * HW), wb = make_rsrc((const T*)p.w + slot_w + (size_t)group0 * 3 * HW);
    const uint32_t cv = (uint32_t)(((plane - first) * HW + jc * sj) * ES), wv = (uint32_t)(((group - group0) * 3 * HW + jc * sj) * ES);

    using R = typename Raw<T>::type;
    auto ld = [](rsrc_t rs, uint32_t v, int so) __attribute__((always_inline)) -> R {
        if constexpr (ES == 4) return __builtin_amdgcn_raw_buffer_load_b32(rs, v, so, 0);
        else return __builtin_amdgcn_raw_buffer_load_b16(rs, v, so, 0);
    };
    auto f = [](R r) __attribute__((always_inline)) -> float { T v; __builtin_memcpy(&v, &r, sizeof(T)); return ldf(&v); };
    auto at = [&](int t) __attribute__((always_inline)) { return (reversed ? S - 1 - t : t) * ss; };

    R x[G], l[G], u[G], w0[G], w1[G], w2[G];
#pragma unroll
    for (int t = 0; t < G; ++t) {
        const int so = at(min(t, S - 1)) * ES;                // (past the last line: that line again)
        x[t] = ld(xb, cv, so); l[t] = ld(lb, cv, so);
        w0[t] = ld(wb, wv, so); w1[t] = ld(wb, wv, so + HW * ES); w2[t] = ld(wb, wv, so + 2 * HW * ES);
        u[t] = ld(ub, cv, so);
    }
    float* const out = &part[d][q][0][0] + j * (vertical ? 1 : G + 1);
    const int step = vertical ? G + 1 : 1;
    const rsrc_t hb = make_rsrc(SAVE ? (const T*)p.hs + (size_t)d * planes * HW + (size_t)first * HW : (const T*)p.y);
    float h = 0.f;
#pragma unroll
    for (int t = 0; t < G; ++t) {
        if (t < S) {
            const float c = f(l[t]) * f(x[t]);
            float a0 = head ? 0.f : f(w0[t]), a1 = f(w1[t]), a2 = tail ? 0.f : f(w2[t]);
            if constexpr (LOGITS) softmax3(a0, a1, a2, head, tail);
            float up = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, h), 0x138, 0xf, 0xf, true));   // wave_shr:1
            float dn = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, h), 0x130, 0xf, 0xf, true));   // wave_shl:1
            up = head ? 0.f : up;
            dn = tail ? 0.f : dn;
            const float n = fmaf(a2, dn, fmaf(a0, up, fmaf(a1, h, c)));
            h = (starts >> t) & 1 ? c : n;                    // no predecessor: its weights are not read
            if (mine) {
                out[(reversed ? S - 1 - t : t) * step] = f(u[t]) * h;
                if constexpr (SAVE) {
                    T v; stf(&v, h);
                    R r; __builtin_memcpy(&r, &v, sizeof(T));
                    if constexpr (ES == 4) __builtin_amdgcn_raw_buffer_store_b32(r, hb, cv, at(t) * ES, 0);
                    else __builtin_amdgcn_raw_buffer_store_b16(r, hb, cv, at(t) * ES, 0);
                }
            }
        }
    }
    __syncthreads();
    // the waves share the planes' rows, 64 / G of them at once
    constexpr int WP = NP < 4 ? NP : 4;                       // planes worked on at once
    for (int s = d % WP; s < NP && first + s < planes; s += WP) {
        for (int i = d / WP * NP + q; i < H; i += NP * (4 / WP)) {
            if (j < W) stf((T*)p.y + (size_t)(first + s) * HW + i * W + j, part[0][s][i][j] + part[1][s][i][j] + part[2][s][i][j] + part[3][s][i][j]);
        }
    }
}

template <typename T, int G>
static hipError_t launch(const SmallArgs& a, hipStream_t s) {
    void (*k)(SmallArgs) = a.p.hs ? a.p.logits ? fwd_small_kernel<T, G, true, true> : fwd_small_kernel<T, G, true, false>
                                  : a.p.logits ? fwd_small_kernel<T, G, false, true> : fwd_small_kernel<T, G, false, false>;
    constexpr int NP = 64 / G;
    hipLaunchKernelGGL(k, dim3((unsigned)(((size_t)a.p.B * a.p.C + NP - 1) / NP)), dim3(256), 0, s, a);
    return hipGetLastError();
}

template <typename T>
static hipError_t launch_lines(const SmallArgs& a, hipStream_t s) {
    const int longest = a.p.H > a.p.W ? a.p.H : a.p.W;
    return longest <= 8 ? launch<T, 8>(a, s) : longest <= 16 ? launch<T, 16>(a, s) : launch<T, 32>(a, s);
}

}  // namespace

bool fwd_small_applicable(const FwdParams& p) { return p.mask == 15 && !p.xt && p.H <= 32 && p.W <= 32 && (size_t)p.B * p.C < (1u << 20); }

hipError_t launch_fwd_small(const FwdParams& p, int dtype, hipStream_t s) {
    SmallArgs a;
    a.p = p;
    for (int d = 0; d < 4; ++d) a.starts[d] = (uint32_t)stretch_start_bits(d < 2 ? p.H : p.W, d & 1, p.kchunk, true);
    return dtype == 0 ? launch_lines<float>(a, s) : dtype == 1 ? launch_lines<bf16_t>(a, s) : launch_lines<f16_t>(a, s);
}

}  // namespace gspn
