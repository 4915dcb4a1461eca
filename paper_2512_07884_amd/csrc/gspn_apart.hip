// Calls of few planes (gspn_apart_impl.hpp): launch shape, launches, the merge of the directions.
#include "gspn_apart_impl.hpp"

namespace gspn {

hipError_t launch_apart_f32(const ApartArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s);
hipError_t launch_apart_bf16(const ApartArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s);
hipError_t launch_apart_f16(const ApartArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s);

// The ranges of lines of either axis (0 vertical, 1 horizontal), and the work items they make: whole stretches of 32 lines and more,
// shorter ones only while that makes fewer than 1024 work items; a horizontal scan's begin at whole granules
static size_t apart_ranges(const FwdParams& p, int E, int range[2], int nrange[2]) {
    const size_t planes = (size_t)p.B * p.C;
    size_t items = 0;
    for (int stretches = 1;; stretches *= 2) {
        items = 0;
        bool longer = false;
        for (int ax = 0; ax < 2; ++ax) {
            const int S = ax ? p.W : p.H;
            const long long lines = (long long)p.kchunk * stretches;
            const bool cut = p.kchunk > 0 && lines < S && (ax == 0 || lines % E == 0);
            range[ax] = cut ? (int)lines : S;
            nrange[ax] = cut ? (int)((S + lines - 1) / lines) : 1;
            items += planes * 2 * nrange[ax];
            longer |= cut && lines < 32;
        }
        if (!longer || items < 1024) return items;
    }
}
size_t apart_items(const FwdParams& p, int dtype) {
    int range[2], nrange[2];
    return apart_ranges(p, dtype == 0 ? 4 : 8, range, nrange);
}

// The launch shape for a call (of all four directions), or false where no shape fits.
static bool apart_plan(const FwdParams& p, int dtype, ApartArgs* out, int* threads, int* nv, size_t* lds) {
    const int H = p.H, W = p.W, es = dtype == 0 ? 4 : 2, E = 16 / es;
    if (p.mask != 15 || p.xt || (size_t)H * W < 16 || (size_t)H * W >= (1u << 29)) return false;
    const bool wide = dtype == 0 || p.logits;
    ApartArgs a = {};
    a.p = p;
    const size_t items = apart_ranges(p, E, a.range, a.nrange);
    if (items * 1024 >= (1ull << 32)) return false;              // (a launch counts its threads in 32 bits)
    const int longest = H > W ? H : W, v = longest <= 64 ? 1 : longest <= 128 ? 2 : 4;
    // chunks in LDS, bytes of an image row per request in the horizontal directions, workgroups per CU, lines of a vertical chunk at most
    auto fits = [&](int nbuf, int seg, int wgs, int kv_most, bool tight) {
        const int thr = 1024 / wgs, waves = thr / 64;
        const size_t room = 160 * 1024 / wgs;
        a.block = ap_block(wide, v, tight);
        a.nbuf = nbuf;
        auto chunk_fits = [&](int ax, int K, size_t* bytes) {
            const int L = ax ? H : W;
            int parts = 1, own = L;
            if (L > 64 * v) {
                own = 64 * v - 2 * K;
                if (own < 2 * K) return false;
                parts = (L + own - 1) / own;
            }
            if (parts >= waves) return false;                        // at least one wave loads
            a.K[ax] = K; a.parts[ax] = parts; a.own[ax] = own;
            const int places = ax ? (L + v - 1) / v * v : (L + E - 1) / E * E;             // (vertical: granules are written whole)
            const int blocks = (places / v * a.block + (places + 7) / 8 * ap_pad(wide, v) + 15) / 16 * 16;
            a.tail[ax] = parts > 1 ? blocks : 0;
            a.pitch[ax] = blocks + (parts > 1 ? parts * 2 * K * 4 : 0);
            // horizontal: granules of a row, E lines apart, are written at once
            a.skew[ax] = ax ? ((32 - E * a.pitch[ax]) % 128 + 128) % 128 : 0;
            a.chunk[ax] = K * a.pitch[ax] + K / E * a.skew[ax];
            a.edge_len[ax] = parts > 1 ? (L + 3) / 4 * 4 : 0;
            a.edge_off[ax] = nbuf * a.chunk[ax] + 16;                // (16 bytes before the edge lines: h of no one's)
            *bytes = a.edge_off[ax] + (size_t)2 * a.edge_len[ax] * 4;
            const int gr = ax ? (K / E) * H : K * ((W + E - 1) / E);
            return gr <= AP_ROUNDS * (waves - parts) * 64 && *bytes <= room;
        };
        const int kmax[2] = {(a.range[0] + 7) / 8 * 8, (a.range[1] + 7) / 8 * 8};
        int kh = seg / es < 8 ? 8 : seg / es, kv = 8;
        if (kh > kmax[1]) kh = kmax[1];
        size_t bv, bh;
        if (!chunk_fits(1, kh, &bh) || !chunk_fits(0, kv, &bv)) return false;
        while (kv + 8 <= kmax[0] && kv + 8 <= kv_most && chunk_fits(0, kv + 8, &bv)) kv += 8;
        chunk_fits(0, kv, &bv);
        *out = a; *threads = thr; *nv = v; *lds = bv > bh ? bv : bh;
        return true;
    };
    // Which of the shapes that fit, by work items: every shape timed on 14 000 random calls (8 to 1100 planes, 20 to 600 positions a
    // side, the three types, all kinds of calls); the first of these that fits takes 1.02 to 1.04 of the best one's time in the mean.  A
    // workgroup alone on its CU takes long chunks and two of them; where several share a CU they hide each other's turns.
    struct Shape { int nbuf, seg, wgs, kv; };
    static const Shape alone[] = {{2, 64, 1, 32}, {2, 32, 1, 32}, {1, 64, 1, 32}, {1, 32, 1, 16}, {2, 16, 1, 16}, {1, 16, 1, 16}};
    static const Shape two[] = {{2, 64, 4, 16}, {2, 64, 2, 16}, {2, 32, 2, 16}};
    static const Shape four[] = {{2, 64, 4, 16}, {1, 64, 4, 16}, {2, 32, 4, 16}, {1, 32, 4, 16}, {1, 64, 2, 16}, {1, 32, 2, 16}, {2, 32, 2, 16}};
    static const Shape more[] = {{1, 64, 4, 16}, {1, 32, 4, 16}, {1, 64, 2, 16}, {2, 32, 2, 16}, {1, 32, 2, 16}};
    auto first_of = [&](const auto& table, bool tight) {
        for (const Shape& t : table)
            if (fits(t.nbuf, t.seg, t.wgs, t.kv, tight)) return true;
        return false;
    };
    for (int tight = 0; tight < 2; ++tight) {
        if (items > 1024 ? first_of(more, tight) : items > 512 ? first_of(four, tight) : items > 256 && first_of(two, tight)) return true;
        if (first_of(alone, tight)) return true;
    }
    return false;
}

namespace {

// The merge: out = sum over the directions of u * h, in direction order.  h in fp32 (HALVES: its high half in `h`, its low half in
// `lo`).  Elementwise, 16 bytes of the output per thread.
struct CombineArgs { const void* u; const void* h; const void* lo; void* out; size_t n; int shared; };
template <typename T, bool HALVES>
__global__ void __launch_bounds__(256) combine_kernel(CombineArgs a) {
    constexpr int E = 16 / (int)sizeof(T);
    const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * E;
    if (i >= a.n) return;
    if (i + E <= a.n) {
        float y[E];
#pragma unroll
        for (int e = 0; e < E; ++e) y[e] = 0.f;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
            const u32x4 u = rg_load((const T*)a.u + (a.shared ? 0 : d * a.n) + i);
            if constexpr (HALVES) {
                const u32x4 hi = rg_load((const T*)a.h + d * a.n + i), lo = rg_load((const T*)a.lo + d * a.n + i);
#pragma unroll
                for (int e = 0; e < E; ++e)
                    y[e] = fmaf(rg_elem<T>(u, e), __uint_as_float(__builtin_amdgcn_perm(hi[e >> 1], lo[e >> 1], (e & 1) ? 0x07060302u : 0x05040100u)), y[e]);
            } else {
                const float* h = (const float*)a.h + d * a.n + i;
#pragma unroll
                for (int q = 0; q < E / 4; ++q) {
                    const u32x4 hv = rg_load(h + 4 * q);
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[4 * q + e] = fmaf(rg_elem<T>(u, 4 * q + e), __uint_as_float(hv[e]), y[4 * q + e]);
                }
            }
        }
        u32x4 v;
        if constexpr (sizeof(T) == 4) v = u32x4{__float_as_uint(y[0]), __float_as_uint(y[1]), __float_as_uint(y[2]), __float_as_uint(y[3])};
        else {
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = pack_word<T>(y[2 * k], y[2 * k + 1]);
        }
        *(u32x4*)((T*)a.out + i) = v;
    } else {
        for (size_t j = i; j < a.n; ++j) {
            float s = 0.f;
            for (int d = 0; d < 4; ++d) {
                float h;
                if constexpr (HALVES) h = __uint_as_float((uint32_t)((const uint16_t*)a.h)[d * a.n + j] << 16 | ((const uint16_t*)a.lo)[d * a.n + j]);
                else h = ((const float*)a.h)[d * a.n + j];
                s = fmaf(ldf((const T*)a.u + (a.shared ? 0 : d * a.n) + j), h, s);
            }
            stf((T*)a.out + j, s);
        }
    }
}

hipError_t launch_combine(const FwdParams& p, int dtype, const void* h, const void* lo, hipStream_t s) {
    const CombineArgs a = {p.u, h, lo, p.y, (size_t)p.B * p.C * p.H * p.W, p.shared};
    const int E = dtype == 0 ? 4 : 8;
    const dim3 grid((unsigned)((a.n + 256 * E - 1) / (256 * E))), block(256);
    void (*k)(CombineArgs) = dtype == 0 ? combine_kernel<float, false> : dtype == 1 ? (lo ? combine_kernel<bf16_t, true> : combine_kernel<bf16_t, false>)
                                                                                    : (lo ? combine_kernel<f16_t, true> : combine_kernel<f16_t, false>);
    hipLaunchKernelGGL(k, grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_states(const ApartArgs& a, int dtype, bool reverse, int threads, int nv, size_t lds, hipStream_t s) {
    return (dtype == 0 ? launch_apart_f32 : dtype == 1 ? launch_apart_bf16 : launch_apart_f16)(a, reverse, threads, nv, lds, s);
}

}  // namespace

bool apart_applicable(const FwdParams& p, int dtype) {
    ApartArgs a;
    int threads, nv;
    size_t lds;
    return apart_plan(p, dtype, &a, &threads, &nv, &lds);
}
bool apart_bwd_applicable(const BwdParams& p, int dtype) { return apart_applicable(reverse_sweep_params(p), dtype) && ragged_finish_fits(p, dtype); }
// bytes of workspace a forward call needs: the fp32 states, unless h_save holds them
size_t apart_workspace_bytes(const FwdParams& p, int dtype) {
    return dtype == 0 && p.hs ? 0 : (size_t)16 * p.B * p.C * p.H * p.W;
}
hipError_t launch_fwd_apart(const FwdParams& p, int dtype, void* states, hipStream_t s) {
    ApartArgs a = {};
    int threads, nv;
    size_t lds;
    if (!apart_plan(p, dtype, &a, &threads, &nv, &lds)) return hipErrorInvalidValue;
    if (dtype == 0 && !p.hs) a.p.hs = states;
    a.part = (float*)states;
    const hipError_t e = launch_states(a, dtype, false, threads, nv, lds, s);
    return e != hipSuccess ? e : launch_combine(p, dtype, dtype == 0 ? a.p.hs : states, nullptr, s);
}
// Backward: the states of the reverse sweep (e, in fp32: glam, in 16-bit storage its halves in glam and gu), gx from them, then the
// sums over the channels, which turn e into glam and write gu.
hipError_t launch_bwd_apart(const BwdParams& p, int dtype, hipStream_t s) {
    ApartArgs a = {};
    int threads, nv;
    size_t lds;
    const FwdParams f = reverse_sweep_params(p);
    if (!apart_plan(f, dtype, &a, &threads, &nv, &lds)) return hipErrorInvalidValue;
    a.hs_lo = dtype == 0 ? nullptr : p.gu;
    hipError_t e = launch_states(a, dtype, true, threads, nv, lds, s);
    if (e == hipSuccess) e = launch_combine(f, dtype, p.glam, a.hs_lo, s);
    return e == hipSuccess ? launch_ragged_finish(p, dtype, s) : e;
}

}  // namespace gspn
