// Maps of any size (gspn_ragged_impl.hpp): choice of the launch shape, launches, and the second pass of the backward call.
#include "gspn_ragged_impl.hpp"

namespace gspn {

hipError_t launch_ragged_f32_tile(const RaggedArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s);
hipError_t launch_ragged_f32_mem(const RaggedArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s);
hipError_t launch_ragged_bf16_tile(const RaggedArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s);
hipError_t launch_ragged_bf16_mem(const RaggedArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s);
hipError_t launch_ragged_f16_tile(const RaggedArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s);
hipError_t launch_ragged_f16_mem(const RaggedArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s);

// The launch shape for a call, or false where no shape fits (the line-by-line kernels then take it).
// merge_rounds: the caller's merged output was rounded once per direction anyway (gx of the backward call).
static bool ragged_plan(const FwdParams& p, int dtype, bool merge_rounds, RaggedArgs* out, int* threads, int* nv, size_t* lds) {
    const int H = p.H, W = p.W, es = dtype == 0 ? 4 : 2, E = 16 / es;
    if (p.xt) return false;
    if ((size_t)H * W < 16 || (size_t)H * W >= (1u << 29)) return false;
    const size_t planes = (size_t)p.B * p.C;
    if (planes > 0x7fffffffull) return false;
    const bool wide = dtype == 0 || p.logits;
    const size_t sb = wide ? 16 : 8;
    const size_t cap = 160 * 1024;
    RaggedArgs a = {};
    a.p = p;
    a.tile_pitch = (W + E - 1) / E * E;
    const size_t tile_bytes = (size_t)H * a.tile_pitch * 4;
    const int longest = H > W ? H : W, shortest = H < W ? H : W;
    // The line-by-line kernel sums the four directions of a 16-bit plane in an fp32 LDS tile where its two line buffers leave
    // room; a merge in global memory rounds once per direction, so it is taken only where that kernel would do so too.
    const bool must_tile = dtype != 0 && !merge_rounds && (size_t)H * W * 4 + 2 * (size_t)longest * 4 <= cap;
    // workgroups a CU is to hold: as many as the call has for it, up to 4; sixteen waves per CU (128 registers) in any case
    int wgs_wanted = 1;
    while (wgs_wanted < 4 && (size_t)wgs_wanted * 256 < planes) wgs_wanted *= 2;

    const int kmax[2] = {(H + 7) / 8 * 8, (W + 7) / 8 * 8};
    // One launch shape: how the output is merged (mode 0: LDS tile and both directions of an axis at once; 1: tile and one; 2: y
    // in global memory), chunks of a direction in LDS, bytes of an image row per request in the horizontal directions,
    // workgroups per CU, lines of a vertical chunk at most.
    auto fits = [&](int mode, int nbuf, int seg, int wgs, int kv_most) -> bool {
        a.nd = mode == 0 ? 2 : 1;
        a.tile = mode < 2;
        a.nbuf = nbuf;
        const size_t fixed = a.tile ? tile_bytes : 0;
        const int thr = 1024 / wgs, waves = thr / 64 / a.nd;
        if (waves < 2 || fixed >= cap / wgs) return false;
        const size_t room = cap / wgs - fixed;
        // positions per lane: a line in one wave (no meetings within a chunk) up to 192 positions, beyond that two, and four
        // where the scanning waves would otherwise leave too few for the loads.  With y in global memory the LDS has room for long
        // chunks, and up to 256 positions four of one wave beat two of two or three that meet, provided that both sides are long,
        // for the other axis pays for the idle lanes (both widths timed on 440 calls: 0.92 of the time with a shorter side of 129
        // and more -- 128 planes 226x207 bf16 176 -> 134 us --, 1.06 with 65 to 128, 1.16 below that); with the tile the chunks are
        // short and they do not (1.16; 128 planes 23x251 38 -> 51).
        const bool both_long = longest <= 256 && shortest > 128;
        const int v = longest <= 64 ? 1 : longest <= 128 ? 2 : longest <= 192 ? 3 : !a.tile && both_long ? 4 : longest <= 448 ? 2 : 4;
        for (int ax = 0; ax < 2; ++ax) {
            const int L = ((ax ? H : W) + v - 1) / v * v;
            if (ax == 0) {                                              // granules are written whole, one slot apart
                a.pitch2[ax] = (L + 7) / 8 * 8;
                a.pitch[ax] = (L + E - 1) / E * (E + 1) + v;        // v spare slots at the end of a line
            } else {                                                    // odd: spreads the banks of the turned writes
                a.pitch[ax] = (L + v) | 1;
                a.pitch2[ax] = v % 2 ? L | 1 : L + 2;
            }
        }
        for (int ax = 0; ax < 2; ++ax) {
            const int L = ax ? H : W;
            int parts = L <= 64 * v ? 1 : (L + 64 * v - 2 * RG_SUB - 1) / (64 * v - 2 * RG_SUB), own = 0;
            for (; parts < waves; ++parts) {
                own = ((L + parts - 1) / parts + v - 1) / v * v;
                if (parts == 1 || own + 2 * RG_SUB <= 64 * v) break;
            }
            if (parts >= waves) return false;                        // at least one wave loads
            a.parts[ax] = parts; a.own[ax] = own;
        }
        auto bytes = [&](int ax, int K) {
            return (size_t)a.nd * (nbuf * K * (a.pitch[ax] * sb + (wide ? 0 : a.pitch2[ax] * 2)) + 2 * a.pitch2[ax] * 4);
        };
        auto chunk_fits = [&](int ax, int K) {
            const int gr = ax ? (K / E) * H : K * ((W + E - 1) / E);
            return gr <= RG_ROUNDS * (waves - a.parts[ax]) * 64 && bytes(ax, K) <= room;
        };
        int kh = seg / es < 8 ? 8 : seg / es;
        if (kh > kmax[1]) kh = kmax[1];
        int kv = 8;
        if (!chunk_fits(1, kh) || !chunk_fits(0, kv)) return false;
        while (kv + 8 <= kmax[0] && kv + 8 <= kv_most && chunk_fits(0, kv + 8)) kv += 8;
        a.K[0] = kv; a.K[1] = kh;
        size_t top = 0;
        for (int ax = 0; ax < 2; ++ax) {
            const size_t lines = (size_t)a.nd * nbuf * a.K[ax];
            a.w2_off[ax] = (int)(lines * a.pitch[ax] * sb);
            a.edge_off[ax] = (int)(lines * (a.pitch[ax] * sb + (wide ? 0 : a.pitch2[ax] * 2)));
            const size_t n = bytes(ax, a.K[ax]);
            if (n > top) top = n;
        }
        top = (top + 15) / 16 * 16;
        a.tile_off = (int)top;
        if (top + fixed > cap) return false;
        *out = a; *threads = thr; *nv = v; *lds = top + fixed;
        return true;
    };
    // Which of the shapes that fit.  Every shape was timed on 130 random calls (16 to 300 positions a side and beyond, 8 to 4000
    // planes, the three types): the first of these that fits takes 1.03 of the best one's time in the mean (the order before, one
    // chunk at a time and the longest request first, 1.17).  Several workgroups hide each other's turns, so there a chunk at a time is
    // enough and longer requests come first; a workgroup alone on its CU works on two chunks.  fp32 granules are four columns, so
    // its 32-byte requests make chunks of eight lines, which cost more barriers than one direction after the other costs passes
    // (4 x 512 channels 104x80: 436 -> 337 us).  Examples (us): 512 planes 85x34 bf16 with h_save: two workgroups and chunks in turn 31, one and
    // two chunks 45; 256 planes 80x68: 34 and 28; 112x120 bf16, 1024 planes: {0, 1, 64} 145, {1, 2, 64} 181.
    struct Shape { int mode, nbuf, seg; };
    static const Shape several16[] = {{0, 1, 64}, {0, 1, 32}, {0, 2, 32}, {0, 2, 16}, {1, 1, 64}, {1, 1, 32}};
    static const Shape several32[] = {{0, 1, 64}, {1, 1, 64}, {0, 1, 32}, {0, 2, 32}};
    static const Shape few16[] = {{0, 2, 64}, {0, 2, 32}, {0, 1, 64}, {0, 1, 32}, {1, 2, 64}, {1, 2, 32}, {0, 2, 16}, {1, 1, 64}, {1, 1, 32}, {0, 1, 16}, {1, 2, 16}, {1, 1, 16}};
    static const Shape few32[] = {{0, 2, 64}, {0, 1, 64}, {2, 2, 64}, {0, 2, 32}, {0, 1, 32}, {1, 2, 64}, {1, 2, 32}, {0, 2, 16}, {1, 1, 64}, {1, 1, 32}, {0, 1, 16}, {1, 2, 16}, {1, 1, 16}};
    static const Shape many16[] = {{0, 2, 64}, {0, 1, 64}, {0, 2, 32}, {0, 1, 32}, {1, 2, 64}, {1, 2, 32}, {1, 1, 64}, {1, 1, 32}, {0, 2, 16}, {0, 1, 16}, {1, 2, 16}, {1, 1, 16}};
    static const Shape many32[] = {{0, 2, 64}, {0, 1, 64}, {1, 2, 64}, {2, 2, 64}, {0, 2, 32}, {0, 1, 32}, {1, 2, 32}, {1, 1, 64}, {1, 1, 32}, {0, 2, 16}, {0, 1, 16}, {1, 2, 16}, {1, 1, 16}};
    // y in global memory: with fewer planes than half of the CUs nothing but the second chunk hides the latency; with more,
    // 64 bytes of a row per request count for more (128 planes 320x320 bf16: one chunk and 64 bytes 290, two and 32 bytes 320)
    static const Shape mem_few[] = {{2, 2, 64}, {2, 2, 32}, {2, 1, 64}, {2, 1, 32}, {2, 2, 16}, {2, 1, 16}};
    static const Shape mem_many[] = {{2, 2, 64}, {2, 1, 64}, {2, 2, 32}, {2, 1, 32}, {2, 2, 16}, {2, 1, 16}};
    auto first_of = [&](const Shape* t, int n, int wgs) {
        for (int i = 0; i < n; ++i)
            if (!(must_tile && t[i].mode == 2) && fits(t[i].mode, t[i].nbuf, t[i].seg, wgs, t[i].mode == 2 ? 16 : 32)) return true;
        return false;
    };
    const bool f32 = dtype == 0;
    // Narrow maps, the longer side over 128 positions and three times the other: one axis has few lines of that many positions, the
    // other many short ones, so that the chunks of the first set the LDS.  There requests of 16 and 32 bytes with both directions at
    // once beat longer ones walked one after the other, above all merged in global memory.  Every shape timed on 2660 calls: the
    // first of these that fits takes 1.02 of the best one's time in the mean, of the orders above 1.10 and up to 1.8 (64 planes
    // 233x13 fp32 with h_save: {2, 2, 64} 64, {0, 2, 32} 34 us; 768 planes 508x17 bf16 with h_save: {1, 1, 32} 501, {0, 1, 16} 338).
    // By planes: up to 256, up to 512, more.  In 16 bits the merge in global memory comes last: it rounds gx once per direction; and
    // where the shorter side is long too (over 48 positions), in calls of more than 64 planes, requests of 16 bytes come after the
    // longer ones, for the bytes count there (256 planes 240x80 fp16 with h_save and stretches 110 -> 97).
    struct ShapeAt { int mode, nbuf, seg, wgs; };
    static const ShapeAt narrow16_few[] = {{0, 2, 64, 1}, {0, 2, 32, 1}, {0, 2, 16, 1}, {0, 1, 64, 1}, {0, 1, 16, 1}, {1, 1, 64, 1}, {1, 1, 16, 1}, {2, 2, 64, 1}, {2, 2, 32, 1}, {2, 2, 16, 1}, {2, 1, 64, 1}, {2, 1, 16, 1}};
    static const ShapeAt narrow16_512[] = {{0, 2, 32, 2}, {0, 2, 16, 2}, {0, 1, 64, 2}, {1, 2, 64, 2}, {0, 1, 32, 2}, {0, 1, 16, 2}, {1, 2, 16, 2}, {1, 1, 64, 2}, {0, 2, 64, 1}, {0, 1, 64, 1}, {1, 1, 16, 2}, {0, 1, 32, 1}, {1, 1, 64, 1}, {0, 1, 16, 1}, {1, 1, 16, 1}, {2, 1, 64, 2}, {2, 1, 64, 1}, {2, 2, 32, 1}, {2, 1, 16, 2}, {2, 1, 16, 1}};
    static const ShapeAt narrow16_more[] = {{1, 2, 64, 4}, {1, 2, 16, 4}, {1, 1, 64, 4}, {0, 1, 64, 2}, {1, 1, 16, 4}, {0, 1, 32, 2}, {1, 2, 64, 2}, {0, 1, 16, 2}, {1, 2, 16, 2}, {1, 1, 64, 2}, {0, 1, 64, 1}, {1, 1, 16, 2}, {1, 2, 64, 1}, {0, 1, 32, 1}, {0, 1, 16, 1}, {1, 1, 64, 1}, {1, 1, 32, 1}, {1, 1, 16, 1}, {2, 1, 64, 2}, {2, 1, 64, 1}, {2, 2, 32, 1}, {2, 1, 16, 1}};
    static const ShapeAt narrow32_few[] = {{0, 2, 64, 1}, {0, 2, 32, 1}, {0, 1, 64, 1}, {0, 1, 32, 1}, {1, 2, 64, 1}, {1, 2, 32, 1}, {2, 2, 64, 1}, {2, 2, 32, 1}, {2, 1, 64, 1}, {1, 1, 32, 1}, {2, 1, 32, 1}};
    static const ShapeAt narrow32_512[] = {{0, 1, 64, 2}, {1, 2, 64, 2}, {1, 1, 64, 2}, {1, 1, 32, 2}, {1, 2, 64, 1}, {0, 1, 32, 1}, {2, 2, 64, 1}, {1, 2, 32, 1}, {2, 1, 64, 1}, {1, 1, 32, 1}, {2, 1, 32, 1}};
    static const ShapeAt narrow32_more[] = {{1, 1, 64, 4}, {0, 1, 64, 2}, {1, 1, 32, 4}, {0, 2, 64, 1}, {1, 1, 64, 2}, {1, 2, 32, 2}, {1, 1, 32, 2}, {1, 2, 64, 1}, {0, 1, 32, 1}, {2, 2, 64, 1}, {1, 1, 64, 1}, {1, 2, 32, 1}, {2, 1, 64, 1}, {1, 1, 32, 1}, {2, 1, 32, 1}};
    auto first_at = [&](const auto& table) {
        for (int late16 = !f32 && shortest > 48 && planes > 64; late16 >= 0; --late16)
            for (const ShapeAt& t : table)
                if (!(late16 && (t.seg == 16 || t.mode == 2)) && !(must_tile && t.mode == 2) && fits(t.mode, t.nbuf, t.seg, t.wgs, t.mode == 2 ? 16 : 32)) return true;
        return false;
    };
    if (longest > 128 && 3 * shortest <= longest) {
        if (f32) return planes <= 256 ? first_at(narrow32_few) : planes <= 512 ? first_at(narrow32_512) : first_at(narrow32_more);
        return planes <= 256 ? first_at(narrow16_few) : planes <= 512 ? first_at(narrow16_512) : first_at(narrow16_more);
    }
    for (int wgs = wgs_wanted; wgs > 1; wgs /= 2)
        if (f32 ? first_of(several32, 4, wgs) : first_of(several16, 6, wgs)) return true;
    if (planes <= 256 ? (f32 ? first_of(few32, 13, 1) : first_of(few16, 12, 1)) : (f32 ? first_of(many32, 13, 1) : first_of(many16, 12, 1))) return true;
    const Shape* const mem = planes < 128 ? mem_few : mem_many;
    for (int i = 0; i < 6; ++i)
        for (int wgs = wgs_wanted; wgs >= 1; wgs /= 2)
            if (first_of(mem + i, 1, wgs)) return true;
    return false;
}

// threads per workgroup of a call, 0 where no launch shape fits.  A launch counts its threads in 32 bits -- what is beyond is
// cut off without an error -- so a call of too many planes is left to the line-by-line kernels, which loop over them.
static int ragged_threads(const FwdParams& p, int dtype, bool merge_rounds) {
    RaggedArgs a;
    int threads, nv;
    size_t lds;
    if (!ragged_plan(p, dtype, merge_rounds, &a, &threads, &nv, &lds)) return 0;
    return (unsigned long long)p.B * p.C * threads < (1ull << 32) ? threads : 0;
}
// {merge (0: LDS tile and both directions at once, 1: tile and one, 2: global memory), chunks, bytes of a row per request, workgroups
// per CU, positions per lane, waves per vertical and per horizontal line}: for gspn_any_size_shape
bool ragged_shape(const FwdParams& p, int dtype, bool merge_rounds, int out[7]) {
    RaggedArgs a;
    int threads, nv;
    size_t lds;
    if (!ragged_plan(p, dtype, merge_rounds, &a, &threads, &nv, &lds)) return false;
    const int shape[7] = {a.tile ? 2 - a.nd : 2, a.nbuf, a.K[1] * (dtype == 0 ? 4 : 2), 1024 / threads, nv, a.parts[0], a.parts[1]};
    for (int i = 0; i < 7; ++i) out[i] = shape[i];
    return true;
}
static int lines_walked(unsigned mask, int H, int W) {
    return (int)((mask & 1u) + ((mask >> 1) & 1u)) * H + (int)(((mask >> 2) & 1u) + ((mask >> 3) & 1u)) * W;
}

// Calls of few scan steps, and of many planes of a few pixels, stay with the line-by-line kernels: a pass here loads, turns and
// scans eight lines whatever there are, and a CU holds four planes at most where theirs holds up to 32.  Measured on
// 1500 random calls of up to 900 steps, line by line -> here: 1712 planes 3x251, top to bottom only, 12 -> 45 us; 35488 planes
// 82x4, left to right, 73 -> 188; 5215 planes 4x7, three directions, 20 -> 42; 4128 planes 18x1, all four, 30 -> 43; 18160
// planes 6x11, all four, 128 -> 134.
// Beyond the lines: 664 planes 16x301, top to bottom, 40 -> 29; 4314 planes 124x17, right to left, 225 -> 67.
int ragged_fwd_threads(const FwdParams& p, int dtype) {
    const long long steps = lines_walked(p.mask, p.H, p.W), HW = (long long)p.H * p.W, planes = (long long)p.B * p.C;
    if (steps <= 12 || steps * HW <= 480 || (steps * HW <= 1000 && planes > 2048) || (steps * HW <= 3400 && planes * HW > 100000)) return 0;
    return ragged_threads(p, dtype, false);
}
bool ragged_applicable(const FwdParams& p, int dtype) { return ragged_fwd_threads(p, dtype) != 0; }

static hipError_t launch_ragged(const FwdParams& p, int dtype, bool reverse, bool merge_rounds, void* e_lo, hipStream_t s) {
    RaggedArgs a = {};
    int threads, nv;
    size_t lds;
    if (!ragged_plan(p, dtype, merge_rounds, &a, &threads, &nv, &lds)) return hipErrorInvalidValue;
    a.hs_lo = e_lo;
    if (dtype == 0) return (a.tile ? launch_ragged_f32_tile : launch_ragged_f32_mem)(a, reverse, threads, nv, lds, s);
    if (dtype == 1) return (a.tile ? launch_ragged_bf16_tile : launch_ragged_bf16_mem)(a, reverse, threads, nv, lds, s);
    return (a.tile ? launch_ragged_f16_tile : launch_ragged_f16_mem)(a, reverse, threads, nv, lds, s);
}
hipError_t launch_fwd_ragged(const FwdParams& p, int dtype, hipStream_t s) { return launch_ragged(p, dtype, false, false, nullptr, s); }

// The first pass of the two-pass backward call: e rounded to storage, and gx merged, as the other kernels of that pass do.
bool reverse_sweep_ragged_applicable(const FwdParams& p, int dtype) { return ragged_threads(p, dtype, false) != 0; }
hipError_t launch_reverse_sweep_ragged(const FwdParams& p, int dtype, hipStream_t s) { return launch_ragged(p, dtype, true, false, nullptr, s); }

namespace {

// A granule moved by one element: element e - 1 (BACK) or e + 1, from the lane before or after across the granule's ends.
template <typename T, bool BACK> __device__ __forceinline__ u32x4 next_element(u32x4 v) {
    const uint32_t below = __float_as_uint(from_lane_below(__uint_as_float(v[3]))), above = __float_as_uint(from_lane_above(__uint_as_float(v[0])));
    if constexpr (sizeof(T) == 4) return BACK ? u32x4{below, v[0], v[1], v[2]} : u32x4{v[1], v[2], v[3], above};
    else if constexpr (BACK) return u32x4{__builtin_amdgcn_alignbit(v[0], below, 16), __builtin_amdgcn_alignbit(v[1], v[0], 16), __builtin_amdgcn_alignbit(v[2], v[1], 16), __builtin_amdgcn_alignbit(v[3], v[2], 16)};
    else return u32x4{__builtin_amdgcn_alignbit(v[1], v[0], 16), __builtin_amdgcn_alignbit(v[2], v[1], 16), __builtin_amdgcn_alignbit(v[3], v[2], 16), __builtin_amdgcn_alignbit(above, v[3], 16)};
}

// Second pass of the backward call: per pixel and direction the sum over the group's channels of e * h of the previous
// line (gw), glam = x*e and gu = gy*h.  A thread owns 16 bytes of an image row.  The states of a tap one column away are the
// same granule's, moved by an element (next_element), not a request of their own: lanes hold consecutive granules, and the first
// and last lane of a wave hold their neighbours' for that and nothing else.  A 16-bit request one element off takes the address
// unit four times as long as an aligned one, and there were two or three of eight: backward call of 1024 planes 80x136 bf16 352 ->
// 323 us, of 384 planes 65x191 with logits 124 -> 114.  e comes
// in fp32: from glam itself in fp32 storage, else its two halves from glam (high) and gu (low).  Every thread reads its
// own e before it overwrites it.  SL = 4: the four waves of a workgroup take every fourth channel of the same pixels and
// add their sums in wave order through LDS -- calls have few (image, group) pairs, and one thread walking all channels
// left four waves per CU waiting on one channel's requests at a time; a channel's requests also go out before the
// previous channel is stored.  Bound by memory: 16 B per pixel, channel and direction in 16-bit storage beside x and gy.
constexpr int RG_LIVE = 62;                                    // granules of a wave: all lanes but the first and the last
template <typename T, int SL, bool VERT>
__device__ __forceinline__ void ragged_finish(const BwdParams& p, int d, unsigned blk, float (*red)[3 * 16 / (int)sizeof(T)][64]) {
    constexpr int E = 16 / (int)sizeof(T);
    const int H = p.H, W = p.W, HW = H * W;
    const int gpr = (W + E - 1) / E;
    const int npb = H * gpr;
    const size_t per_dir = (size_t)p.B * p.G * npb;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, slice = SL == 1 ? 0 : wave;
    const long long want = (long long)(SL == 1 ? blk * 4 + wave : blk) * RG_LIVE + lane - 1;
    const bool live = lane > 0 && lane <= RG_LIVE && want < (long long)per_dir;
    const size_t rem = (size_t)min(max(want, 0ll), (long long)per_dir - 1);   // spare lanes read some granule and store nothing
    const int bg = (int)(rem / npb);
    const int q = (int)(rem - (size_t)bg * npb);
    const int row = q / gpr, col = (q - row * gpr) * E;
    const int off = row * W + col;
    const int n = min(E, W - col);                             // valid elements
    const int b = bg / p.G, g = bg - b * p.G;
    const size_t planes = (size_t)p.B * p.C, groups = (size_t)p.B * p.G;
    constexpr bool vert = VERT;
    const int back = (d & 1) ? 1 : -1;                         // to the previous line of the scan
    const int S = vert ? H : W, L = vert ? W : H;
    // windows: own pixels, and per tap; kept inside the tensor (they may reach into neighbouring planes)
    const int lo = bg == 0 ? 0 : -HW, hi = bg == (int)groups - 1 ? HW - E : 2 * HW - E;
    const int sh = off - min(max(off, lo), hi);
    // of a vertical scan the row the states come from, of a horizontal one the rows above and below (its own is hc)
    int toff[2], tsh[2];
    uint32_t tmask[3];                                         // bit e: tap k of element e exists
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int o = off + (vert ? back * W : i == 0 ? -W : W);
        tsh[i] = o - min(max(o, lo), hi);
        toff[i] = o - tsh[i];
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        tmask[k] = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int r = vert ? row + back : row + k - 1, c = vert ? col + e + k - 1 : col + e + back;
            const int line = vert ? row : col + e;
            const bool starts = starts_stretch((d & 1) ? S - 1 - line : line, S, d & 1, p.kchunk);
            if (r >= 0 && r < H && c >= 0 && c < W && e < n && !starts) tmask[k] |= 1u << e;
        }
    }
    const bool moved = __any(sh != 0 || tsh[0] != 0 || tsh[1] != 0);
    const size_t plane0 = ((size_t)b * p.C + (size_t)g * p.cpg) * HW;
    const T* X = (const T*)p.x + plane0 + (off - sh);
    const T* GY = (const T*)p.gy + plane0 + (off - sh);
    const T* HS = (const T*)p.hs + (size_t)d * planes * HW + plane0;
    T* GL = (T*)p.glam + (size_t)d * planes * HW + plane0;
    T* GU = (T*)p.gu + (size_t)d * planes * HW + plane0;
    float acc[3][E];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int e = 0; e < E; ++e) acc[k][e] = 0.f;

    u32x4 eh, el = {0, 0, 0, 0}, xv, gv, hc, ta, tb = {0, 0, 0, 0};
    auto request = [&](int ci, u32x4& eh_, u32x4& el_, u32x4& xv_, u32x4& gv_, u32x4& hc_, u32x4& ta_, u32x4& tb_) {
        const size_t po = (size_t)ci * HW;
        eh_ = rg_load((const T*)GL + po + (off - sh));
        if constexpr (sizeof(T) == 2) el_ = rg_load((const T*)GU + po + (off - sh));
        xv_ = rg_load(X + po); gv_ = rg_load(GY + po); hc_ = rg_load(HS + po + (off - sh));
        ta_ = rg_load(HS + po + toff[0]);
        if constexpr (!VERT) tb_ = rg_load(HS + po + toff[1]);
    };
    request(slice < p.cpg ? slice : 0, eh, el, xv, gv, hc, ta, tb);
    for (int ci = slice; ci < p.cpg; ci += SL) {
        const size_t po = (size_t)ci * HW;
        // the next channel's values before this one's are stored
        u32x4 eh_n, el_n = {0, 0, 0, 0}, xv_n, gv_n, hc_n, ta_n, tb_n = {0, 0, 0, 0};
        const bool more = ci + SL < p.cpg;
        if (more) request(ci + SL, eh_n, el_n, xv_n, gv_n, hc_n, ta_n, tb_n);
        if (moved) {
            eh = rg_realign<T>(eh, sh); el = rg_realign<T>(el, sh); xv = rg_realign<T>(xv, sh); gv = rg_realign<T>(gv, sh); hc = rg_realign<T>(hc, sh);
            ta = rg_realign<T>(ta, tsh[0]); tb = rg_realign<T>(tb, tsh[1]);
        }
        u32x4 t0, t1, t2;
        if constexpr (VERT) {
            t0 = next_element<T, true>(ta); t1 = ta; t2 = next_element<T, false>(ta);
        } else if (d & 1) {
            t0 = next_element<T, false>(ta); t1 = next_element<T, false>(hc); t2 = next_element<T, false>(tb);
        } else {
            t0 = next_element<T, true>(ta); t1 = next_element<T, true>(hc); t2 = next_element<T, true>(tb);
        }
        float gl[E], gu[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            float ev;
            if constexpr (sizeof(T) == 4) ev = __uint_as_float(eh[e]);
            else ev = __uint_as_float((e & 1) ? __builtin_amdgcn_perm(eh[e >> 1], el[e >> 1], 0x07060302u) : __builtin_amdgcn_perm(eh[e >> 1], el[e >> 1], 0x05040100u));
            acc[0][e] = fmaf(((tmask[0] >> e) & 1u) ? ev : 0.f, ((tmask[0] >> e) & 1u) ? rg_elem<T>(t0, e) : 0.f, acc[0][e]);
            acc[1][e] = fmaf(((tmask[1] >> e) & 1u) ? ev : 0.f, ((tmask[1] >> e) & 1u) ? rg_elem<T>(t1, e) : 0.f, acc[1][e]);
            acc[2][e] = fmaf(((tmask[2] >> e) & 1u) ? ev : 0.f, ((tmask[2] >> e) & 1u) ? rg_elem<T>(t2, e) : 0.f, acc[2][e]);
            gl[e] = rg_elem<T>(xv, e) * ev;
            gu[e] = rg_elem<T>(gv, e) * rg_elem<T>(hc, e);
        }
        u32x4 vl, vu;
        if constexpr (sizeof(T) == 4) {
            vl = u32x4{__float_as_uint(gl[0]), __float_as_uint(gl[1]), __float_as_uint(gl[2]), __float_as_uint(gl[3])};
            vu = u32x4{__float_as_uint(gu[0]), __float_as_uint(gu[1]), __float_as_uint(gu[2]), __float_as_uint(gu[3])};
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) { vl[i] = pack_word<T>(gl[2 * i], gl[2 * i + 1]); vu[i] = pack_word<T>(gu[2 * i], gu[2 * i + 1]); }
        }
        if (!live) {
        } else if (n == E) {
            rg_store(GL + po + off, vl);
            rg_store(GU + po + off, vu);
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (e < n) { rg_store_bits(GL + po + off + e, rg_bits<T>(vl, e)); rg_store_bits(GU + po + off + e, rg_bits<T>(vu, e)); }
        }
        if (more) { eh = eh_n; el = el_n; xv = xv_n; gv = gv_n; hc = hc_n; ta = ta_n; tb = tb_n; }
    }
    if constexpr (SL > 1) {
        if (slice > 0) {
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int e = 0; e < E; ++e) red[slice - 1][k * E + e][lane] = acc[k][e];
        }
        __syncthreads();
        if (slice > 0) return;
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int e = 0; e < E; ++e) {
#pragma unroll
                for (int i = 0; i < SL - 1; ++i) acc[k][e] += red[i][k * E + e][lane];
            }
    }
    if (!live) return;
    if (p.logits) {
        // the sum over the group's channels goes through the softmax of its pixel once; logits that are never read stay
        // out, with a gradient of exactly 0
        const T* Z = (const T*)p.w + ((p.shared ? (size_t)0 : (size_t)d * groups) + bg) * 3 * HW;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int line = vert ? row : col + e, pos = vert ? col + e : row;
            const bool unread = e >= n || starts_stretch((d & 1) ? S - 1 - line : line, S, d & 1, p.kchunk);
            float z0 = 0.f, z1 = 0.f, z2 = 0.f;
            if (!unread) { z0 = ldf(Z + off + e); z1 = ldf(Z + HW + off + e); z2 = ldf(Z + 2 * (size_t)HW + off + e); }
            softmax3(z0, z1, z2, pos == 0, pos == L - 1);
            softmax3_grad(acc[0][e], acc[1][e], acc[2][e], z0, z1, z2);
            if (unread) { acc[0][e] = 0.f; acc[1][e] = 0.f; acc[2][e] = 0.f; }
        }
    }
    T* GW = (T*)p.gw + ((size_t)d * groups + bg) * 3 * HW + off;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        u32x4 v;
        if constexpr (sizeof(T) == 4) v = u32x4{__float_as_uint(acc[k][0]), __float_as_uint(acc[k][1]), __float_as_uint(acc[k][2]), __float_as_uint(acc[k][3])};
        else {
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = pack_word<T>(acc[k][2 * i], acc[k][2 * i + 1]);
        }
        if (n == E) rg_store(GW + (size_t)k * HW, v);
        else {
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (e < n) rg_store_bits(GW + (size_t)k * HW + e, rg_bits<T>(v, e));
        }
    }
}

template <typename T, int SL>
__global__ void __launch_bounds__(256) ragged_finish_kernel(BwdParams p, int ndirs) {
    __shared__ float red[SL > 1 ? SL - 1 : 1][3 * 16 / (int)sizeof(T)][64];
    // the workgroups that work on the same pixels in the different directions read the same x and gy: indices 8 apart
    // go to the same XCD one after the other
    const unsigned wg = blockIdx.x;
    int dsel = (int)((wg / 8) % (unsigned)ndirs);
    const unsigned blk = (wg / (8 * (unsigned)ndirs)) * 8 + (wg % 8);
    int d = 0;
    for (;; ++d)
        if ((p.mask >> d) & 1u) { if (dsel == 0) break; --dsel; }
    if (d < 2) ragged_finish<T, SL, true>(p, d, blk, red);
    else ragged_finish<T, SL, false>(p, d, blk, red);
}

// channels of a group over the waves of a workgroup where there are that many
int ragged_slices(const BwdParams& p) { return p.cpg >= 4 ? 4 : 1; }
unsigned long long ragged_finish_blocks(const BwdParams& p, int dtype) {
    const int E = dtype == 0 ? 4 : 8;
    const unsigned long long per_dir = (unsigned long long)p.B * p.G * p.H * ((p.W + E - 1) / E);
    int ndirs = 0;
    for (int d = 0; d < 4; ++d) ndirs += (p.mask >> d) & 1u;
    const unsigned long long gpb = ragged_slices(p) > 1 ? RG_LIVE : 4 * RG_LIVE;
    return ((per_dir + gpb - 1) / gpb + 7) / 8 * 8 * ndirs;         // per direction: a multiple of 8 workgroups
}

}  // namespace

// (a launch counts its threads in 32 bits)
bool ragged_finish_fits(const BwdParams& p, int dtype) { return ragged_finish_blocks(p, dtype) * 256 < (1ull << 32); }

// As for the forward call, with two launches here; line by line a workgroup takes a whole weight group, so more channels per
// group draw the line nearer.  Line by line -> here: 1712 planes 3x251, 16 per group, top to bottom, 39 -> 70 us; 35488 planes
// 82x4, left to right, 148 -> 284; 5215 planes 4x7, one per group, three directions, 44 -> 60.  Beyond the lines: 107 planes
// 14x95, one per group, top to bottom, 21 -> 18; 16 planes 11x5, 16 per group, three directions, logits, 253 -> 37.
int ragged_bwd_threads(const BwdParams& p, int dtype) {
    const long long steps = lines_walked(p.mask, p.H, p.W), HW = (long long)p.H * p.W, groups = (long long)p.B * p.G;
    if (steps <= 2 || (steps <= 4 && p.cpg <= 16) || (steps <= 10 && p.cpg <= 2) || (steps * HW <= 520 && groups > 512)) return 0;
    return ragged_finish_fits(p, dtype) ? ragged_threads(reverse_sweep_params(p), dtype, true) : 0;
}
bool ragged_bwd_applicable(const BwdParams& p, int dtype) { return ragged_bwd_threads(p, dtype) != 0; }

// The second pass: the sums over the channels (e as the first pass left it: glam, in 16-bit storage its halves in glam and gu).
hipError_t launch_ragged_finish(const BwdParams& p, int dtype, hipStream_t s) {
    int ndirs = 0;
    for (int d = 0; d < 4; ++d) ndirs += (p.mask >> d) & 1u;
    const dim3 grid((unsigned)ragged_finish_blocks(p, dtype)), block(256);
    const bool sliced = ragged_slices(p) > 1;
    void (*k)(BwdParams, int) = dtype == 0 ? (sliced ? ragged_finish_kernel<float, 4> : ragged_finish_kernel<float, 1>)
                              : dtype == 1 ? (sliced ? ragged_finish_kernel<bf16_t, 4> : ragged_finish_kernel<bf16_t, 1>)
                                           : (sliced ? ragged_finish_kernel<f16_t, 4> : ragged_finish_kernel<f16_t, 1>);
    hipLaunchKernelGGL(k, grid, block, 0, s, p, ndirs);
    return hipGetLastError();
}

// The two passes of the backward call on any map: the reverse sweep (merged gx, e per direction in fp32), then the sums
// over the channels.
hipError_t launch_bwd_ragged(const BwdParams& p, int dtype, hipStream_t s) {
    const FwdParams f = reverse_sweep_params(p);
    const hipError_t e = launch_ragged(f, dtype, true, true, dtype == 0 ? nullptr : p.gu, s);
    return e == hipSuccess ? launch_ragged_finish(p, dtype, s) : e;
}

}  // namespace gspn
