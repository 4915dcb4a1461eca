// Scan kernel for maps of any height and width: odd sides, rows that start at any element.  Lines of up to 768 positions in fp32
// storage and 1280 in 16-bit storage (1072 with logits): a chunk of eight lines is at most two granules per loading thread.
// 16-bit forward calls whose merged output the line-by-line kernels sum in fp32 on chip keep the fp32 tile: with it the LDS
// ends at 900 positions on narrow maps (687 with logits) and has no room for planes of about 33 700 (30 000) to 40 500 pixels.
// Forward, forward with h_save, and the reverse sweep of the backward call; global scan, GSPN-local, weights as logits.
//
// One workgroup owns one (image, channel) plane.  A direction is walked in chunks of K scan lines that pass through LDS:
//   load    a loading thread holds one or two granules of a chunk (16 B of one image row: x, lam, u and the three weights)
//           in registers, requested a whole chunk ahead.  16-byte requests at element alignment: rows of an odd width start
//           anywhere, and the memory pipe takes them, so no width needs a narrower path;
//   stage   lam*x in fp32 and the weights (taps outside the line and lines without a predecessor zeroed, logits
//           normalised in fp32) go to LDS as [scan line][position]: a vertical scan's granules along a line, a horizontal
//           scan's across eight (four) lines, which is where the horizontal directions are turned;
//   scan    a line is cut into parts, one wave each, NV positions per lane.  A part covers 8 positions of its neighbours on
//           either side beside its own, so that 8 scan steps need nothing from outside: the waves meet once per 8 lines
//           (one barrier), not once per line.  h replaces lam*x in LDS;
//   finish  the thread that loaded a granule reads its h back, multiplies by u and adds the
//           product to the merged output: an fp32 tile of the plane in LDS (one rounding when all directions are in),
//           or, for planes that do not fit, y in global memory, one direction after the other in a fixed order.
// Both directions of an axis run at once where the tile fits, half of the waves each; where their chunks cross in the
// middle of the map the second waits for the first, so the order of every sum is fixed.
//
// What bounds it: the chain of the scanning wave -- one per direction of a plane, and the LDS holds one plane of 100x167 -- and
// the LDS traffic of staging behind it.  2 x 256 channels 100x167 in bf16: 122 us forward (1.5 TB/s of its 0.18 GB; line by
// line 968), 130 with h_save, 303 backward; the LDS index unit is active in 32 % of a CU's busy cycles, 14 % bank conflicts.
#pragma once
#include "gspn_unaligned.hpp"

namespace gspn {

constexpr int RG_FWD = 0, RG_SAVE = 1, RG_BWD = 2;
constexpr int RG_ROUNDS = 2;     // granules of a chunk per loading thread, at most
constexpr int RG_SUB = 8;        // scan steps between two meetings of the waves = positions a part shares with each neighbour

struct RaggedArgs {
    FwdParams p;
    void* hs_lo;                 // reverse sweep in 16-bit storage: low halves of e (high halves: p.hs); e stays fp32 between the passes
    int nd;                      // directions of an axis walked at once (1 or 2)
    int tile;                    // 1: merged output in an LDS tile; 0: in global memory
    int tile_pitch, tile_off;    // floats per row, byte offset in LDS
    int K[2], parts[2], own[2], pitch[2], pitch2[2];     // per axis (0 vertical, 1 horizontal): lines per chunk, waves per line, positions a wave owns, LDS slots per line (of {lam*x, w0, w1}; of tap 2)
    int w2_off[2], edge_off[2];               // byte offsets in LDS: tap 2 (16-bit weights), edge lines
};

bool ragged_plan(const FwdParams& p, int dtype, bool merge_rounds, RaggedArgs* out, int* threads, int* nv, size_t* lds);

namespace {

// element e (compile-time) of a granule in storage bits / widened
template <typename T> __device__ __forceinline__ uint32_t rg_bits(u32x4 v, int e) {
    if constexpr (sizeof(T) == 4) return v[e];
    else return (e & 1) ? v[e >> 1] >> 16 : v[e >> 1] & 0xffffu;
}
template <typename T> __device__ __forceinline__ float rg_elem(u32x4 v, int e) {
    if constexpr (sizeof(T) == 4) return __uint_as_float(v[e]);
    else return (e & 1) ? word_hi<T>(v[e >> 1]) : word_lo<T>(v[e >> 1]);
}
template <typename T> __device__ __forceinline__ void rg_store_bits(T* p, uint32_t bits) {
    if constexpr (sizeof(T) == 4) *(uint32_t*)p = bits;
    else *(uint16_t*)p = (uint16_t)bits;
}
// LDS by byte address (the pointer form costs an addition of the array's base per access)
template <typename V> __device__ __forceinline__ V lds_get(uint32_t addr) { return *(const __attribute__((address_space(3))) V*)addr; }
template <typename V> __device__ __forceinline__ void lds_set(uint32_t addr, V v) { *(__attribute__((address_space(3))) V*)addr = v; }

// One pass over the plane: one direction, or both directions of an axis at once.
template <typename T, int MODE, bool LOGITS, int NV, bool HORZ>
struct RaggedPass {
    static constexpr int E = 16 / (int)sizeof(T);
    static constexpr bool BWD = MODE == RG_BWD;
    static constexpr bool WIDE = LOGITS || sizeof(T) == 4;        // weights in LDS as fp32
    static constexpr int SB = WIDE ? 16 : 8;                      // bytes of {lam*x, w0, w1[, w2]} per position

    const RaggedArgs& a;
    char* lds;
    int H, W, HW, S, L, K, pitch, pitch2;
    int tid, nthr;               // this thread among the threads of its direction
    int wave, part, parts;
    int d, rev;                  // direction slot; rev: this pass walks the lines from the last to the first
    int plane, bg;
    int lo, hi;                  // where a 16-byte window may start, relative to the plane
    const T *X, *LAM, *U, *W0;
    T *Y, *HS, *LO;
    int dsel, dcount, nchunks;
    bool first;                  // global merge: y is overwritten
    char* stA; char* stW2; float* edge; float* tile;

    struct Regs { u32x4 x, l, u, w0, w1, w2, y; };       // a granule: x, lam, weights of the next chunk; u and y of the current one

    __device__ __forceinline__ RaggedPass(const RaggedArgs& args, char* l) : a(args), lds(l) {}

    struct Gran { bool on; int off, col, row, slot, step, slot2, step2, sh, shw, n; };
    // slot of a position of a line: a vertical scan's line has one slot of padding per granule, which spreads the banks of
    // lanes a granule apart
    static __device__ __forceinline__ int line_slot(int pos) { return HORZ ? pos : pos + pos / E; }
    // this thread's granule of chunk k: image row and first column (a multiple of E), pixel offset, LDS slot of its
    // element 0 and the step to the next, the number of elements inside the row, the shifts of its windows
    __device__ __forceinline__ Gran gran(int r, int k) const {
        Gran g;
        const int q = tid + r * nthr;
        if constexpr (HORZ) {
            const int gpr = K / E;
            const int row = q / gpr, gi = q - row * gpr;
            g.row = row;
            g.col = rev ? S - k * K - gi * E - E : k * K + gi * E;         // S: the width in whole granules
            const int t0 = gi * E + (rev ? E - 1 : 0);
            g.slot = t0 * pitch + row;
            g.step = rev ? -pitch : pitch;
            g.slot2 = t0 * pitch2 + row;
            g.step2 = rev ? -pitch2 : pitch2;
            g.n = min(E, W - g.col);
            g.on = row < H && g.col >= 0 && g.n > 0;
        } else {
            const int gpl = (W + E - 1) / E;
            const int t = q / gpl;
            g.col = (q - t * gpl) * E;
            const int st = k * K + t;
            g.row = rev ? S - 1 - st : st;
            g.slot = t * pitch + line_slot(g.col);
            g.step = 1;
            g.slot2 = t * pitch2 + g.col;
            g.step2 = 1;
            g.n = min(E, W - g.col);
            g.on = t < K && st < S;
        }
        g.off = g.row * W + g.col;
        asm volatile("" : "+v"(g.slot), "+v"(g.slot2), "+v"(g.off));       // addresses are computed per chunk, not kept in registers
        const int offw = g.off + wshift();
        g.sh = g.off - min(max(g.off, lo), hi);
        g.shw = offw - min(max(offw, lo), hi);
        return g;
    }
    // reverse sweep: a line takes the weights of the line swept before it
    __device__ __forceinline__ int wshift() const { return BWD ? (rev ? 1 : -1) * (HORZ ? 1 : W) : 0; }

    __device__ __forceinline__ void load(int k, int r, Regs& q) const {
        const Gran g = gran(r, k);
        if (!g.on) return;
        const int o = g.off - g.sh;
        q.x = rg_load(X + o);
        q.l = rg_load(LAM + o);
        const int ow = g.off + wshift() - g.shw;
        q.w0 = rg_load(W0 + ow);
        q.w1 = rg_load(W0 + HW + ow);
        q.w2 = rg_load(W0 + 2 * (size_t)HW + ow);
    }
    // what finish() of the chunk needs: requested with the chunk's scan
    __device__ __forceinline__ void load_late(int k, int r, Regs& q) const {
        const Gran g = gran(r, k);
        if (!g.on) return;
        q.u = rg_load(U + (g.off - g.sh));
        if (!a.tile && !first) q.y = rg_load((const T*)Y + (g.off - g.sh));
    }

    // registers of the chunk -> LDS
    __device__ __forceinline__ void stage(int k, int r, const Regs& in) const {
        const Gran g = gran(r, k);
        if (!g.on) return;
        __builtin_amdgcn_sched_barrier(0);
        u32x4 x = in.x, l = in.l, w0 = in.w0, w1 = in.w1, w2 = in.w2;
        if (__any(g.sh != 0 || g.shw != 0)) {        // first / last granule of a tensor
            x = rg_realign<T>(x, g.sh); l = rg_realign<T>(l, g.sh);
            w0 = rg_realign<T>(w0, g.shw); w1 = rg_realign<T>(w1, g.shw); w2 = rg_realign<T>(w2, g.shw);
        }
        // lines whose weights are never read: the first line of the scan, of a stretch (by the line the weights
        // belong to), and, in a reverse sweep, the line after the last
        const int S1 = (HORZ ? W : H) - 1, drev = d & 1, kc = a.p.kchunk;
        int wl = (HORZ ? g.col : g.row) + (BWD ? (rev ? 1 : -1) : 0);      // line the weights of element 0 belong to
        uint32_t dead = 0;                                                 // bit e: the weights of element e are not read
        if constexpr (HORZ) {
            const int e0 = (drev ? S1 : 0) - wl;                           // element on the first line of the scan
            if (e0 >= 0 && e0 < E) dead |= 1u << e0;
            if constexpr (BWD) { const int e1 = (drev ? -1 : W) - wl; if (e1 >= 0 && e1 < E) dead |= 1u << e1; }
            if (kc > 0) {
                int m = (wl + (drev ? 1 : 0) + 2 * kc) % kc;               // wl >= -E; 2*kc + wl may be negative only for kc < 4
                if (m < 0) m += kc;
#pragma unroll
                for (int e = 0; e < E; ++e) { if (m == 0) dead |= 1u << e; m = m + 1 == kc ? 0 : m + 1; }
            }
            dead |= ~((1u << g.n) - 1u) & ((1u << E) - 1u);                // beyond the row: a scan from the right starts there, with 0
        } else {
            const bool z = (BWD && (wl < 0 || wl > S1)) || starts_stretch(drev ? S1 - wl : wl, S, drev, kc);
            dead = z ? (1u << E) - 1 : 0u;
        }
        const bool row_first = g.row == 0, row_last = g.row == H - 1;
        float av[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            av[e] = rg_elem<T>(l, e) * rg_elem<T>(x, e);
            if constexpr (HORZ) av[e] = e < g.n ? av[e] : 0.f;
        }
        if constexpr (WIDE) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if constexpr (sizeof(T) == 2) __builtin_amdgcn_sched_barrier(0);        // element by element: registers
                const bool o0 = HORZ ? row_first : (e == 0 && g.col == 0);
                const bool o2 = HORZ ? row_last : (g.col + e == W - 1);
                float f0 = rg_elem<T>(w0, e), f1 = rg_elem<T>(w1, e), f2 = rg_elem<T>(w2, e);
                if constexpr (LOGITS) softmax3(f0, f1, f2, o0, o2);
                const bool dd = (dead >> e) & 1u;
                f0 = (dd || o0) ? 0.f : f0; f1 = dd ? 0.f : f1; f2 = (dd || o2) ? 0.f : f2;
                const u32x4 v = {__float_as_uint(av[e]), __float_as_uint(f0), __float_as_uint(f1), __float_as_uint(f2)};
                *(u32x4*)(stA + (size_t)(g.slot + e * g.step) * 16) = v;
            }
        } else {
            if (dead) {                                     // few granules: clear the elements that are not read
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t m = (((dead >> (2 * i)) & 1u) ? 0u : 0xffffu) | (((dead >> (2 * i + 1)) & 1u) ? 0u : 0xffff0000u);
                    w0[i] &= m; w1[i] &= m; w2[i] &= m;
                }
            }
            if constexpr (HORZ) {
                const uint32_t m0 = row_first ? 0u : 0xffffffffu, m2 = row_last ? 0u : 0xffffffffu;
#pragma unroll
                for (int i = 0; i < 4; ++i) { w0[i] &= m0; w2[i] &= m2; }
            } else {
                if (g.col == 0) w0[0] &= 0xffff0000u;
                const int el = W - 1 - g.col;
                if (el < E) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) w2[i] &= (el >> 1) != i ? 0xffffffffu : ((el & 1) ? 0xffffu : 0xffff0000u);
                }
            }
            uint32_t w01[E];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                w01[2 * i] = __builtin_amdgcn_perm(w1[i], w0[i], 0x05040100u);          // {w0 lo, w1 lo}
                w01[2 * i + 1] = __builtin_amdgcn_perm(w1[i], w0[i], 0x07060302u);      // {w0 hi, w1 hi}
            }
            if constexpr (HORZ) {
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const int s = g.slot + e * g.step;
                    *(u32x2*)(stA + (size_t)s * 8) = u32x2{__float_as_uint(av[e]), w01[e]};
                    *(uint16_t*)(stW2 + (size_t)(g.slot2 + e * g.step2) * 2) = (uint16_t)rg_bits<T>(w2, e);
                }
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) *(u32x2*)(stA + (size_t)(g.slot + e) * 8) = u32x2{__float_as_uint(av[e]), w01[e]};
                *(u32x4*)(stW2 + (size_t)g.slot2 * 2) = w2;
            }
        }
    }

    // h of the chunk from LDS: merged output, and h_save (e of the reverse sweep)
    __device__ __forceinline__ void finish(int k, int r, const Regs& in) const {
        const Gran g = gran(r, k);
        if (!g.on) return;
        __builtin_amdgcn_sched_barrier(0);
        u32x4 u = in.u, yv = in.y;
        if (__any(g.sh != 0)) {
            u = rg_realign<T>(u, g.sh);
            if (!a.tile && !first) yv = rg_realign<T>(yv, g.sh);
        }
        float h[E], y[E];
#pragma unroll
        for (int e = 0; e < E; ++e) h[e] = *(const float*)(stA + (size_t)(g.slot + e * g.step) * SB);
#pragma unroll
        for (int e = 0; e < E; ++e) y[e] = rg_elem<T>(u, e) * h[e];
        const bool full = g.n == E;
        if constexpr (MODE != RG_FWD) {
            u32x4 v, lw;
            if constexpr (sizeof(T) == 4) {
                v = u32x4{__float_as_uint(h[0]), __float_as_uint(h[1]), __float_as_uint(h[2]), __float_as_uint(h[3])};
            } else if constexpr (BWD) {                  // e as two 16-bit halves of its fp32 word
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[i] = __builtin_amdgcn_perm(__float_as_uint(h[2 * i + 1]), __float_as_uint(h[2 * i]), 0x07060302u);
                    lw[i] = __builtin_amdgcn_perm(__float_as_uint(h[2 * i + 1]), __float_as_uint(h[2 * i]), 0x05040100u);
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = pack_word<T>(h[2 * i], h[2 * i + 1]);
            }
            if (full) {
                rg_store(HS + g.off, v);
                if constexpr (BWD && sizeof(T) == 2) rg_store(LO + g.off, lw);
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e)
                    if (e < g.n) {
                        rg_store_bits(HS + g.off + e, rg_bits<T>(v, e));
                        if constexpr (BWD && sizeof(T) == 2) rg_store_bits(LO + g.off + e, rg_bits<T>(lw, e));
                    }
            }
        }
        if (a.tile) {
            float* tp = tile + g.row * a.tile_pitch + g.col;
            // the tile's rows are whole granules: what lies beyond the image row is never read
#pragma unroll
            for (int i = 0; i < E / 4; ++i) {
                float4 t = ((float4*)tp)[i];
                t.x += y[4 * i]; t.y += y[4 * i + 1]; t.z += y[4 * i + 2]; t.w += y[4 * i + 3];
                ((float4*)tp)[i] = t;
            }
        } else {
            if (!first) {
#pragma unroll
                for (int e = 0; e < E; ++e) y[e] += rg_elem<T>(yv, e);
            }
            u32x4 v;
            if constexpr (sizeof(T) == 4) v = u32x4{__float_as_uint(y[0]), __float_as_uint(y[1]), __float_as_uint(y[2]), __float_as_uint(y[3])};
            else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = pack_word<T>(y[2 * i], y[2 * i + 1]);
            }
            if (full) rg_store(Y + g.off, v);
            else {
#pragma unroll
                for (int e = 0; e < E; ++e)
                    if (e < g.n) rg_store_bits(Y + g.off + e, rg_bits<T>(v, e));
            }
        }
    }

    // The scan of nsub * 8 lines of the chunk by a scanning wave; h: state of this lane's positions.  The LDS reads of HL
    // lines are issued while the HL lines before them are computed: one wave per SIMD scans, and nothing else hides their
    // latency.  MEET: the line is shared with other waves, which exchange the last line every 8 steps (a line's h then goes
    // to LDS after the meeting, when no neighbour reads lam*x there any more).
    template <bool MEET>
    __device__ __forceinline__ void scan(int nsub, float (&h)[NV], int& parity, int& until) const {
        constexpr int HL = WIDE ? (NV == 1 ? 4 : NV == 2 ? 2 : 1) : (NV <= 2 ? 4 : 2);      // what the registers hold twice
        constexpr int NB = RG_SUB / HL;
        constexpr int NW2 = WIDE ? 1 : (NV % 2 ? NV : NV / 2);
        const int lane = threadIdx.x & 63;
        const int pos = part * a.own[HORZ] - (MEET ? RG_SUB : 0) + lane * NV;
        const int own_end = min(L, (part + 1) * a.own[HORZ]);
        const bool mine = pos >= part * a.own[HORZ] && pos < own_end;      // own[] and pos are multiples of NV
        // lanes without a position use the NV spare slots at the end of the lines (their state is kept at 0)
        const int pc = min(max(pos, 0), (L - 1) / NV * NV);
        const bool spare = !MEET && pos >= L;
        const int first_slot = spare ? pitch - NV : line_slot(pc);
        bool valid[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) valid[v] = pos + v >= 0 && pos + v < L;
        int dv[NV];                                     // bytes from the lane's first slot to that of position v
#pragma unroll
        for (int v = 0; v < NV; ++v) dv[v] = (NV == 3 && !HORZ && !spare) ? (line_slot(pc + v) - line_slot(pc)) * SB : v * SB;
        struct Lines { float a[HL][NV]; uint32_t w[HL][NV][WIDE ? 3 : 1], w2[HL][NW2]; };
        // byte offsets in LDS of the next line to read and of the next line whose h is stored: running sums, one addition per
        // line (left to itself the compiler keeps an address per line of the block in registers and adds to each)
        const uint32_t line_a = (uint32_t)(pitch * SB), line_w = (uint32_t)(pitch2 * 2);
        const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
        uint32_t ra = lds0 + (uint32_t)(stA - lds) + (uint32_t)(first_slot * SB), rw = lds0 + (uint32_t)(stW2 - lds) + (uint32_t)(pc * 2), rh = ra;
        auto read = [&](Lines& q) {
#pragma unroll
            for (int j = 0; j < HL; ++j) {
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    if constexpr (WIDE) {
                        const u32x4 t = lds_get<u32x4>(ra + dv[v]);
                        q.a[j][v] = __uint_as_float(t[0]); q.w[j][v][0] = t[1]; q.w[j][v][1] = t[2]; q.w[j][v][2] = t[3];
                    } else {
                        const u32x2 t = lds_get<u32x2>(ra + dv[v]);
                        q.a[j][v] = __uint_as_float(t[0]); q.w[j][v][0] = t[1];
                    }
                }
                ra += line_a;
                asm volatile("" : "+v"(ra));
                if constexpr (!WIDE) {
#pragma unroll
                    for (int i = 0; i < NW2; ++i) {
                        if constexpr (NV % 2) q.w2[j][i] = lds_get<uint16_t>(rw + 2 * i);
                        else q.w2[j][i] = lds_get<uint32_t>(rw + 4 * i);
                    }
                    rw += line_w;
                    asm volatile("" : "+v"(rw));
                }
            }
        };
        float hout[NV];                                           // h of the line, for LDS
        auto line = [&](const Lines& q, int j) {
            // a stretch starts with the next line: nothing is carried into it, whatever the state holds (the weights there
            // are 0 already); a mask, not a branch: a wave alone on its SIMD pays some 16 clocks for each
            const bool keep = --until != 0;
            until = keep ? until : a.p.kchunk;
            float av[NV], w0[NV], w1[NV], w2[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                av[v] = q.a[j][v];
                if constexpr (WIDE) { w0[v] = __uint_as_float(q.w[j][v][0]); w1[v] = __uint_as_float(q.w[j][v][1]); w2[v] = __uint_as_float(q.w[j][v][2]); }
                else { w0[v] = word_lo<T>(q.w[j][v][0]); w1[v] = word_hi<T>(q.w[j][v][0]); w2[v] = NV % 2 ? word_lo<T>(q.w2[j][v % NW2]) : (v & 1) ? word_hi<T>(q.w2[j][v / 2]) : word_lo<T>(q.w2[j][v / 2]); }
            }
            // one chain of FMAs per position in the line-by-line kernels' order -- own tap, the neighbour before, the neighbour
            // after -- so that the states are theirs bit for bit (products of the reverse sweep summed in pairs instead: glam of
            // fp32 maps 9 % further from 64 bits in the mean, up to 2.4 times)
            float hn[NV];
            if constexpr (BWD) {
                // (a lane's positions beyond the line come after those inside, or are all of its positions: their taps are read as 0)
#pragma unroll
                for (int v = 0; v < NV; ++v) hn[v] = fmaf(w1[v], h[v], av[v]);
                const float lt = from_lane_below(valid[NV - 1] ? w2[NV - 1] : 0.f), lh = from_lane_below(h[NV - 1]);
#pragma unroll
                for (int v = 0; v < NV; ++v) hn[v] = fmaf(v == 0 ? lt : w2[v - 1], v == 0 ? lh : h[v - 1], hn[v]);
#pragma unroll
                for (int v = 0; v < NV; ++v) w0[v] = valid[v] ? w0[v] : 0.f;
                const float rt = from_lane_above(w0[0]), rh_ = from_lane_above(h[0]);
#pragma unroll
                for (int v = 0; v < NV; ++v) hn[v] = fmaf(v == NV - 1 ? rt : w0[v + 1], v == NV - 1 ? rh_ : h[v + 1], hn[v]);
            } else {
                const float lin = from_lane_below(h[NV - 1]), rin = from_lane_above(h[0]);
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const float lf = v == 0 ? lin : h[v - 1], rt = v == NV - 1 ? rin : h[v + 1];
                    hn[v] = fmaf(w2[v], rt, fmaf(w0[v], lf, fmaf(w1[v], h[v], av[v])));
                }
            }
#pragma unroll
            for (int v = 0; v < NV; ++v) { hout[v] = hn[v]; h[v] = (valid[v] && keep) ? hn[v] : 0.f; }
        };
        auto put = [&](const float (&hv)[NV]) {                   // h of the next line
#pragma unroll
            for (int v = 0; v < NV; ++v) lds_set<float>(rh + dv[v], hv[v]);
            rh += line_a;
            asm volatile("" : "+v"(rh));
        };
        Lines buf[2];
        read(buf[0]);
        for (int s = 0; s < nsub; ++s) {
            float hb[MEET ? RG_SUB : 1][NV];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                static_assert(NB % 2 == 0, "the two line sets alternate");
                if (i + 1 < NB || s + 1 < nsub) read(buf[(i + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < HL; ++j) {
                    line(buf[i & 1], j);
                    if constexpr (MEET) {
#pragma unroll
                        for (int v = 0; v < NV; ++v) hb[i * HL + j][v] = hout[v];
                    } else {
                        put(hout);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (MEET) {
                float* el = edge + (parity ? pitch2 : 0);
                if (mine) {
#pragma unroll
                    for (int v = 0; v < NV; ++v) el[pc + v] = h[v];
                }
                lds_barrier();             // every wave has read this block of lines; the last line is in `el`
#pragma unroll
                for (int v = 0; v < NV; ++v) { const float t = el[pc + v]; h[v] = valid[v] ? t : 0.f; }
                parity ^= 1;
                if (mine) {
#pragma unroll
                    for (int j = 0; j < RG_SUB; ++j) put(hb[j]);
                } else {
                    rh += RG_SUB * line_a;
                }
            }
        }
    }

    __device__ __forceinline__ void run(int d_first, int dcount_, bool first_) {
        const FwdParams& p = a.p;
        constexpr int ax = HORZ ? 1 : 0;
        dcount = dcount_; first = first_;
        const int nwaves = __builtin_amdgcn_readfirstlane(blockDim.x >> 6);
        const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int per = dcount == 2 ? nwaves / 2 : nwaves;       // waves of a direction
        dsel = w >= per ? 1 : 0;
        part = w - dsel * per;
        d = d_first + dsel;
        rev = BWD ? !(d & 1) : (d & 1);
        H = p.H; W = p.W; HW = H * W;
        S = HORZ ? (W + E - 1) / E * E : H; L = HORZ ? H : W;
        K = a.K[ax]; pitch = a.pitch[ax]; pitch2 = a.pitch2[ax]; parts = a.parts[ax];
        nthr = (per - parts) * 64;                               // the first `parts` waves of a direction scan, the others load
        tid = (int)threadIdx.x - (dsel * per + parts) * 64;
        const size_t planes = (size_t)p.B * p.C, groups = (size_t)p.B * p.G;
        const size_t pc = (size_t)plane * HW;
        const size_t slot_c = p.shared ? 0 : (size_t)d * planes * HW;
        const size_t slot_w = p.shared ? 0 : (size_t)d * groups * 3 * HW;
        X = (const T*)p.x + pc; LAM = (const T*)p.lam + slot_c + pc; U = (const T*)p.u + slot_c + pc;
        W0 = (const T*)p.w + slot_w + (size_t)bg * 3 * HW;
        Y = (T*)p.y + pc;
        HS = MODE != RG_FWD ? (T*)p.hs + (size_t)d * planes * HW + pc : nullptr;
        LO = (BWD && sizeof(T) == 2) ? (T*)a.hs_lo + (size_t)d * planes * HW + pc : nullptr;
        // a window may reach into the neighbouring planes of the tensor, not beyond its ends
        lo = bg == 0 ? 0 : -HW;
        hi = bg == (int)groups - 1 ? HW - E : 2 * HW - E;
        stA = lds + (size_t)dsel * K * pitch * SB;
        stW2 = lds + a.w2_off[ax] + (size_t)dsel * K * pitch2 * 2;
        edge = (float*)(lds + a.edge_off[ax]) + dsel * 2 * pitch2;
        tile = (float*)(lds + a.tile_off);

        nchunks = (S + K - 1) / K;
        auto subs = [&](int k) { return (min(K, S - k * K) + RG_SUB - 1) / RG_SUB; };
        // both directions add to the same rows / columns of the tile while their chunks cross
        auto cross = [&](int k) { return dcount == 2 && 2 * (k + 1) * K > S && 2 * k * K < S; };
        if (part < parts) {
            __builtin_amdgcn_s_setprio(3);       // the chain the others wait for (a few per cent either way: 2048 planes 25x31 33.7 -> 32.4 us, 768 of 50x83 63.3 -> 64.7)
            float h[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) h[v] = 0.f;
            int parity = 0;
            // scan steps to the next stretch: cuts lie before image lines 0, kchunk, 2 * kchunk, ..
            int until = 1 << 30;
            if (a.p.kchunk > 0) until = rev && S % a.p.kchunk ? S % a.p.kchunk : a.p.kchunk;
            lds_barrier();
            for (int k = 0; k < nchunks; ++k) {
                if (NV % 2 == 0 && parts > 1) scan<NV % 2 == 0>(subs(k), h, parity, until);      // (lines of one or three positions per lane are one wave's)
                else scan<false>(subs(k), h, parity, until);
                lds_barrier();
                if (cross(k)) lds_barrier();
                lds_barrier();
            }
            __builtin_amdgcn_s_setprio(0);
        } else {
            Regs q[RG_ROUNDS];
            const int gr = HORZ ? (K / E) * H : K * ((W + E - 1) / E);
            const bool two = gr > nthr;                         // a second granule per thread
            load(0, 0, q[0]);
            if (two) load(0, 1, q[1]);
            stage(0, 0, q[0]);
            if (two) stage(0, 1, q[1]);
            lds_barrier();
            for (int k = 0; k < nchunks; ++k) {
                load_late(k, 0, q[0]);
                if (two) load_late(k, 1, q[1]);
                if (k + 1 < nchunks) {
                    load(k + 1, 0, q[0]);
                    if (two) load(k + 1, 1, q[1]);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (parts > 1) for (int s = subs(k); s > 0; --s) lds_barrier();
                lds_barrier();
                if (cross(k)) {
                    if (dsel == 1) lds_barrier();
                    finish(k, 0, q[0]);
                    if (two) finish(k, 1, q[1]);
                    if (dsel == 0) lds_barrier();
                } else {
                    finish(k, 0, q[0]);
                    if (two) finish(k, 1, q[1]);
                }
                if (k + 1 < nchunks) {
                    stage(k + 1, 0, q[0]);
                    if (two) stage(k + 1, 1, q[1]);
                }
                lds_barrier();
            }
        }
    }
};

template <typename T, int MODE, bool LOGITS, int NV>
__global__ void __launch_bounds__(1024) ragged_kernel(RaggedArgs a) {
    extern __shared__ __attribute__((aligned(16))) char rg_lds[];
    constexpr int E = 16 / (int)sizeof(T);
    const FwdParams& p = a.p;
    const int plane = (int)xcd_contiguous_item(blockIdx.x, gridDim.x);
    const int b = plane / p.C, c = plane - b * p.C;
    const int bg = b * p.G + c / p.cpg;
    float* tile = (float*)(rg_lds + a.tile_off);
    if (a.tile) {
        for (int i = threadIdx.x; i < p.H * a.tile_pitch; i += blockDim.x) tile[i] = 0.f;
        // (visible after the first barrier of the first pass)
    }
    bool first = true;
    {
        RaggedPass<T, MODE, LOGITS, NV, false> v(a, rg_lds);
        v.plane = plane; v.bg = bg;
        const int m = p.mask & 3;
        if (m == 3 && a.nd == 2) { v.run(0, 2, first); first = false; }
        else
            for (int i = 0; i < 2; ++i)
                if ((m >> i) & 1) { v.run(i, 1, first); if (!a.tile) __syncthreads(); first = false; }
    }
    {
        RaggedPass<T, MODE, LOGITS, NV, true> v(a, rg_lds);
        v.plane = plane; v.bg = bg;
        const int m = (p.mask >> 2) & 3;
        if (m == 3 && a.nd == 2) v.run(2, 2, first);
        else
            for (int i = 0; i < 2; ++i)
                if ((m >> i) & 1) { v.run(2 + i, 1, first); if (!a.tile) __syncthreads(); first = false; }
    }
    if (a.tile) {
        T* Y = (T*)p.y + (size_t)plane * p.H * p.W;
        const int gpr = (p.W + E - 1) / E;
        for (int q = threadIdx.x; q < p.H * gpr; q += blockDim.x) {
            const int row = q / gpr, col = (q - row * gpr) * E;
            float t[E];
#pragma unroll
            for (int i = 0; i < E / 4; ++i) {
                const float4 f = *(const float4*)(tile + row * a.tile_pitch + col + 4 * i);
                t[4 * i] = f.x; t[4 * i + 1] = f.y; t[4 * i + 2] = f.z; t[4 * i + 3] = f.w;
            }
            u32x4 v;
            if constexpr (sizeof(T) == 4) v = u32x4{__float_as_uint(t[0]), __float_as_uint(t[1]), __float_as_uint(t[2]), __float_as_uint(t[3])};
            else {
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = pack_word<T>(t[2 * i], t[2 * i + 1]);
            }
            T* yp = Y + row * p.W + col;
            if (col + E <= p.W) rg_store(yp, v);
            else {
#pragma unroll
                for (int e = 0; e < E; ++e)
                    if (col + e < p.W) rg_store_bits(yp + e, rg_bits<T>(v, e));
            }
        }
    }
}

template <typename T, int MODE, bool LOGITS>
hipError_t launch_ragged_one(const RaggedArgs& a, int threads, int nv, size_t lds, hipStream_t s) {
    const dim3 grid((unsigned)((size_t)a.p.B * a.p.C)), block(threads);
    void (*k)(RaggedArgs) = nv == 1 ? ragged_kernel<T, MODE, LOGITS, 1> : nv == 2 ? ragged_kernel<T, MODE, LOGITS, 2>
                                    : nv == 3 ? ragged_kernel<T, MODE, LOGITS, 3> : ragged_kernel<T, MODE, LOGITS, 4>;
    const hipError_t e = allow_dynamic_lds((const void*)k, 160 * 1024);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, grid, block, lds, s, a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_ragged_type(const FwdParams& p, int dtype, bool reverse, void* e_lo, hipStream_t s) {
    RaggedArgs a = {};
    int threads, nv;
    size_t lds;
    if (!ragged_plan(p, dtype, reverse, &a, &threads, &nv, &lds)) return hipErrorInvalidValue;
    a.hs_lo = e_lo;
    if (reverse) return p.logits ? launch_ragged_one<T, RG_BWD, true>(a, threads, nv, lds, s) : launch_ragged_one<T, RG_BWD, false>(a, threads, nv, lds, s);
    if (p.hs) return p.logits ? launch_ragged_one<T, RG_SAVE, true>(a, threads, nv, lds, s) : launch_ragged_one<T, RG_SAVE, false>(a, threads, nv, lds, s);
    return p.logits ? launch_ragged_one<T, RG_FWD, true>(a, threads, nv, lds, s) : launch_ragged_one<T, RG_FWD, false>(a, threads, nv, lds, s);
}

}  // namespace
}  // namespace gspn
