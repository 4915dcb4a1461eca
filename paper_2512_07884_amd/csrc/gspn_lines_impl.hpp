// Scan kernel of a wave per line: global scan in all four directions, maps of up to 208 positions a side, rows of at least 16 bytes.
// Forward, forward with h_save, and the reverse sweep of the backward call; weights or logits.
//
// One workgroup owns one (image, channel) plane: two waves, one per direction of an axis, or two per part of a line that one wave does not
// hold.  A wave does everything for its line itself -- requests, turning, the scan, the merge -- and nothing but the output tile is shared:
//   request  16 bytes of an image row per lane, whole rows in a vertical scan, 64 bytes of each row in a horizontal one.  What is on its way
//            stands in registers, four units of eight lines or a chunk of 64 bytes (24 granules per lane), the chip's largest store;
//   turn     tensor by tensor through a block of LDS of the wave's own, written as it was loaded and read back a position per lane (vertical)
//            or a row per lane (horizontal).  An LDS queue works in order, so no wait and no barrier stands between;
//   scan     eight lines with the states in registers, neighbours by DPP (gspn_line_step.hpp), u * h added to the fp32 output tile in LDS
//            (vertical: the direction that reaches a row first stores there).  The two directions change halves at a barrier, so every
//            sum has one order.
// Lines of 65 to 112 positions have two waves, up to 160 three, up to 208 four, which cover eight positions of each neighbour beside their own and
// meet once per eight lines, after the next unit is turned; 16-bit lines of 113 to 128 one wave with two positions per lane and the
// registers of a whole SIMD (128x112 f16, 1128 planes: three waves 1.7 times as long; up to 112 positions it is the two waves that are faster,
// 768 planes 50x83 fp32 57 against 81 us).  The last granule of a tensor, whose window would end beyond it, is read element by element beforehand.
//
// What bounds it: with many planes the lines that the L1s take in (24 planes of 16 bytes' requests per channel, 190 KB at 63x63: 5.6 TB/s over the
// chip, near the fabric's rate), before that the issue of a wave alone with its chain, 13 vector instructions per line.  Counters on
// 4096 planes 128x136 bf16: vector ALUs 19 %, LDS 22 %, address units 55 % of a CU's cycles.  Against the kernels in its place (us):
// 4224 planes 63x63 bf16 192 -> 146, 2304 planes 64x64 84 -> 63 (with h_save 129 -> 88), 1024 planes 160x160 329 -> 242, 768 planes 43x44 with
// logits 36 -> 26, 2648 planes 64x48 with weights of each channel's own 224 -> 84.  Tried and no faster: several channels of a group in step
// for the sake of their weights in the L1 (barriers cost more: 63x63 164 -> 176), requests for lam and u with the non-temporal bit
// (lines that begin inside a 128-byte line are asked for twice: 146 -> 159), turning a unit ahead of the scan (registers).
#pragma once
#include "gspn_line_step.hpp"
#include "gspn_unaligned.hpp"

namespace gspn {

constexpr int LN_FWD = 0, LN_SAVE = 1, LN_BWD = 2;
constexpr int LN_UNIT = 8;       // scan steps whose operands a wave turns and walks at a time = positions a wave shares with its neighbours
constexpr int LN_BLOCK = 4096;   // bytes of a wave's turning block per position of a lane: 64 rows of 64 bytes
// Waves of a line: the first and the last own up to 56 positions, those between 48, each beside 8 of every neighbour's.
__host__ __device__ constexpr int ln_first(int part) { return part == 0 ? 0 : 56 + (part - 1) * 48; }
__host__ __device__ constexpr int ln_parts(int L) { return L <= 64 ? 1 : (L - 64 + 47) / 48 + 1; }

struct LinesArgs {
    FwdParams p;
    void* hs_lo;                 // reverse sweep in 16-bit storage: low halves of e (high halves: p.hs)
    int parts[2];                // waves of a line per axis (0 vertical, 1 horizontal)
    int pitch;                   // floats per row of the output tile
    int blk_off, tail_off, edge_off, edge_len;      // byte offsets in LDS, floats of an edge line
};

namespace {

template <typename T> struct LnBits { typedef uint16_t type; };
template <> struct LnBits<float> { typedef uint32_t type; };

// NV: positions of a line per lane.  Lines are shared between waves with one only.
template <typename T, int MODE, bool LOGITS, int NV>
struct Lines {
    static constexpr int ES = (int)sizeof(T), E = 16 / ES;
    static constexpr bool BWD = MODE == LN_BWD, SAVE = MODE != LN_FWD;
    static constexpr int UC = 64 / ES / LN_UNIT;          // units of a horizontal chunk of 64 bytes; units of a vertical scan in flight
    static constexpr int GPR = 64 * NV / E, NRV = LN_UNIT * GPR / 64;      // granules of a line; per lane and tensor of a vertical unit
    static constexpr int NR = 4 * NV;                     // granules of a chunk per lane and tensor
    typedef typename LnBits<T>::type bits_t;
    // what stands in for a tap that points outside the line
    static __device__ __forceinline__ uint32_t outside() {
        if constexpr (!LOGITS) return 0u;
        else if constexpr (ES == 4) return 0xff800000u;
        else if constexpr (__is_same(T, f16_t)) return 0xfc00fc00u;
        else return 0xff80ff80u;
    }
    // a word with the bits of `outside` where `keep` is clear
    static __device__ __forceinline__ uint32_t put_outside(uint32_t keep, uint32_t w) {
        if constexpr (LOGITS) return (w & keep) | (outside() & ~keep);
        else return w & keep;
    }

    const LinesArgs& a;
    uint32_t lds0, blk;
    int H, W, HW, lane, part, d, plane, bg;
    bool at_end;                 // a window of this plane can meet the end of a tensor
    uint32_t top;                // where a 16-byte window may start at most: bytes from the tensors' pointers
    const char* X;
    char *HS, *LO;
    int parts, start, wn, own_lo, own_hi;        // waves of a line; this wave's window: first position, positions; those it owns
    bool in, mine, valid[NV];    // this lane has a position; ... which the wave owns; ... which of its positions it has

    __device__ __forceinline__ Lines(const LinesArgs& args, char* l) : a(args) {
        lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)l;
    }

    // what a direction reads
    struct From { const char *lam, *u, *w; };
    __device__ __forceinline__ From from(int dir) const {
        const FwdParams& p = a.p;
        const size_t planes = (size_t)p.B * p.C, groups = (size_t)p.B * p.G, pc = (size_t)plane * HW;
        const size_t slot_c = p.shared ? 0 : (size_t)dir * planes * HW, slot_w = p.shared ? 0 : (size_t)dir * groups * 3 * HW;
        From f;
        f.lam = (const char*)((const T*)p.lam + slot_c + pc);
        f.u = (const char*)((const T*)p.u + slot_c + pc);
        f.w = (const char*)((const T*)p.w + slot_w + (size_t)bg * 3 * HW);
        return f;
    }
    __device__ __forceinline__ void load(const From& f, uint32_t o, u32x4& x, u32x4& l, u32x4& u, u32x4& w0, u32x4& w1, u32x4& w2) const {
        x = rg_load((const T*)(X + o));
        l = rg_load((const T*)(f.lam + o));
        w0 = rg_load((const T*)(f.w + o));
        w1 = rg_load((const T*)(f.w + (size_t)HW * ES + o));
        w2 = rg_load((const T*)(f.w + (size_t)HW * (2 * ES) + o));
        u = rg_load((const T*)(f.u + o));
    }
    __device__ __forceinline__ void set_direction(int dir) {
        const FwdParams& p = a.p;
        d = dir;
        const size_t at = (size_t)d * ((size_t)p.B * p.C) * HW + (size_t)plane * HW;
        HS = SAVE ? (char*)((T*)p.hs + at) : nullptr;
        LO = (BWD && ES == 2) ? (char*)((T*)a.hs_lo + at) : nullptr;
    }
    // this wave's window of a line: first position, positions
    __device__ __forceinline__ void window(int axis, int L, int& first, int& count) const {
        const int hi = part == a.parts[axis] - 1 ? L : ln_first(part + 1);
        first = part == 0 ? 0 : ln_first(part) - LN_UNIT;
        count = min(L, hi + LN_UNIT) - first;
    }
    __device__ __forceinline__ void set_window(int axis, int L) {
        parts = a.parts[axis];
        window(axis, L, start, wn);
        own_lo = ln_first(part); own_hi = part == parts - 1 ? L : ln_first(part + 1);
        in = lane * NV < wn;
        mine = start + lane * NV >= own_lo && start + lane * NV < own_hi;
#pragma unroll
        for (int v = 0; v < NV; ++v) valid[v] = lane * NV + v < wn;
    }
    // Granules in registers: a vertical scan has UC units of eight lines on their way, a horizontal one a chunk.
    typedef u32x4 Unit[6][NRV];
    From fv, fh;
    uint32_t offh[NR];           // the wave's granules of that chunk, moved on by every chunk
    // the wave's granules of the horizontal scan's chunk 0 of the row
    __device__ __forceinline__ void place_horizontal() {
        int first = 0, count = 1;
        if (part < a.parts[1]) window(1, H, first, count);
#pragma unroll
        for (int j = 0; j < NR; ++j) offh[j] = (uint32_t)((first + min(j * 16 + lane / 4, count - 1)) * W * ES + (lane & 3) * 16);
    }
    __device__ __forceinline__ void request_chunk(int ch, int s, Unit& r) const {
        const uint32_t lim = ch >= 0 ? top : 0;            // (nothing is left to request: one line)
#pragma unroll
        for (int j = 0; j < NRV; ++j) load(fh, min(offh[s * NRV + j] + (uint32_t)(ch * 64), lim), r[0][j], r[1][j], r[2][j], r[3][j], r[4][j], r[5][j]);
    }

    // the states one line further (forward) or back (reverse sweep; p0, p1, p2: the taps of the line swept before, handed on)
    typedef float fnv __attribute__((ext_vector_type(NV)));
    struct State { float h[NV], p0[NV], p1[NV], p2[NV]; };
    __device__ __forceinline__ void line(State& z, float (&r)[NV], const float (&av)[NV], float (&w0)[NV], float (&w1)[NV], float (&w2)[NV]) const {
        if constexpr (LOGITS) {
#pragma unroll
            for (int v = 0; v < NV; ++v) softmax3(w0[v], w1[v], w2[v], false, false);
        }
        if constexpr (BWD) {
            float wb[NV], wa[NV];
            wb[0] = from_lane_below(z.p2[NV - 1]);
            wa[NV - 1] = from_lane_above(z.p0[0]);
#pragma unroll
            for (int v = 1; v < NV; ++v) { wb[v] = z.p2[v - 1]; wa[v - 1] = z.p0[v]; }
            line_step<NV>(r, av, z.h, wb, z.p1, wa);
#pragma unroll
            for (int v = 0; v < NV; ++v) { z.p0[v] = v == 0 || valid[v] ? w0[v] : 0.f; z.p1[v] = w1[v]; z.p2[v] = w2[v]; }
        } else if constexpr (__is_same(T, f16_t) && !LOGITS) {
            // (taps straight from their 16 bits: the conversion is an operand's, but not of a DPP instruction)
            const float before = from_lane_below(z.h[NV - 1]), after = from_lane_above(z.h[0]);
#pragma unroll
            for (int v = 0; v < NV; ++v) r[v] = fmaf(w1[v], z.h[v], av[v]);
#pragma unroll
            for (int v = 0; v < NV; ++v) r[v] = fmaf(w0[v], v == 0 ? before : z.h[v == 0 ? 0 : v - 1], r[v]);
#pragma unroll
            for (int v = 0; v < NV; ++v) r[v] = fmaf(w2[v], v == NV - 1 ? after : z.h[v == NV - 1 ? v : v + 1], r[v]);
        } else {
            line_step<NV>(r, av, z.h, w0, w1, w2);
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) z.h[v] = v == 0 || valid[v] ? r[v] : 0.f;
    }

    // The last states of a unit pass between the waves of a line: left in LDS after it, taken up before the next one, when that
    // one's operands are turned.
    __device__ __forceinline__ uint32_t edge(int k) const { return lds0 + a.edge_off + (uint32_t)((((d & 1) * 2 + (k & 1)) * a.edge_len + start + lane) * 4); }
    __device__ __forceinline__ void leave(const State& z, int k) const {
        if constexpr (NV == 1) { if (parts > 1 && in && mine) lds_set<float>(edge(k), z.h[0]); }
    }
    __device__ __forceinline__ void take_up(State& z, int k) const {
        if constexpr (NV == 1) {
            if (parts == 1 || k == 0) return;
            lds_barrier();
            if (in && !mine) z.h[0] = lds_get<float>(edge(k - 1));
        }
    }
    // the barriers of a wave that a line does not need
    __device__ __forceinline__ void stand_by(int axis, int n) const {
        for (int k = a.parts[axis] > 1 ? n : 1; k > 0; --k) lds_barrier();
    }
    __device__ __forceinline__ void store(char* to, int row, int col, u32x4 v) const {
        T* const q = (T*)to + (row * W + col);
        if (col + E <= W) rg_store(q, v);
        else {
#pragma unroll
            for (int e = 0; e < E - 1; ++e)
                if (col + e < W) rg_store_bits(q + e, rg_bits<T>(v, e));
        }
    }
    // ---------------------------------------------------------------- vertical directions: a lane holds NV columns
    static constexpr int LINE = 64 * NV * ES;             // bytes of a line in the turning block
    static constexpr int LW = ES == 4 ? NV : 1;           // words of a lane's positions of a line (one 16-bit value: the low half)
    typedef uint32_t VUnit[6][LN_UNIT * LW];              // a lane's values of a unit, in walking order
    static __device__ __forceinline__ float vval(const uint32_t (&c)[LN_UNIT * LW], int i, int v) {
        if constexpr (ES == 4) return __uint_as_float(c[i * LW + v]);
        else return v ? word_hi<T>(c[i]) : word_lo<T>(c[i]);
    }

    // first_ch: the chunk that the wave's horizontal scan begins with, requested here before the last unit is walked
    template <int rev>
    __device__ __forceinline__ void vertical(int first_ch, Unit (&chunk)[UC]) {
        const int n = (H + LN_UNIT - 1) / LN_UNIT;
        const int xat = rev ? n / 2 : (n + 1) / 2;         // units before the two directions change halves
        if (part >= a.parts[0]) {
            place_horizontal();
#pragma unroll
            for (int s = 0; s < UC; ++s) request_chunk(first_ch, s, chunk[s]);
            stand_by(0, n);
            return;
        }
        set_window(0, W);
        const int gcount = (wn + E - 1) / E, flip = rev ? LN_UNIT - 1 : 0, gl = lane % GPR;
        uint32_t off[NRV], wat[NRV];
#pragma unroll
        for (int j = 0; j < NRV; ++j) {
            const int row = j * (64 / GPR) + lane / GPR, g = min(gl, gcount - 1);
            off[j] = (uint32_t)((row * W + start + g * E) * ES);
            wat[j] = blk + (row ^ flip) * LINE + gl * 16;
        }
        const int unit_bytes = LN_UNIT * W * ES;
        const bool has_first = start == 0, has_last = start + wn == W;
        // taps that point outside the line: bits to keep of w0's first word, of w2's words
        const uint32_t one = ES == 4 ? 0xffffffffu : 0xffffu;
        uint32_t keep0 = has_first && gl == 0 ? ~one : 0xffffffffu, keep2[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int el = (W - 1 - start) % E;
            const bool here = has_last && gl == gcount - 1 && (ES == 4 ? el : el >> 1) == i;
            keep2[i] = here ? ~(ES == 2 && (el & 1) ? one << 16 : one) : 0xffffffffu;
        }
        Unit rg[UC];
        auto request = [&](int k, Unit& r) {
            const int u = rev ? n - 1 - k : k;
            const uint32_t lim = k < n ? top : 0;          // (nothing is left to request: one line)
#pragma unroll
            for (int j = 0; j < NRV; ++j) load(fv, min(off[j] + (uint32_t)(u * unit_bytes), lim), r[0][j], r[1][j], r[2][j], r[3][j], r[4][j], r[5][j]);
        };
        // a unit's granules to lines in walking order, a lane's position of each
        auto turn = [&](int k, Unit& r, VUnit& c) {
#pragma unroll
            for (int j = 0; j < NRV; ++j) {
                r[3][j][0] = put_outside(keep0, r[3][j][0]);
#pragma unroll
                for (int i = 0; i < 4; ++i) r[5][j][i] = put_outside(keep2[i], r[5][j][i]);
            }
            const uint32_t at = blk + lane * (NV * ES);
#pragma unroll
            for (int t = 0; t < 6; ++t) {
#pragma unroll
                for (int j = 0; j < NRV; ++j) lds_set<u32x4>(wat[j], r[t][j]);
#pragma unroll
                for (int i = 0; i < LN_UNIT; ++i) {
                    if constexpr (NV * ES == 2) c[t][i] = lds_get<uint16_t>(at + i * LINE);
                    else if constexpr (NV * ES == 4) c[t][i] = lds_get<uint32_t>(at + i * LINE);
                    else { const u32x2 w = lds_get<u32x2>(at + i * LINE); c[t][i * LW] = w[0]; c[t][i * LW + LW - 1] = w[1]; }
                }
            }
            const int u = rev ? n - 1 - k : k;
            if (at_end && u == n - 1 && has_last) {        // the last granule of the tensor, read element by element beforehand
                asm volatile("");                          // (a branch: selects for it would run every time)
                const int line_at = (H - 1 - u * LN_UNIT) ^ flip;
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    const int pos = start + lane * NV + v, e = pos - (W - 1) / E * E;
                    const bool here = e >= 0 && pos < W;
#pragma unroll
                    for (int t = 0; t < 6; ++t) {
                        uint32_t q = lds_get<bits_t>(lds0 + a.tail_off + (d * 6 + t) * 16 + (here ? e * ES : 0));
                        if ((t == 3 && pos == 0) || (t == 5 && pos == W - 1)) q = outside() & one;
#pragma unroll
                        for (int i = 0; i < LN_UNIT; ++i) {
                            uint32_t& w = c[t][ES == 4 ? i * LW + v : i];
                            const uint32_t to = ES == 4 || NV == 1 ? q : v ? (w & 0xffffu) | q << 16 : (w & 0xffff0000u) | q;
                            w = here && i == line_at ? to : w;
                        }
                    }
                }
            }
        };
        State z = {};
        const int row_step = a.pitch * (rev ? -4 : 4);
        const uint32_t tile0 = lds0 + (uint32_t)((start + lane * NV) * 4) + (uint32_t)((rev ? n * LN_UNIT - 1 : 0) * a.pitch * 4);
        auto scan = [&](int k, const VUnit& c) {
            const int u = rev ? n - 1 - k : k;
            take_up(z, k);
            if (k == xat) lds_barrier();
            float hv[LN_UNIT][NV];
            if (in) {
                fnv y[LN_UNIT];
                // the direction that reaches a row first leaves its products there, the other adds to them
                const uint32_t at = tile0 + (uint32_t)(k * LN_UNIT * row_step);
                if (k >= xat) {
#pragma unroll
                    for (int i = 0; i < LN_UNIT; ++i) y[i] = lds_get<fnv>(at + (uint32_t)(i * row_step));
                } else {
#pragma unroll
                    for (int i = 0; i < LN_UNIT; ++i) y[i] = fnv(0.f);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < LN_UNIT; ++i) {
                    float av[NV], w0[NV], w1[NV], w2[NV];
#pragma unroll
                    for (int v = 0; v < NV; ++v) { av[v] = vval(c[1], i, v) * vval(c[0], i, v); w0[v] = vval(c[3], i, v); w1[v] = vval(c[4], i, v); w2[v] = vval(c[5], i, v); }
                    line(z, hv[i], av, w0, w1, w2);
#pragma unroll
                    for (int v = 0; v < NV; ++v) y[i][v] = fmaf(vval(c[2], i, v), hv[i][v], y[i][v]);
                }
                if (NV > 1 || mine) {
#pragma unroll
                    for (int i = 0; i < LN_UNIT; ++i) lds_set<fnv>(at + (uint32_t)(i * row_step), y[i]);
                }
            }
            if constexpr (SAVE) {
                // the states back to granules
#pragma unroll
                for (int half = 0; half < (BWD && ES == 2 ? 2 : 1); ++half) {
#pragma unroll
                    for (int i = 0; i < LN_UNIT; ++i) {
                        const uint32_t at = blk + i * LINE + lane * (NV * ES);
                        if constexpr (ES == 4) {
                            fnv t;
#pragma unroll
                            for (int v = 0; v < NV; ++v) t[v] = hv[i][v];
                            lds_set<fnv>(at, t);
                        } else if constexpr (NV == 1) {
                            if constexpr (BWD) lds_set<uint16_t>(at, (uint16_t)(half == 0 ? __float_as_uint(hv[i][0]) >> 16 : __float_as_uint(hv[i][0])));
                            else { T b; stf(&b, hv[i][0]); lds_set<uint16_t>(at, __builtin_bit_cast(uint16_t, b)); }
                        } else {
                            if constexpr (BWD) lds_set<uint32_t>(at, __builtin_amdgcn_perm(__float_as_uint(hv[i][NV - 1]), __float_as_uint(hv[i][0]), half == 0 ? 0x07060302u : 0x05040100u));
                            else lds_set<uint32_t>(at, pack_word<T>(hv[i][0], hv[i][NV - 1]));
                        }
                    }
                    char* const to = half == 0 ? HS : LO;
                    u32x4 q[NRV];
#pragma unroll
                    for (int j = 0; j < NRV; ++j) q[j] = lds_get<u32x4>(wat[j]);
#pragma unroll
                    for (int j = 0; j < NRV; ++j) {
                        const int row = u * LN_UNIT + j * (64 / GPR) + lane / GPR, col = start + gl * E;
                        if (row < H && col >= own_lo && col < own_hi) store(to, row, col, q[j]);
                    }
                }
            }
            leave(z, k);
        };
        VUnit c;
        auto take = [&](int k, Unit& r) {
            __builtin_amdgcn_sched_barrier(0);
            turn(k, r, c);
            __builtin_amdgcn_sched_barrier(0);
            // (words: left as halves, their conversions are spread over the loads and keep registers)
            if constexpr (__is_same(T, f16_t)) {
#pragma unroll
                for (int t = 0; t < 6; ++t)
#pragma unroll
                    for (int i = 0; i < LN_UNIT * LW; ++i) asm volatile("" : "+v"(c[t][i]));
            }
            if (k == 0) {
                asm volatile("");
                // lines beyond the map (walked backwards they come first), and weights that are never read, those of the first line
                const int beyond = rev ? n * LN_UNIT - H : 0;
#pragma unroll
                for (int t = 0; t < 6; ++t) {
                    if (t == 2) continue;
                    const int end = beyond + (!BWD && t >= 3 ? 1 : 0);
#pragma unroll
                    for (int i = 0; i < LN_UNIT * LW; ++i) c[t][i] = i / LW < end ? 0u : c[t][i];
                }
            }
        };
#pragma unroll
        for (int s = 0; s < UC; ++s) request(s, rg[s]);
        for (int k = 0;; k += UC) {                        // (ways out of the middle, none around a unit: the waits count requests)
            bool last = false;
#pragma unroll
            for (int s = 0; s < UC; ++s) {
                take(k + s, rg[s]);
                if (k + s + 1 == n) { last = true; break; }
                request(k + s + UC, rg[s]);
                __builtin_amdgcn_sched_barrier(0);
                scan(k + s, c);
            }
            if (last) break;
        }
        place_horizontal();
#pragma unroll
        for (int s = 0; s < UC; ++s) request_chunk(first_ch, s, chunk[s]);
        __builtin_amdgcn_sched_barrier(0);
        scan(n - 1, c);
        if (xat == n) lds_barrier();
    }

    // ---------------------------------------------------------------- horizontal directions: a lane holds NV rows
    // The turning block has rows of 64 bytes; their four granules are moved so that the reads of eight neighbouring lanes meet no bank twice.
    static __device__ __forceinline__ uint32_t turned(int row, int g) { return (uint32_t)(row * 64 + ((g ^ (row >> 2)) & 3) * 16); }
    template <bool REV>
    __device__ __forceinline__ void horizontal(Unit (&rg)[UC]) {
        const int n = (W + LN_UNIT - 1) / LN_UNIT, nch = (n + UC - 1) / UC;
        const int xat = REV ? n / 2 : (n + 1) / 2;
        if (part >= a.parts[1]) { stand_by(1, n); return; }
        set_window(1, H);
        const int gl = lane & 3;
        const uint32_t wat = blk + turned(lane / 4, gl);  // (+ j * 1024: rows 16 apart)
        const bool has_first = start == 0, has_last = start + wn == H;
        uint32_t c[6][NV][16];
        auto turn = [&](int ch) {
            // taps that point outside the line
            const uint32_t keep0 = has_first && lane < 4 ? 0u : 0xffffffffu;
#pragma unroll
            for (int i = 0; i < 4; ++i) rg[0][3][0][i] = put_outside(keep0, rg[0][3][0][i]);
#pragma unroll
            for (int t = 0; t < 6; ++t) {
#pragma unroll
                for (int j = 0; j < NR; ++j) lds_set<u32x4>(wat + j * 1024, rg[j / NRV][t][j % NRV]);
#pragma unroll
                for (int v = 0; v < NV; ++v)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const u32x4 q = lds_get<u32x4>(blk + turned(lane * NV + v, g));
#pragma unroll
                        for (int i = 0; i < 4; ++i) c[t][v][g * 4 + i] = q[i];
                    }
            }
            const int gend = (W - 1) / E - ch * 4;         // granule of this chunk with the last column (may lie beyond)
            if (at_end && gend < 4 && has_last) {          // the last granule of the tensor, read element by element beforehand
                asm volatile("");
#pragma unroll
                for (int t = 0; t < 6; ++t) {
                    const u32x4 q = lds_get<u32x4>(lds0 + a.tail_off + (d * 6 + t) * 16);
#pragma unroll
                    for (int v = 0; v < NV; ++v)
#pragma unroll
                        for (int i = 0; i < 16; ++i) c[t][v][i] = lane * NV + v == wn - 1 && i >> 2 == gend ? q[i & 3] : c[t][v][i];
                }
                if (H == 1) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) c[3][0][i] = outside();
                }
            }
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const uint32_t keep2 = has_last && lane * NV + v == wn - 1 ? 0u : 0xffffffffu;
#pragma unroll
                for (int i = 0; i < 16; ++i) c[5][v][i] = put_outside(keep2, c[5][v][i]);
            }
        };
        State z = {};
        uint32_t tile0[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) tile0[v] = lds0 + (uint32_t)((start + min(lane * NV + v, wn - 1)) * a.pitch * 4);
        int kd = 0;                                        // units done
        for (int k = 0; k < nch; ++k) {
            const int ch = REV ? nch - 1 - k : k;
            turn(ch);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < UC; ++s) request_chunk(k + 1 == nch ? -1 : REV ? ch - 1 : ch + 1, s, rg[s]);
            __builtin_amdgcn_sched_barrier(0);
            if (k == 0) {
                asm volatile("");
                // columns beyond the map (walked backwards they come first); weights that are never read: those of the first column
                const int e0 = W - ch * (64 / ES);         // of this chunk: columns inside the map
#pragma unroll
                for (int t = 0; t < 6; ++t) {
                    if (t == 2) continue;
                    const bool weights = !BWD && t >= 3;
                    if (!REV && !weights) continue;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        uint32_t keep;
                        if constexpr (REV) {
                            const int end = weights ? e0 - 1 : e0;         // columns from here on are cleared
                            if constexpr (ES == 4) keep = i < end ? 0xffffffffu : 0u;
                            else keep = 2 * i + 1 < end ? 0xffffffffu : 2 * i < end ? 0xffffu : 0u;
                        } else {
                            if (i > 0) break;
                            keep = ES == 4 ? 0u : 0xffff0000u;
                        }
#pragma unroll
                        for (int v = 0; v < NV; ++v) c[t][v][i] &= keep;
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < UC; ++q) {
                const int uq = REV ? UC - 1 - q : q;       // unit of the chunk
                const int u = ch * UC + uq;
                if (u < n) {
                    take_up(z, kd);
                    if (kd == xat) lds_barrier();
                    // (the words as they are: what is made of them early would have to be kept)
#pragma unroll
                    for (int t = 0; t < 6; ++t)
#pragma unroll
                        for (int v = 0; v < NV; ++v)
#pragma unroll
                            for (int i = 0; i < 16 / UC; ++i) asm("" : "+v"(c[t][v][uq * (16 / UC) + i]));
                    if (in) {
                        float y[NV][LN_UNIT], hv[NV][LN_UNIT];
                        typedef float f32x4 __attribute__((ext_vector_type(4)));
                        const uint32_t col_at = (uint32_t)(u * LN_UNIT * 4);
#pragma unroll
                        for (int v = 0; v < NV; ++v) {
                            const f32x4 ta = lds_get<f32x4>(tile0[v] + col_at), tb = lds_get<f32x4>(tile0[v] + col_at + 16);
#pragma unroll
                            for (int i = 0; i < 4; ++i) { y[v][i] = ta[i]; y[v][4 + i] = tb[i]; }
                        }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int i = 0; i < LN_UNIT; ++i) {
                            const int e = uq * LN_UNIT + (REV ? LN_UNIT - 1 - i : i), o = e % LN_UNIT;     // element of the chunk's row, of the unit's
                            auto val = [&](int t, int v) { if constexpr (ES == 4) return __uint_as_float(c[t][v][e]); else return (e & 1) ? word_hi<T>(c[t][v][e >> 1]) : word_lo<T>(c[t][v][e >> 1]); };
                            float av[NV], w0[NV], w1[NV], w2[NV], r[NV];
#pragma unroll
                            for (int v = 0; v < NV; ++v) { av[v] = val(1, v) * val(0, v); w0[v] = val(3, v); w1[v] = val(4, v); w2[v] = val(5, v); }
                            line(z, r, av, w0, w1, w2);
#pragma unroll
                            for (int v = 0; v < NV; ++v) { hv[v][o] = r[v]; y[v][o] = fmaf(val(2, v), r[v], y[v][o]); }
                        }
#pragma unroll
                        for (int v = 0; v < NV; ++v) {
                            if (!(NV > 1 ? valid[v] : mine)) continue;
                            lds_set<f32x4>(tile0[v] + col_at, f32x4{y[v][0], y[v][1], y[v][2], y[v][3]});
                            lds_set<f32x4>(tile0[v] + col_at + 16, f32x4{y[v][4], y[v][5], y[v][6], y[v][7]});
                            if constexpr (SAVE) {
                                const int row = start + lane * NV + v, col = u * LN_UNIT;
                                const float (&hr)[LN_UNIT] = hv[v];
                                if constexpr (ES == 4) {
#pragma unroll
                                    for (int g = 0; g < 2; ++g)
                                        if (col + 4 * g < W)
                                            store(HS, row, col + 4 * g, u32x4{__float_as_uint(hr[4 * g]), __float_as_uint(hr[4 * g + 1]), __float_as_uint(hr[4 * g + 2]), __float_as_uint(hr[4 * g + 3])});
                                } else {
                                    u32x4 hi, lo;
#pragma unroll
                                    for (int i = 0; i < 4; ++i) {
                                        if constexpr (BWD) {
                                            hi[i] = __builtin_amdgcn_perm(__float_as_uint(hr[2 * i + 1]), __float_as_uint(hr[2 * i]), 0x07060302u);
                                            lo[i] = __builtin_amdgcn_perm(__float_as_uint(hr[2 * i + 1]), __float_as_uint(hr[2 * i]), 0x05040100u);
                                        } else hi[i] = pack_word<T>(hr[2 * i], hr[2 * i + 1]);
                                    }
                                    store(HS, row, col, hi);
                                    if constexpr (BWD) store(LO, row, col, lo);
                                }
                            }
                        }
                    }
                    leave(z, kd);
                    ++kd;
                }
            }
        }
        if (xat == n) lds_barrier();
    }

    // one direction of either axis
    template <int REV>
    __device__ __forceinline__ void walk(int dsel) {
        Unit chunk[UC];
        set_direction(dsel);
        vertical<REV>(REV ? (W * ES + 63) / 64 - 1 : 0, chunk);
        lds_barrier();
        set_direction(2 + dsel);
        horizontal<REV != 0>(chunk);
    }
};

template <typename T, int MODE, bool LOGITS, int NV>
__global__ void __launch_bounds__(NV == 1 ? 512 : 128, NV == 1 ? 2 : 1) lines_kernel(LinesArgs a) {
    extern __shared__ __attribute__((aligned(16))) char ln_lds[];
    typedef Lines<T, MODE, LOGITS, NV> K;
    constexpr int E = K::E;
    const FwdParams& p = a.p;
    const int plane = (int)xcd_contiguous_item(blockIdx.x, gridDim.x);
    const int b = plane / p.C, c = plane - b * p.C;
    K v(a, ln_lds);
    v.H = p.H; v.W = p.W; v.HW = p.H * p.W;
    v.plane = plane;
    v.bg = b * p.G + c / p.cpg;
    v.lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), dsel = w & 1;
    v.part = w >> 1;
    v.blk = v.lds0 + a.blk_off + w * (LN_BLOCK * NV);
    v.X = (const char*)((const T*)p.x + (size_t)plane * v.HW);
    v.at_end = p.W % E != 0 && v.bg == p.B * p.G - 1;
    v.top = (uint32_t)((v.bg == p.B * p.G - 1 ? 1 : 2) * v.HW * K::ES - 16);
    if (v.at_end && threadIdx.x < 24) {
        // the last granule of the plane, whose window would end beyond the tensor: its elements one by one
        const int dd = threadIdx.x / 6, t = threadIdx.x - dd * 6;
        const typename K::From f = v.from(dd);
        const char* q = t == 0 ? v.X : t == 1 ? f.lam : t == 2 ? f.u : f.w + (size_t)(t - 3) * v.HW * K::ES;
        const int col = (p.W - 1) / E * E;
        for (int e = 0; e < E; ++e) {
            typename K::bits_t bits = 0;
            if (col + e < p.W) bits = *((const typename K::bits_t*)q + (size_t)(p.H - 1) * p.W + col + e);
            lds_set<typename K::bits_t>(v.lds0 + a.tail_off + threadIdx.x * 16 + e * K::ES, bits);
        }
    }
    if (v.at_end) __syncthreads();
    const int rev = K::BWD ? !dsel : dsel;
    v.fv = v.from(dsel); v.fh = v.from(2 + dsel);
    if (rev) v.template walk<1>(dsel);
    else v.template walk<0>(dsel);
    lds_barrier();
    const float* const tile = (const float*)ln_lds;
    T* const Y = (T*)p.y + (size_t)plane * v.HW;
    const int gpr = (p.W + E - 1) / E;
    const int rows = (int)blockDim.x / gpr, cols = (int)blockDim.x - rows * gpr;      // from one of a thread's granules to the next
    int row = (int)threadIdx.x / gpr, g = (int)threadIdx.x - row * gpr;
    for (; row < p.H; row += rows, g += cols) {
        if (g >= gpr) { g -= gpr; if (++row >= p.H) break; }
        const int col = g * E;
        float t[E];
#pragma unroll
        for (int i = 0; i < E / 4; ++i) {
            const float4 f = *(const float4*)(tile + row * a.pitch + col + 4 * i);
            t[4 * i] = f.x; t[4 * i + 1] = f.y; t[4 * i + 2] = f.z; t[4 * i + 3] = f.w;
        }
        u32x4 o;
        if constexpr (K::ES == 4) o = u32x4{__float_as_uint(t[0]), __float_as_uint(t[1]), __float_as_uint(t[2]), __float_as_uint(t[3])};
        else {
#pragma unroll
            for (int i = 0; i < 4; ++i) o[i] = pack_word<T>(t[2 * i], t[2 * i + 1]);
        }
        v.store((char*)Y, row, col, o);
    }
}

template <typename T, int MODE, bool LOGITS>
hipError_t launch_lines_one(const LinesArgs& a, int nv, int threads, size_t lds, hipStream_t s) {
    const dim3 grid((unsigned)((size_t)a.p.B * a.p.C)), block(threads);
    void (*k)(LinesArgs) = nv == 1 ? lines_kernel<T, MODE, LOGITS, 1> : lines_kernel<T, MODE, LOGITS, 2>;
    const hipError_t e = allow_dynamic_lds((const void*)k, 160 * 1024);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, grid, block, lds, s, a);
    return hipGetLastError();
}
template <typename T>
hipError_t launch_lines_type(const LinesArgs& a, bool reverse, int nv, int threads, size_t lds, hipStream_t s) {
    if (reverse) return a.p.logits ? launch_lines_one<T, LN_BWD, true>(a, nv, threads, lds, s) : launch_lines_one<T, LN_BWD, false>(a, nv, threads, lds, s);
    if (a.p.hs) return a.p.logits ? launch_lines_one<T, LN_SAVE, true>(a, nv, threads, lds, s) : launch_lines_one<T, LN_SAVE, false>(a, nv, threads, lds, s);
    return a.p.logits ? launch_lines_one<T, LN_FWD, true>(a, nv, threads, lds, s) : launch_lines_one<T, LN_FWD, false>(a, nv, threads, lds, s);
}

}  // namespace
}  // namespace gspn
