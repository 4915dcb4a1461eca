// Scan kernel for maps of any height and width: odd sides, rows that start at any element.  Lines of up to 768 positions in fp32
// storage and 1280 in 16-bit storage (1072 with logits): a chunk of eight lines is at most two granules per loading thread.
// 16-bit forward calls whose merged output the line-by-line kernels sum in fp32 on chip keep the fp32 tile: they need room in the 160 KB
// for the tile (4 bytes per position) and a chunk of eight lines of either axis in one direction (10 bytes per position and line, 16 with
// logits, and the slots between granules), which maps of 435x67, 325x101 and 190x190 no longer have (with logits 386x67, 297x101 and
// 184x184): those run line by line, up to the 40 500 pixels that fit there (593x67, 397x101, 201x201).
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
// Where the LDS holds two chunks of a direction, the scan of one runs beside the finishing of the chunk before and the staging
// of the one after, with one barrier per chunk (move_ahead, the usual form of calls of up to 256 planes; the turns before took as long
// as the scan itself: 256 planes 80x68 in bf16 32 -> 26 us).  Where several workgroups share a CU they hide each other's turns and one
// chunk does (move_in_turn: 768 planes 50x83 and 1024 planes 64x168 in fp32, 288 planes 64x64 with logits), and one has to do where the
// tile leaves no room for a second that is as long (512 planes 100x167).  What these calls gained at the same time came from addresses
// as running sums, operands unpacked a line ahead and stores behind the next requests.
//
// What bounds it, kernel times on buffers in turn.  With many planes the L1s: 1024 planes 64x168 in fp32 162 us for 1.06 GB of requests,
// 6.5 TB/s, the chip's rate of pulling lines into its L1s; the LDS index unit is active in 36 % of a CU's busy cycles (45 % of them
// bank conflicts), the vector ALUs issue in 6 %.  With few planes the chain of the scanning wave (some 180 clocks per line) and the latency
// of a chunk's requests: 256 planes 80x68 in bf16 26 us, 148 lines each.  Neither where one workgroup per CU takes turns: 2 x 256
// channels 100x167 in bf16 134 us, with logits 174, of which the scans' chains are a quarter (267 lines a plane, two planes per CU);
// with logits the chunks are 8 and 16 lines, 168 and 200 granules for 448 loading threads a direction, so that about half of the
// loading waves stand by while the others stage a softmax per element, and scan and loads wait for each other.  A 16-bit request at an
// odd element costs the address unit four times an aligned one (64 clocks per wave against 16).
#pragma once
#include "gspn_unaligned.hpp"

namespace gspn {

constexpr int RG_FWD = 0, RG_SAVE = 1, RG_BWD = 2;
constexpr int RG_ROUNDS = 2;     // granules of a chunk per loading thread, at most
constexpr int RG_SUB = 8;        // scan steps between two meetings of the waves = positions a part shares with each neighbour

struct RaggedArgs {
    FwdParams p;
    void* hs_lo;                 // reverse sweep in 16-bit storage: low halves of e (high halves: p.hs), which stays fp32 between the passes; null: e is rounded
    int nd;                      // directions of an axis walked at once (1 or 2)
    int tile;                    // 1: merged output in an LDS tile; 0: in global memory
    int nbuf;                    // chunks of a direction in LDS: 2 (scan, load and finish work on neighbouring chunks at once) or 1 (in turn)
    int tile_pitch, tile_off;    // floats per row, byte offset in LDS
    int K[2], parts[2], own[2], pitch[2], pitch2[2];     // per axis (0 vertical, 1 horizontal): lines per chunk, waves per line, positions a wave owns, LDS slots per line (of {lam*x, w0, w1}; of tap 2)
    int w2_off[2], edge_off[2];               // byte offsets in LDS: tap 2 (16-bit weights), edge lines
};

namespace {

// One pass over the plane: one direction, or both directions of an axis at once.
template <typename T, int MODE, bool LOGITS, int NV, bool TILE, bool HORZ>
struct RaggedPass {
    static constexpr int E = 16 / (int)sizeof(T);
    static constexpr bool BWD = MODE == RG_BWD;
    static constexpr bool WIDE = LOGITS || sizeof(T) == 4;        // weights in LDS as fp32
    static constexpr int SB = WIDE ? 16 : 8;                      // bytes of {lam*x, w0, w1[, w2]} per position

    const RaggedArgs& a;
    char* lds;
    uint32_t lds0;               // LDS address of `lds`
    int H, W, HW, S, L, K, pitch, pitch2;
    int tid, nthr;               // this thread among the loading threads of its direction
    int part, parts;
    int d, rev;                  // direction slot; rev: this pass walks the lines from the last to the first
    int plane, bg;
    int dsel, dcount, nchunks;
    bool first;                  // global merge: y is overwritten
    // where a 16-byte window may start: byte offsets in [0, top] from the tensors' pointers here, which lie a plane before this
    // one where there is one (a window may reach into the neighbouring planes, not beyond the ends of the tensor)
    bool at_ends;                // a window of this plane can meet an end of the tensor
    int top;
    const char *X, *LAM, *U, *W0, *W1, *W2;
    char *Y, *HS, *LO;           // (these at the plane itself)
    float* edge;

    int bufA, bufW2;             // bytes from a chunk's place in LDS to the next one's
    uint32_t stA, stW2;          // LDS addresses of this direction's place for the first chunk
    __device__ __forceinline__ int buf(int k) const { return a.nbuf == 2 ? k & 1 : 0; }

    struct Regs { u32x4 x, l, u, w0, w1, w2, y; };       // a granule: x, lam, weights of a coming chunk; u and y of the one to finish

    __device__ __forceinline__ RaggedPass(const RaggedArgs& args, char* l) : a(args), lds(l) {
        lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    }

    // slot of a position of a line: a vertical scan's line has one slot of padding per granule, which spreads the banks of
    // lanes a granule apart
    static __device__ __forceinline__ int line_slot(int pos) { return HORZ ? pos : pos + pos / E; }

    // This thread's granule of every chunk: the same lines of the chunk (vertical: one, horizontal: E) and the same positions,
    // so a chunk's addresses are the first one's plus a multiple of a uniform step.
    struct Gran {
        int t;                   // first line of the chunk it holds; beyond the chunk where the thread has none
        int col, row;            // of chunk 0
        int off;                 // bytes from the tensors' pointers in chunk 0
        uint32_t slot, slot2;    // LDS addresses of its element 0 in buffer 0
        uint32_t tile;           // ... of its place in the output tile in chunk 0
    };
    __device__ __forceinline__ int col_step() const { return HORZ ? (rev ? -K : K) : 0; }
    __device__ __forceinline__ int row_step() const { return HORZ ? 0 : (rev ? -K : K); }
    __device__ __forceinline__ int off_step() const { return (HORZ ? K : K * W) * (rev ? -1 : 1) * (int)sizeof(T); }
    __device__ __forceinline__ int slot_step() const { return HORZ ? (rev ? -pitch : pitch) * SB : SB; }        // to the next element
    __device__ __forceinline__ int slot2_step() const { return HORZ ? (rev ? -pitch2 : pitch2) * 2 : 2; }
    __device__ __forceinline__ int granules() const { return HORZ ? (K / E) * H : K * ((W + E - 1) / E); }
    __device__ __forceinline__ Gran place(int r) const {
        Gran g;
        const int per = HORZ ? K / E : (W + E - 1) / E, last = granules() - 1;
        const int want = tid + r * nthr, q = min(want, last);       // a thread without a granule requests the last one's
        const int major = q / per, minor = (q - major * per) * E;
        if constexpr (HORZ) {
            g.row = major;
            g.col = rev ? S - minor - E : minor;                    // S: the width in whole granules
            g.t = minor;
            const int t0 = minor + (rev ? E - 1 : 0);
            g.slot = stA + (t0 * pitch + g.row) * SB;
            g.slot2 = stW2 + (t0 * pitch2 + g.row) * 2;
        } else {
            g.col = minor;
            g.row = rev ? S - 1 - major : major;
            g.t = major;
            g.slot = stA + (major * pitch + line_slot(g.col)) * SB;
            g.slot2 = stW2 + (major * pitch2 + g.col) * 2;
        }
        g.off = (g.row * W + g.col) * (int)sizeof(T);
        g.tile = lds0 + a.tile_off + (g.row * a.tile_pitch + g.col) * 4;
        if (want > last) g.t = 1 << 29;
        return g;
    }
    // is the granule of chunk k inside the scan?  (chunks -1 and those beyond the last: none is)
    __device__ __forceinline__ bool live(const Gran& g, int k) const { return g.t + k * K < S; }
    __device__ __forceinline__ int clamped(int off) const { return min(max(off, 0), top); }
    // reverse sweep: a line takes the weights of the line swept before it
    __device__ __forceinline__ int wshift() const { return BWD ? (rev ? 1 : -1) * (HORZ ? 1 : W) : 0; }

    // No request hangs on a branch, so that the waits count them; what lies outside the scan is read from some place of the tensor.
    __device__ __forceinline__ void load(int k, const Gran& g, Regs& q) const {
        const int off = g.off + base_off() + k * off_step();
        const uint32_t o = (uint32_t)clamped(off), ow = BWD ? (uint32_t)clamped(off + wshift() * (int)sizeof(T)) : o;
        q.x = rg_load((const T*)(X + o));
        q.l = rg_load((const T*)(LAM + o));
        q.w0 = rg_load((const T*)(W0 + ow));
        q.w1 = rg_load((const T*)(W1 + ow));
        q.w2 = rg_load((const T*)(W2 + ow));
    }
    // what finish() of the chunk needs
    __device__ __forceinline__ void load_late(int k, const Gran& g, Regs& q) const {
        const uint32_t o = (uint32_t)clamped(g.off + base_off() + k * off_step());
        q.u = rg_load((const T*)(U + o));
        if constexpr (!TILE) q.y = rg_load((const T*)(Y + ((int)o - base_off())));      // (not used by the first direction)
    }
    __device__ __forceinline__ int base_off() const { return bg == 0 ? 0 : HW * (int)sizeof(T); }

    // Bit e: the weights of element e are never read: the first line of the scan, of a stretch (by the line the weights belong
    // to), and, in a reverse sweep, the line after the last.
    __device__ __forceinline__ uint32_t dead_elements(const Gran& g, int k) const {
        const int col = g.col + k * col_step(), row = g.row + k * row_step();
        const int S1 = (HORZ ? W : H) - 1, drev = d & 1, kc = a.p.kchunk;
        int wl = (HORZ ? col : row) + (BWD ? (rev ? 1 : -1) : 0);          // line the weights of element 0 belong to
        uint32_t dead = 0;
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
            const int n = min(E, W - col);
            dead |= ~((1u << n) - 1u) & ((1u << E) - 1u);                  // beyond the row: a scan from the right starts there, with 0
        } else {
            const bool z = (BWD && (wl < 0 || wl > S1)) || starts_stretch(drev ? S1 - wl : wl, S, drev, kc);
            dead = z ? (1u << E) - 1 : 0u;
        }
        return dead;
    }

    // registers of the chunk -> LDS
    __device__ __forceinline__ void stage(int k, const Gran& g, const Regs& in) const {
        if (!live(g, k)) return;
        __builtin_amdgcn_sched_barrier(0);
        u32x4 x = in.x, l = in.l, w0 = in.w0, w1 = in.w1, w2 = in.w2;
        const int col = HORZ ? g.col + k * col_step() : g.col;
        if (at_ends) {                               // first / last granule of a tensor
            const int off = g.off + base_off() + k * off_step(), offw = off + wshift() * (int)sizeof(T);
            const int sh = (off - clamped(off)) / (int)sizeof(T), shw = (offw - clamped(offw)) / (int)sizeof(T);
            if (__any(sh != 0 || shw != 0)) {
                x = rg_realign<T>(x, sh); l = rg_realign<T>(l, sh);
                w0 = rg_realign<T>(w0, shw); w1 = rg_realign<T>(w1, shw); w2 = rg_realign<T>(w2, shw);
            }
        }
        // the first chunk holds the first line of the scan (and, from the right, what lies beyond the row)
        uint32_t dead = 0;
        if (k == 0 || a.p.kchunk > 0) dead = dead_elements(g, k);
        float av[E];
#pragma unroll
        for (int e = 0; e < E; ++e) av[e] = rg_elem<T>(l, e) * rg_elem<T>(x, e);
        if (HORZ && k == 0) {
#pragma unroll
            for (int e = 0; e < E; ++e) av[e] = col + e < W ? av[e] : 0.f;
        }
        const uint32_t s0 = g.slot + buf(k) * bufA;
        const int ss = slot_step();
        if constexpr (WIDE) {
            const bool row_first = g.row == 0, row_last = g.row == H - 1;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if constexpr (sizeof(T) == 2) __builtin_amdgcn_sched_barrier(0);        // element by element: registers
                const bool o0 = HORZ ? row_first : (e == 0 && col == 0);
                const bool o2 = HORZ ? row_last : (col + e == W - 1);
                float f0 = rg_elem<T>(w0, e), f1 = rg_elem<T>(w1, e), f2 = rg_elem<T>(w2, e);
                if constexpr (LOGITS) softmax3(f0, f1, f2, o0, o2);
                const bool dd = (dead >> e) & 1u;
                f0 = (dd || o0) ? 0.f : f0; f1 = dd ? 0.f : f1; f2 = (dd || o2) ? 0.f : f2;
                lds_set<u32x4>(s0 + e * ss, u32x4{__float_as_uint(av[e]), __float_as_uint(f0), __float_as_uint(f1), __float_as_uint(f2)});
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
                if (g.row == 0) w0 = u32x4{0, 0, 0, 0};
                if (g.row == H - 1) w2 = u32x4{0, 0, 0, 0};
            } else {
                if (col == 0) w0[0] &= 0xffff0000u;
                const int el = W - 1 - col;
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
            const uint32_t s2 = g.slot2 + buf(k) * bufW2;
            if constexpr (HORZ) {
                const int ss2 = slot2_step();
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    lds_set<u32x2>(s0 + e * ss, u32x2{__float_as_uint(av[e]), w01[e]});
                    lds_set<uint16_t>(s2 + e * ss2, (uint16_t)((e & 1) ? w2[e >> 1] >> 16 : w2[e >> 1]));
                }
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) lds_set<u32x2>(s0 + e * SB, u32x2{__float_as_uint(av[e]), w01[e]});
                lds_set<u32x4>(s2, w2);
            }
        }
    }

    // h of the chunk from LDS: the merged output in LDS, and what goes to global memory -- h_save (e of the reverse sweep), y
    // merged there -- in registers for store().  The two are apart because a wait for a request counts the stores issued
    // behind it: store() comes when the next chunk's requests have been waited for.
    struct Out { u32x4 v, lw, y; };
    __device__ __forceinline__ void finish(int k, const Gran& g, const Regs& in, Out& out) const {
        if (!live(g, k)) return;
        __builtin_amdgcn_sched_barrier(0);
        u32x4 u = in.u, yv = in.y;
        if (at_ends) {
            const int off = g.off + base_off() + k * off_step(), sh = (off - clamped(off)) / (int)sizeof(T);
            if (__any(sh != 0)) {
                u = rg_realign<T>(u, sh);
                if constexpr (!TILE) yv = rg_realign<T>(yv, sh);
            }
        }
        const uint32_t s0 = g.slot + buf(k) * bufA;
        const int ss = slot_step();
        float h[E], y[E];
#pragma unroll
        for (int e = 0; e < E; ++e) h[e] = lds_get<float>(s0 + e * (HORZ ? ss : SB));
#pragma unroll
        for (int e = 0; e < E; ++e) y[e] = rg_elem<T>(u, e) * h[e];
        if constexpr (MODE != RG_FWD) {
            if constexpr (sizeof(T) == 4) {
                out.v = u32x4{__float_as_uint(h[0]), __float_as_uint(h[1]), __float_as_uint(h[2]), __float_as_uint(h[3])};
            } else if (BWD && a.hs_lo) {                 // e as two 16-bit halves of its fp32 word
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    out.v[i] = __builtin_amdgcn_perm(__float_as_uint(h[2 * i + 1]), __float_as_uint(h[2 * i]), 0x07060302u);
                    out.lw[i] = __builtin_amdgcn_perm(__float_as_uint(h[2 * i + 1]), __float_as_uint(h[2 * i]), 0x05040100u);
                }
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) out.v[i] = pack_word<T>(h[2 * i], h[2 * i + 1]);
            }
        }
        if constexpr (TILE) {
            const uint32_t tp = g.tile + (uint32_t)(k * (HORZ ? col_step() : row_step() * a.tile_pitch) * 4);
            // the tile's rows are whole granules: what lies beyond the image row is never read
            typedef float f32x4 __attribute__((ext_vector_type(4)));
            f32x4 t[E / 4];
#pragma unroll
            for (int i = 0; i < E / 4; ++i) t[i] = lds_get<f32x4>(tp + 16 * i);
#pragma unroll
            for (int i = 0; i < E / 4; ++i) lds_set<f32x4>(tp + 16 * i, f32x4{t[i][0] + y[4 * i], t[i][1] + y[4 * i + 1], t[i][2] + y[4 * i + 2], t[i][3] + y[4 * i + 3]});
        } else {
            if (!first) {
#pragma unroll
                for (int e = 0; e < E; ++e) y[e] += rg_elem<T>(yv, e);
            }
            if constexpr (sizeof(T) == 4) out.y = u32x4{__float_as_uint(y[0]), __float_as_uint(y[1]), __float_as_uint(y[2]), __float_as_uint(y[3])};
            else {
#pragma unroll
                for (int i = 0; i < 4; ++i) out.y[i] = pack_word<T>(y[2 * i], y[2 * i + 1]);
            }
        }
    }
    __device__ __forceinline__ void store(int k, const Gran& g, const Out& out) const {
        if constexpr (MODE == RG_FWD && TILE) return;
        if (!live(g, k)) return;
        const int n = W - (HORZ ? g.col + k * col_step() : g.col);           // elements inside the row
        const uint32_t off = (uint32_t)(g.off + k * off_step());
        if (n >= E) {
            if constexpr (MODE != RG_FWD) rg_store((T*)(HS + off), out.v);
            if constexpr (BWD && sizeof(T) == 2) { if (a.hs_lo) rg_store((T*)(LO + off), out.lw); }
            if constexpr (!TILE) rg_store((T*)(Y + off), out.y);
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (e < n) {
                    if constexpr (MODE != RG_FWD) rg_store_bits((T*)(HS + off) + e, rg_bits<T>(out.v, e));
                    if constexpr (BWD && sizeof(T) == 2) { if (a.hs_lo) rg_store_bits((T*)(LO + off) + e, rg_bits<T>(out.lw, e)); }
                    if constexpr (!TILE) rg_store_bits((T*)(Y + off) + e, rg_bits<T>(out.y, e));
                }
        }
    }

    // The scan of nsub * 8 lines of the chunk by a scanning wave; h: state of this lane's positions.  The LDS reads of HL
    // lines are issued while the HL lines before them are computed: one wave per SIMD scans, and nothing else hides their
    // latency.  MEET: the line is shared with other waves, which exchange the last line every 8 steps (a line's h then goes
    // to LDS after the meeting, when no neighbour reads lam*x there any more).
    template <bool MEET, bool LOCAL>
    __device__ __forceinline__ void scan(int k, int nsub, float (&h)[NV], int& parity, int& until) const {
        constexpr int HL = WIDE ? (NV == 1 ? 4 : NV <= 3 ? 2 : 1) : (NV <= 2 ? 4 : 2);      // what the registers hold twice
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
        uint32_t ra = stA + buf(k) * bufA + (uint32_t)(first_slot * SB), rw = stW2 + buf(k) * bufW2 + (uint32_t)(pc * 2), rh = ra;
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
        // A line's operands in fp32, unpacked in three parts while the line before it is computed: an instruction that waits for
        // the one before it costs a lone wave twice its issue, and the chain of a line alone leaves every second slot empty.
        struct Taps { float a[NV], w0[NV], w1[NV], w2[NV], lt, rt; };
        auto unpack = [&](const Lines& q, int j, Taps& t, int what) {
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                if constexpr (WIDE) {
                    if (what == 0) { t.a[v] = q.a[j][v]; t.w1[v] = __uint_as_float(q.w[j][v][1]); }
                    if (what == 1) t.w0[v] = __uint_as_float(q.w[j][v][0]);
                    if (what == 2) t.w2[v] = __uint_as_float(q.w[j][v][2]);
                } else {
                    if (what == 0) { t.a[v] = q.a[j][v]; t.w1[v] = word_hi<T>(q.w[j][v][0]); }
                    if (what == 1) t.w0[v] = word_lo<T>(q.w[j][v][0]);
                    if (what == 2) t.w2[v] = NV % 2 ? word_lo<T>(q.w2[j][v % NW2]) : (v & 1) ? word_hi<T>(q.w2[j][v / 2]) : word_lo<T>(q.w2[j][v / 2]);
                }
            }
            if constexpr (BWD) {
                // the taps that reach this lane's positions from its neighbours' (a lane's positions beyond the line come after
                // those inside, or are all of its positions: their taps are read as 0)
                if (what == 1) {
#pragma unroll
                    for (int v = 0; v < NV; ++v) t.w0[v] = valid[v] ? t.w0[v] : 0.f;
                    t.rt = from_lane_above(t.w0[0]);
                }
                if (what == 2) t.lt = from_lane_below(valid[NV - 1] ? t.w2[NV - 1] : 0.f);
            }
        };
        float hout[NV];                                           // h of the line, for LDS
        auto line = [&](const Taps& t, const Lines& qn, int jn, Taps& tn) {
            // a stretch starts with the next line: nothing is carried into it, whatever the state holds (the weights there
            // are 0 already); a mask, not a branch: a wave alone on its SIMD pays some 16 clocks for each
            bool keep = true;
            if constexpr (LOCAL) {
                keep = --until != 0;
                until = keep ? until : a.p.kchunk;
            }
            // one chain of FMAs per position in the line-by-line kernels' order -- own tap, the neighbour before, the neighbour
            // after -- so that the states are theirs bit for bit (products of the reverse sweep summed in pairs instead: glam of
            // fp32 maps 9 % further from 64 bits in the mean, up to 2.4 times)
            float hn[NV];
            const float lin = from_lane_below(h[NV - 1]), rin = from_lane_above(h[0]);
#pragma unroll
            for (int v = 0; v < NV; ++v) hn[v] = fmaf(t.w1[v], h[v], t.a[v]);
            __builtin_amdgcn_sched_barrier(0);
            unpack(qn, jn, tn, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const float w = BWD ? (v == 0 ? t.lt : t.w2[v > 0 ? v - 1 : 0]) : t.w0[v];
                hn[v] = fmaf(w, v == 0 ? lin : h[v > 0 ? v - 1 : 0], hn[v]);
            }
            __builtin_amdgcn_sched_barrier(0);
            unpack(qn, jn, tn, 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const float w = BWD ? (v == NV - 1 ? t.rt : t.w0[v < NV - 1 ? v + 1 : v]) : t.w2[v];
                hn[v] = fmaf(w, v == NV - 1 ? rin : h[v < NV - 1 ? v + 1 : v], hn[v]);
            }
            __builtin_amdgcn_sched_barrier(0);
            unpack(qn, jn, tn, 2);
            __builtin_amdgcn_sched_barrier(0);
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
        Taps taps[2];
        read(buf[0]);
        read(buf[1]);
#pragma unroll
        for (int i = 0; i < 3; ++i) unpack(buf[0], 0, taps[0], i);
        for (int s = 0; s < nsub; ++s) {
            float hb[MEET ? RG_SUB : 1][NV];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                static_assert(NB % 2 == 0, "the two line sets alternate");
#pragma unroll
                for (int j = 0; j < HL; ++j) {
                    // (after the last line of the chunk what is unpacked next is never used)
                    constexpr int odd = HL & 1;
                    const int at = odd ? (i * HL + j) & 1 : j & 1;
                    line(taps[at], buf[(j + 1 < HL ? i : i + 1) & 1], (j + 1) % HL, taps[at ^ 1]);
                    if constexpr (MEET) {
#pragma unroll
                        for (int v = 0; v < NV; ++v) hb[i * HL + j][v] = hout[v];
                    } else {
                        put(hout);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                if (i + 2 < NB || s + 1 < nsub) read(buf[i & 1]);
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
        const size_t back = bg == 0 ? 0 : (size_t)HW;             // the neighbouring plane a window may reach into
        X = (const char*)((const T*)p.x + pc - back);
        LAM = (const char*)((const T*)p.lam + slot_c + pc - back);
        U = (const char*)((const T*)p.u + slot_c + pc - back);
        W0 = (const char*)((const T*)p.w + slot_w + (size_t)bg * 3 * HW - back);
        W1 = W0 + (size_t)HW * sizeof(T);
        W2 = W1 + (size_t)HW * sizeof(T);
        Y = (char*)((T*)p.y + pc);
        HS = MODE != RG_FWD ? (char*)((T*)p.hs + (size_t)d * planes * HW + pc) : nullptr;
        LO = (BWD && sizeof(T) == 2) ? (char*)((T*)a.hs_lo + (size_t)d * planes * HW + pc) : nullptr;
        at_ends = bg == 0 || bg == (int)groups - 1;
        top = ((int)back + (bg == (int)groups - 1 ? HW : 2 * HW) - E) * (int)sizeof(T);
        bufA = a.nd * K * pitch * SB; bufW2 = a.nd * K * pitch2 * 2;
        stA = lds0 + dsel * K * pitch * SB;
        stW2 = lds0 + a.w2_off[ax] + dsel * K * pitch2 * 2;
        edge = (float*)(lds + a.edge_off[ax]) + dsel * 2 * pitch2;

        nchunks = (S + K - 1) / K;
        if (part < parts) {
            __builtin_amdgcn_s_setprio(3);       // the chain the others wait for (a few per cent either way: 2048 planes 25x31 33.7 -> 32.4 us, 768 of 50x83 63.3 -> 64.7)
            if (a.p.kchunk > 0) scan_all<true>();
            else scan_all<false>();
            __builtin_amdgcn_s_setprio(0);
        } else {
            if (__builtin_amdgcn_readfirstlane(tid) >= granules()) { stand_by(); return; }      // (the same for the whole wave)
            const bool two = granules() > nthr;                     // granules of a chunk per thread
            if (a.nbuf == 2) {
                if (two) move_ahead<2>(); else move_ahead<1>();
            } else {
                if (two) move_in_turn<2>(); else move_in_turn<1>();
            }
        }
    }

    __device__ __forceinline__ int subs(int k) const { return (min(K, S - k * K) + RG_SUB - 1) / RG_SUB; }
    // both directions add to the same rows / columns of the tile while their chunks cross
    __device__ __forceinline__ bool cross(int k) const { return dcount == 2 && 2 * (k + 1) * K > S && 2 * k * K < S; }

    // A scanning wave's part of a pass: the barriers below are the ones of move_ahead / move_in_turn.
    template <bool LOCAL>
    __device__ __forceinline__ void scan_all() {
        float h[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) h[v] = 0.f;
        int parity = 0;
        // scan steps to the next stretch: cuts lie before image lines 0, kchunk, 2 * kchunk, ..
        int until = 1 << 30;
        if (LOCAL) until = rev && S % a.p.kchunk ? S % a.p.kchunk : a.p.kchunk;
        const bool ahead = a.nbuf == 2;
        lds_barrier();
        for (int k = 0; k < nchunks; ++k) {
            if (NV % 2 == 0 && parts > 1) scan<NV % 2 == 0, LOCAL>(k, subs(k), h, parity, until);      // (lines of one or three positions per lane are one wave's)
            else scan<false, LOCAL>(k, subs(k), h, parity, until);
            if (ahead) {
                if (k > 0 && cross(k - 1)) lds_barrier();
            } else {
                lds_barrier();
                if (cross(k)) lds_barrier();
            }
            lds_barrier();
        }
        if (ahead) {
            if (cross(nchunks - 1)) lds_barrier();
            lds_barrier();
        }
    }

    // A loading wave without a granule: the barriers of the others.
    __device__ __forceinline__ void stand_by() const {
        lds_barrier();
        for (int k = 0; k <= nchunks; ++k) {
            const int meetings = parts > 1 && k < nchunks ? subs(k) : 0;
            int n = a.nbuf == 2 ? meetings + (k > 0 && cross(k - 1) ? 2 : 1) : k < nchunks ? meetings + (cross(k) ? 3 : 2) : 0;
            for (; n > 0; --n) lds_barrier();
        }
    }

    // A loading wave's part with two chunks in LDS: while chunk k is scanned, chunk k - 1 is finished, chunk k + 1 takes its
    // place and the requests of chunk k + 2 go out.  A thread reads and writes its own granules' places there, so nothing but
    // the end of the scan is waited for.  R: granules of a chunk per thread.
    template <int R>
    __device__ __forceinline__ void move_ahead() {
        Regs q[R];
        Gran g[R];
        Out out[R];
#pragma unroll
        for (int r = 0; r < R; ++r) g[r] = place(r);
#pragma unroll
        for (int r = 0; r < R; ++r) load(0, g[r], q[r]);
#pragma unroll
        for (int r = 0; r < R; ++r) stage(0, g[r], q[r]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < R; ++r) load(1, g[r], q[r]);
        lds_barrier();
        for (int k = 0; k <= nchunks; ++k) {
            const bool crossing = k > 0 && cross(k - 1);
            int meetings = parts > 1 && k < nchunks ? subs(k) : 0;
            if (crossing && dsel == 1) lds_barrier();
            if (k > 0) {
#pragma unroll
                for (int r = 0; r < R; ++r) finish(k - 1, g[r], q[r], out[r]);
            }
            if (crossing && dsel == 0) lds_barrier();
            if (meetings > 1) { lds_barrier(); --meetings; }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < R; ++r) load_late(k, g[r], q[r]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < R; ++r) stage(k + 1, g[r], q[r]);
            __builtin_amdgcn_sched_barrier(0);
            if (k > 0) {
#pragma unroll
                for (int r = 0; r < R; ++r) store(k - 1, g[r], out[r]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < R; ++r) load(k + 2, g[r], q[r]);
            __builtin_amdgcn_sched_barrier(0);
            for (; meetings > 0; --meetings) lds_barrier();
            lds_barrier();
        }
    }

    // ... and with one: scan and loads take turns
    template <int R>
    __device__ __forceinline__ void move_in_turn() {
        Regs q[R];
        Gran g[R];
        Out out[R];
#pragma unroll
        for (int r = 0; r < R; ++r) g[r] = place(r);
#pragma unroll
        for (int r = 0; r < R; ++r) load(0, g[r], q[r]);
#pragma unroll
        for (int r = 0; r < R; ++r) stage(0, g[r], q[r]);
        lds_barrier();
        for (int k = 0; k < nchunks; ++k) {
#pragma unroll
            for (int r = 0; r < R; ++r) load_late(k, g[r], q[r]);
#pragma unroll
            for (int r = 0; r < R; ++r) load(k + 1, g[r], q[r]);
            __builtin_amdgcn_sched_barrier(0);
            if (parts > 1) for (int s = subs(k); s > 0; --s) lds_barrier();
            lds_barrier();
            if (cross(k) && dsel == 1) lds_barrier();
#pragma unroll
            for (int r = 0; r < R; ++r) finish(k, g[r], q[r], out[r]);
            if (cross(k) && dsel == 0) lds_barrier();
#pragma unroll
            for (int r = 0; r < R; ++r) stage(k + 1, g[r], q[r]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < R; ++r) store(k, g[r], out[r]);
            lds_barrier();
        }
    }
};

template <typename T, int MODE, bool LOGITS, int NV, bool TILE>
__global__ void __launch_bounds__(1024) ragged_kernel(RaggedArgs a) {
    extern __shared__ __attribute__((aligned(16))) char rg_lds[];
    constexpr int E = 16 / (int)sizeof(T);
    const FwdParams& p = a.p;
    const int plane = (int)xcd_contiguous_item(blockIdx.x, gridDim.x);
    const int b = plane / p.C, c = plane - b * p.C;
    const int bg = b * p.G + c / p.cpg;
    float* tile = (float*)(rg_lds + a.tile_off);
    if constexpr (TILE) {
        for (int i = threadIdx.x; i < p.H * a.tile_pitch; i += blockDim.x) tile[i] = 0.f;
        // (visible after the first barrier of the first pass)
    }
    bool first = true;
    {
        RaggedPass<T, MODE, LOGITS, NV, TILE, false> v(a, rg_lds);
        v.plane = plane; v.bg = bg;
        const int m = p.mask & 3;
        if (m == 3 && a.nd == 2) { v.run(0, 2, first); first = false; }
        else
            for (int i = 0; i < 2; ++i)
                if ((m >> i) & 1) { v.run(i, 1, first); if constexpr (!TILE) __syncthreads(); first = false; }
    }
    {
        RaggedPass<T, MODE, LOGITS, NV, TILE, true> v(a, rg_lds);
        v.plane = plane; v.bg = bg;
        const int m = (p.mask >> 2) & 3;
        if (m == 3 && a.nd == 2) v.run(2, 2, first);
        else
            for (int i = 0; i < 2; ++i)
                if ((m >> i) & 1) { v.run(2 + i, 1, first); if constexpr (!TILE) __syncthreads(); first = false; }
    }
    if constexpr (TILE) {
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

template <typename T, int MODE, bool LOGITS, bool TILE>
hipError_t launch_ragged_one(const RaggedArgs& a, int threads, int nv, size_t lds, hipStream_t s) {
    const dim3 grid((unsigned)((size_t)a.p.B * a.p.C)), block(threads);
    void (*k)(RaggedArgs) = nv == 2 ? ragged_kernel<T, MODE, LOGITS, 2, TILE> : nv == 3 ? ragged_kernel<T, MODE, LOGITS, 3, TILE> : ragged_kernel<T, MODE, LOGITS, 4, TILE>;
    if constexpr (TILE) { if (nv == 1) k = ragged_kernel<T, MODE, LOGITS, 1, TILE>; }
    else if (nv == 1) return hipErrorInvalidValue;              // (lines of up to 64 positions: the tile of a plane always fits)
    const hipError_t e = allow_dynamic_lds((const void*)k, 160 * 1024);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, grid, block, lds, s, a);
    return hipGetLastError();
}

template <typename T, bool TILE>
hipError_t launch_ragged_type(const RaggedArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s) {
    if (reverse) return a.p.logits ? launch_ragged_one<T, RG_BWD, true, TILE>(a, threads, nv, lds, s) : launch_ragged_one<T, RG_BWD, false, TILE>(a, threads, nv, lds, s);
    if (a.p.hs) return a.p.logits ? launch_ragged_one<T, RG_SAVE, true, TILE>(a, threads, nv, lds, s) : launch_ragged_one<T, RG_SAVE, false, TILE>(a, threads, nv, lds, s);
    return a.p.logits ? launch_ragged_one<T, RG_FWD, true, TILE>(a, threads, nv, lds, s) : launch_ragged_one<T, RG_FWD, false, TILE>(a, threads, nv, lds, s);
}

}  // namespace
}  // namespace gspn
