// Scan kernel for calls of few planes: a workgroup per (plane, direction, range of lines).
//
// The other kernels give a plane to one workgroup, so a call of fewer planes than the chip has CUs leaves the rest of them idle and walks
// the directions one axis after the other.  Here every direction of every plane is a work item of its own, and so is every stretch of
// GSPN-local; each stores its states h in fp32 (in fp32 storage: as h_save; the reverse sweep: e, in 16-bit storage as two halves in the
// buffers of glam and gu; else in a workspace of the caller's), and a second launch forms y = sum of u * h from them, the sum over the
// directions in fp32 and in direction order (combine_kernel).  It costs 8 bytes per pixel and direction across the memory system,
// half of it where the call stores the states anyway.
//
// A workgroup walks its lines in chunks of K that pass through LDS:
//   load    a loading thread holds one or two granules (16 B of an image row: x, lam and the three weights) of the coming chunks in
//           registers.  16-byte requests at element alignment;
//   stage   lam*x and the weights (taps outside the line and lines without a predecessor zeroed, logits normalised in fp32) go to LDS,
//           a horizontal scan's granules across eight (four) lines, which is where the horizontal directions are turned;
//   scan    one wave walks lines of up to 256 positions, 1, 2 or 4 per lane; longer lines are shared between waves that cover K positions
//           of their neighbours on either side beside their own, so that the K lines of a chunk need nothing from outside;
//   finish  the thread that loaded a granule reads its h back and stores it.
// Where the LDS holds two chunks, the scan of one runs beside the finishing of the one before and the staging of the one after.
//
// What bounds it (clocks read in the kernel): the chain of the scanning wave, some 70, 100 and 165 clocks per line with 1, 2 and 4 positions
// per lane (104, 148 and 255 with the two taps across lanes as moves of their own, a select per position and lam*x beside the weights
// position by position, which costs ten LDS accesses per line and lane at four positions and here five), and, at four, the LDS: 28 (16-bit
// weights) or 40 bytes per position and line.  1 x 32 channels 128x128 fp32 with stretches of 32, training step, 76 -> 49 us; 64 planes
// 256x256 bf16 123 -> 67 us, of which the merge some 8.
#pragma once
#include "gspn_line_step.hpp"
#include "gspn_unaligned.hpp"

namespace gspn {

constexpr int AP_FWD = 0, AP_SAVE = 1, AP_BWD = 2;       // (fp32 storage: AP_SAVE in forward calls, the states of a call without h_save in the workspace)
constexpr int AP_ROUNDS = 2;     // granules of a chunk per loading thread, at most
constexpr int AP_SUB = 8;        // chunks are multiples of this many lines

// LDS of a line: blocks of NV positions, one per lane of the scanning wave, {lam*x[NV], w0[NV], w1[NV], w2[NV]} in fp32 (WIDE) or
// {lam*x[NV], {w0, w1}[NV], w2[NV]} with 16-bit weights, h in place of lam*x.  A lane's reads are a few of 8 or 16 bytes and the arrays
// of a block lie at constant offsets.  Block and padding (bytes per 8 positions) spread the banks: an odd number of 4 (8, 16) bytes
// from lane to lane for accesses of that size.  Four fp32 positions are 64 bytes, padded to 80 where that leaves the chunk its place.
__host__ __device__ constexpr int ap_block(bool wide, int nv, bool tight) { return wide ? (nv == 4 && !tight ? 80 : 16 * nv) : nv == 1 ? 12 : 10 * nv; }
__host__ __device__ constexpr int ap_pad(bool wide, int nv) { return nv == 4 ? 0 : wide ? 16 : 4; }

struct ApartArgs {
    FwdParams p;
    void* hs_lo;                     // reverse sweep in 16-bit storage: low halves of e (high halves: p.hs)
    float* part;                     // forward calls in 16-bit storage: states in fp32, [direction][plane][H][W]
    int range[2], nrange[2];         // per axis (0 vertical, 1 horizontal): lines of a range (a stretch of GSPN-local, else the map), ranges
    int nbuf;                        // chunks in LDS: 2 (scan, load and finish work on neighbouring chunks at once) or 1 (in turn)
    int K[2], parts[2], own[2];      // lines per chunk, waves per line, positions a wave owns
    int pitch[2], skew[2], chunk[2]; // bytes in LDS per line, beside that per E lines, per chunk
    int block;                       // bytes per block
    int tail[2];                     // of lines shared by several waves: bytes to the h of positions that two waves read, behind the blocks; else 0
    int edge_off[2], edge_len[2];    // byte offset in LDS and floats of the line that passes a chunk's last states between the waves
};

namespace {

// One direction of one plane, one range of its lines.
template <typename T, int MODE, bool LOGITS, int NV, bool HORZ>
struct ApartPass {
    static constexpr int E = 16 / (int)sizeof(T);
    static constexpr bool BWD = MODE == AP_BWD;
    static constexpr bool HSAVE = MODE != AP_FWD, PART = MODE != AP_BWD && sizeof(T) == 2;
    static constexpr bool WIDE = LOGITS || sizeof(T) == 4;        // weights in LDS as fp32

    const ApartArgs& a;
    char* lds;
    uint32_t lds0;               // LDS address of `lds`
    int H, W, HW, S, L, K, pitch, skew;
    int tid, nthr;               // this thread among the loading threads of its direction
    int part, parts;
    int d, rev;                  // direction; rev: this pass walks the lines from the last to the first
    int plane, bg;
    int lo, lines;               // range of lines of this pass: first image line, image lines
    int nchunks;
    // where a 16-byte window may start: byte offsets in [0, top] from the tensors' pointers here, which lie a plane before this
    // one where there is one (a window may reach into the neighbouring planes, not beyond the ends of the tensor)
    bool at_ends;                // a window of this plane can meet an end of the tensor
    int top;
    const char *X, *LAM, *W0, *W1, *W2;
    char *HS, *LO;               // (these at the plane itself)
    float* PT;
    float* edge;

    int next_buf;                // bytes from a chunk's place in LDS to the next one's
    __device__ __forceinline__ uint32_t buf(int k) const { return a.nbuf == 2 ? (k & 1) * next_buf : 0; }

    struct Regs { u32x4 x, l, w0, w1, w2; };             // a granule of a coming chunk

    __device__ __forceinline__ ApartPass(const ApartArgs& args, char* l) : a(args), lds(l) {
        lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds;
    }

    __device__ __forceinline__ int block_bytes() const { return NV == 4 && WIDE ? a.block : ap_block(WIDE, NV, false); }
    // bytes from a line's place in LDS to a position's (to its lam*x)
    __device__ __forceinline__ int place_of(int pos) const { return pos / NV * block_bytes() + pos % NV * 4 + pos / 8 * ap_pad(WIDE, NV); }
    // ... to its h: in place of lam*x, unless a neighbouring wave scans the position too and still reads that
    __device__ __forceinline__ bool h_apart(int pos) const {
        if (NV < 4 || parts == 1) return false;
        const int w = pos % a.own[HORZ];
        return w < K || w >= a.own[HORZ] - K;
    }
    __device__ __forceinline__ int h_of(int pos) const {
        if (!h_apart(pos)) return place_of(pos);
        const int own = a.own[HORZ], q = pos / own, w = pos - q * own;
        return a.tail[HORZ] + (q * 2 * K + (w < K ? w : w - own + 2 * K)) * 4;
    }
    // ... and from its lam*x to its other values: {w0, w1, w2} or {{w0, w1}, w2}
    static constexpr int ARR = 4 * NV;
    // This thread's granule of every chunk: the same lines of the chunk (vertical: one, horizontal: E) and the same positions,
    // so a chunk's addresses are the first one's plus a multiple of a uniform step.
    struct Gran {
        int t;                   // first line of the chunk it holds; beyond the chunk where the thread has none
        int col, row;            // of chunk 0
        int off;                 // bytes from the tensors' pointers in chunk 0
        uint32_t slot, h;        // LDS addresses of its element 0 and its h in buffer 0
        int hstep;               // ... bytes from a block's h to the next one's (vertical)
    };
    __device__ __forceinline__ int col_step() const { return HORZ ? (rev ? -K : K) : 0; }
    __device__ __forceinline__ int row_step() const { return HORZ ? 0 : (rev ? -K : K); }
    __device__ __forceinline__ int off_step() const { return (HORZ ? K : K * W) * (rev ? -1 : 1) * (int)sizeof(T); }
    __device__ __forceinline__ int slot_step() const { return rev ? -pitch : pitch; }        // to the next element of a horizontal scan's granule
    __device__ __forceinline__ int granules() const { return HORZ ? (K / E) * H : K * ((W + E - 1) / E); }
    __device__ __forceinline__ Gran place(int r) const {
        Gran g;
        const int per = HORZ ? K / E : (W + E - 1) / E, last = granules() - 1;
        const int want = tid + r * nthr, q = min(want, last);       // a thread without a granule requests the last one's
        const int major = q / per, minor = (q - major * per) * E;
        if constexpr (HORZ) {
            g.row = major;
            g.col = lo + (rev ? S - minor - E : minor);             // S: the range in whole granules
            g.t = minor;
            const int t0 = minor + (rev ? E - 1 : 0);
            g.slot = lds0 + t0 * pitch + minor / E * skew + place_of(g.row);
            g.h = g.slot + h_of(g.row) - place_of(g.row);
        } else {
            g.col = minor;
            g.row = lo + (rev ? S - 1 - major : major);
            g.t = major;
            g.slot = lds0 + major * pitch + place_of(g.col);
            g.h = g.slot + h_of(g.col) - place_of(g.col);
            g.hstep = h_apart(g.col) ? 16 : block_bytes();
        }
        g.off = (g.row * W + g.col) * (int)sizeof(T);
        if (want > last) g.t = 1 << 29;
        return g;
    }
    // is the granule of chunk k inside the scan?  (chunks -1 and those beyond the last: none is)
    __device__ __forceinline__ bool live(const Gran& g, int k) const { return g.t + k * K < S; }
    __device__ __forceinline__ int clamped(int off) const { return min(max(off, 0), top); }
    // reverse sweep: a line takes the weights of the line swept before it
    __device__ __forceinline__ int wshift() const { return BWD ? (rev ? 1 : -1) * (HORZ ? 1 : W) : 0; }

    // No request hangs on a branch, so that the waits count them; what lies outside the scan is read from some place of the tensor.
    // (beyond the last chunk, its requests once more, from the caches)
    __device__ __forceinline__ void load(int k, const Gran& g, Regs& q) const {
        k = min(k, nchunks - 1);
        const int off = g.off + base_off() + k * off_step();
        const uint32_t o = (uint32_t)clamped(off), ow = BWD ? (uint32_t)clamped(off + wshift() * (int)sizeof(T)) : o;
        q.x = rg_load((const T*)(X + o));
        q.l = rg_load((const T*)(LAM + o));
        q.w0 = rg_load((const T*)(W0 + ow));
        q.w1 = rg_load((const T*)(W1 + ow));
        q.w2 = rg_load((const T*)(W2 + ow));
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
            const bool z = (BWD && (wl < 0 || wl > S1)) || starts_stretch(drev ? S1 - wl : wl, S1 + 1, drev, kc);
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
        const uint32_t s0 = g.slot + buf(k);
        const int ss = slot_step();
        if constexpr (WIDE) {
            const bool row_first = g.row == 0, row_last = g.row == H - 1;
            // a vertical scan's granule is E / NV blocks, a horizontal scan's element e lies on a line of its own
            constexpr int N = HORZ ? 1 : NV;
#pragma unroll
            for (int b = 0; b < E; b += N) {
                if constexpr (sizeof(T) == 2) __builtin_amdgcn_sched_barrier(0);        // block by block: registers
                float f[3][N];
#pragma unroll
                for (int v = 0; v < N; ++v) {
                    const int e = b + v;
                    const bool o0 = HORZ ? row_first : (e == 0 && col == 0);
                    const bool o2 = HORZ ? row_last : (col + e == W - 1);
                    float f0 = rg_elem<T>(w0, e), f1 = rg_elem<T>(w1, e), f2 = rg_elem<T>(w2, e);
                    if constexpr (LOGITS) softmax3(f0, f1, f2, o0, o2);
                    const bool dd = (dead >> e) & 1u;
                    f[0][v] = (dd || o0) ? 0.f : f0; f[1][v] = dd ? 0.f : f1; f[2][v] = (dd || o2) ? 0.f : f2;
                }
                if constexpr (HORZ) {
                    const uint32_t s = s0 + b * ss;
                    if constexpr (NV == 1) lds_set<u32x4>(s, u32x4{__float_as_uint(av[b]), __float_as_uint(f[0][0]), __float_as_uint(f[1][0]), __float_as_uint(f[2][0])});
                    else {
                        lds_set<float>(s, av[b]); lds_set<float>(s + ARR, f[0][0]); lds_set<float>(s + 2 * ARR, f[1][0]); lds_set<float>(s + 3 * ARR, f[2][0]);
                    }
                } else {
                    const uint32_t s = s0 + b / NV * block_bytes();
                    if constexpr (NV == 1) lds_set<u32x4>(s, u32x4{__float_as_uint(av[b]), __float_as_uint(f[0][0]), __float_as_uint(f[1][0]), __float_as_uint(f[2][0])});
                    else if constexpr (NV == 2) {
                        lds_set<u32x4>(s, u32x4{__float_as_uint(av[b]), __float_as_uint(av[b + 1]), __float_as_uint(f[0][0]), __float_as_uint(f[0][1])});
                        lds_set<u32x4>(s + 16, u32x4{__float_as_uint(f[1][0]), __float_as_uint(f[1][1]), __float_as_uint(f[2][0]), __float_as_uint(f[2][1])});
                    } else {
                        lds_set<u32x4>(s, u32x4{__float_as_uint(av[b]), __float_as_uint(av[b + 1]), __float_as_uint(av[b + 2]), __float_as_uint(av[b + 3])});
#pragma unroll
                        for (int i = 0; i < 3; ++i)
                            lds_set<u32x4>(s + 16 + 16 * i, u32x4{__float_as_uint(f[i][0]), __float_as_uint(f[i][1]), __float_as_uint(f[i][2]), __float_as_uint(f[i][3])});
                    }
                }
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
            if constexpr (HORZ) {
                const uint32_t s2 = s0 + 2 * ARR - (NV == 1 ? 0 : g.row % NV * 2);         // (tap 2 is two bytes of NV positions side by side)
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    lds_set<uint32_t>(s0 + e * ss, __float_as_uint(av[e]));
                    lds_set<uint32_t>(s0 + e * ss + ARR, w01[e]);
                    lds_set<uint16_t>(s2 + e * ss, (uint16_t)((e & 1) ? w2[e >> 1] >> 16 : w2[e >> 1]));
                }
            } else {
#pragma unroll
                for (int b = 0; b < E; b += NV) {
                    const uint32_t s = s0 + b / NV * block_bytes();
                    if constexpr (NV == 1) {
                        lds_set<float>(s, av[b]); lds_set<uint32_t>(s + 4, w01[b]); lds_set<uint32_t>(s + 8, (b & 1) ? w2[b >> 1] >> 16 : w2[b >> 1]);
                    } else if constexpr (NV == 2) {
                        lds_set<float>(s, av[b]); lds_set<float>(s + 4, av[b + 1]);
                        lds_set<uint32_t>(s + 8, w01[b]); lds_set<uint32_t>(s + 12, w01[b + 1]);
                        lds_set<uint32_t>(s + 16, w2[b >> 1]);
                    } else {
                        lds_set<u32x2>(s, u32x2{__float_as_uint(av[b]), __float_as_uint(av[b + 1])});
                        lds_set<u32x2>(s + 8, u32x2{__float_as_uint(av[b + 2]), __float_as_uint(av[b + 3])});
                        lds_set<u32x2>(s + 16, u32x2{w01[b], w01[b + 1]});
                        lds_set<u32x2>(s + 24, u32x2{w01[b + 2], w01[b + 3]});
                        lds_set<u32x2>(s + 32, u32x2{w2[b >> 1], w2[(b >> 1) + 1]});
                    }
                }
            }
        }
    }

    // h of the chunk from LDS, in registers for store().  The two are apart because a wait for a request counts the stores issued
    // behind it: store() comes when the next chunk's requests have been waited for.
    struct Out { u32x4 v, lw; u32x4 h[E / 4]; };
    __device__ __forceinline__ void finish(int k, const Gran& g, Out& out) const {
        if (!live(g, k)) return;
        __builtin_amdgcn_sched_barrier(0);
        const uint32_t s0 = (NV == 4 ? g.h : g.slot) + buf(k);
        float h[E];
        if constexpr (HORZ) {
            const int ss = slot_step();
#pragma unroll
            for (int e = 0; e < E; ++e) h[e] = lds_get<float>(s0 + e * ss);
        } else {
#pragma unroll
            for (int b = 0; b < E; b += NV) {
                const uint32_t s = s0 + b / NV * (NV == 4 ? g.hstep : block_bytes());
                if constexpr (NV == 1) h[b] = lds_get<float>(s);
                else if constexpr (NV == 2) { h[b] = lds_get<float>(s); h[b + 1] = lds_get<float>(s + 4); }
                else {
                    u32x4 t;
                    if constexpr (WIDE) t = lds_get<u32x4>(s);
                    else { const u32x2 t0 = lds_get<u32x2>(s), t1 = lds_get<u32x2>(s + 8); t = u32x4{t0[0], t0[1], t1[0], t1[1]}; }
#pragma unroll
                    for (int v = 0; v < 4; ++v) h[b + v] = __uint_as_float(t[v]);
                }
            }
        }
        if constexpr (PART) {
#pragma unroll
            for (int i = 0; i < E / 4; ++i)
                out.h[i] = u32x4{__float_as_uint(h[4 * i]), __float_as_uint(h[4 * i + 1]), __float_as_uint(h[4 * i + 2]), __float_as_uint(h[4 * i + 3])};
        }
        if constexpr (HSAVE) {
            if constexpr (sizeof(T) == 4) {
                out.v = u32x4{__float_as_uint(h[0]), __float_as_uint(h[1]), __float_as_uint(h[2]), __float_as_uint(h[3])};
            } else if (BWD) {                 // e as two 16-bit halves of its fp32 word
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
    }
    __device__ __forceinline__ void store(int k, const Gran& g, const Out& out) const {
        if (!live(g, k)) return;
        const int n = W - (HORZ ? g.col + k * col_step() : g.col);           // elements inside the row
        const uint32_t off = (uint32_t)(g.off + k * off_step());
        if (n >= E) {
            if constexpr (HSAVE) rg_store((T*)(HS + off), out.v);
            if constexpr (BWD && sizeof(T) == 2) rg_store((T*)(LO + off), out.lw);
            if constexpr (PART) {
#pragma unroll
                for (int i = 0; i < E / 4; ++i) rg_store(PT + off / sizeof(T) + 4 * i, out.h[i]);
            }
        } else {
#pragma unroll
            for (int e = 0; e < E; ++e)
                if (e < n) {
                    if constexpr (HSAVE) rg_store_bits((T*)(HS + off) + e, rg_bits<T>(out.v, e));
                    if constexpr (BWD && sizeof(T) == 2) rg_store_bits((T*)(LO + off) + e, rg_bits<T>(out.lw, e));
                    if constexpr (PART) PT[off / sizeof(T) + e] = __uint_as_float(out.h[e / 4][e % 4]);
                }
        }
    }

    // The scan of nsub * 8 lines of chunk k by a scanning wave; h: state of this lane's positions.  The LDS reads of HL lines are
    // issued while the HL lines before them are computed: one wave per SIMD scans, and nothing else hides their latency.
    // Lanes beyond the line are switched off: what they would hold never reaches a position of the line.
    template <bool LOCAL>
    __device__ __forceinline__ void scan(int k, int nsub, int start, float (&h)[NV], int until) const {
        constexpr int HL = NV == 4 ? 2 : 4;             // what the registers hold twice
        constexpr int NB = AP_SUB / HL;
        const int pos = start + ((int)threadIdx.x & 63) * NV;
        const int own = part * a.own[HORZ];
        const bool mine = pos >= own && pos < own + a.own[HORZ];
        if (pos < L) {
            bool valid[NV];                             // (a lane's first position is)
#pragma unroll
            for (int v = 1; v < NV; ++v) valid[v] = pos + v < L;
            uint32_t ra = lds0 + buf(k) + place_of(pos);
            // positions that another wave owns are computed for their neighbours' sake: their h goes to a place of no one's
            uint32_t rh = mine ? lds0 + buf(k) + h_of(pos) : lds0 + a.edge_off[HORZ] - 16, step_h = mine ? pitch : 0, skew_h = mine ? skew : 0;
            struct Line { float a[NV], w0[NV], w1[NV], w2[NV]; };
            struct Raw { u32x4 q[WIDE ? NV : NV == 4 ? 3 : 2]; };
            auto read = [&](Raw& q) {
                if constexpr (WIDE) {
#pragma unroll
                    for (int i = 0; i < NV; ++i) q.q[i] = lds_get<u32x4>(ra + 16 * i);
                } else if constexpr (NV == 1) {
                    q.q[0] = u32x4{lds_get<uint32_t>(ra), lds_get<uint32_t>(ra + 4), lds_get<uint32_t>(ra + 8), 0};
                } else if constexpr (NV == 2) {
                    q.q[0] = u32x4{lds_get<uint32_t>(ra), lds_get<uint32_t>(ra + 4), lds_get<uint32_t>(ra + 8), lds_get<uint32_t>(ra + 12)};
                    q.q[1][0] = lds_get<uint32_t>(ra + 16);
                } else {
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const u32x2 t0 = lds_get<u32x2>(ra + 16 * i), t1 = lds_get<u32x2>(ra + 16 * i + 8);
                        q.q[i] = u32x4{t0[0], t0[1], t1[0], t1[1]};
                    }
                    const u32x2 t = lds_get<u32x2>(ra + 32);
                    q.q[2][0] = t[0]; q.q[2][1] = t[1];
                }
                ra += pitch;
            };
            auto unpack = [&](const Raw& q, Line& t) {
                auto word = [&](int i) { return q.q[i / 4][i % 4]; };
#pragma unroll
                for (int v = 0; v < NV; ++v) {
                    t.a[v] = __uint_as_float(word(v));
                    if constexpr (WIDE) {
                        t.w0[v] = __uint_as_float(word(NV + v)); t.w1[v] = __uint_as_float(word(2 * NV + v)); t.w2[v] = __uint_as_float(word(3 * NV + v));
                    } else {
                        t.w0[v] = word_lo<T>(word(NV + v)); t.w1[v] = word_hi<T>(word(NV + v));
                        const uint32_t w = word(2 * NV + v / 2);
                        t.w2[v] = (v & 1) ? word_hi<T>(w) : word_lo<T>(w);
                    }
                }
            };
            auto line = [&](const Raw& q) {
                Line t;
                unpack(q, t);
                float r[NV];
                bool keep = true;
                if constexpr (LOCAL) {
                    // a stretch starts with the next line: nothing is carried into it, whatever the state holds (the weights there are
                    // 0 already)
                    keep = --until != 0;
                    until = keep ? until : a.p.kchunk;
                }
                if constexpr (BWD) {
                    // a position takes the taps that reach it from its neighbours
                    float wb[NV], wa[NV];
#pragma unroll
                    for (int v = 1; v < NV; ++v) t.w0[v] = valid[v] ? t.w0[v] : 0.f;
                    wb[0] = from_lane_below(t.w2[NV - 1]);
                    wa[NV - 1] = from_lane_above(t.w0[0]);
#pragma unroll
                    for (int v = 1; v < NV; ++v) { wb[v] = t.w2[v - 1]; wa[v - 1] = t.w0[v]; }
                    line_step<NV>(r, t.a, h, wb, t.w1, wa);
                } else {
                    line_step<NV>(r, t.a, h, t.w0, t.w1, t.w2);
                }
                if constexpr (NV == 1) lds_set<float>(rh, r[0]);
                else if constexpr (NV == 2) { lds_set<float>(rh, r[0]); lds_set<float>(rh + 4, r[1]); }
                else if constexpr (!WIDE) {
                    lds_set<u32x2>(rh, u32x2{__float_as_uint(r[0]), __float_as_uint(r[1])});
                    lds_set<u32x2>(rh + 8, u32x2{__float_as_uint(r[2]), __float_as_uint(r[3])});
                } else lds_set<u32x4>(rh, u32x4{__float_as_uint(r[0]), __float_as_uint(r[1]), __float_as_uint(r[2]), __float_as_uint(r[3])});
                rh += step_h;
#pragma unroll
                for (int v = 0; v < NV; ++v) h[v] = ((v == 0 || valid[v]) && keep) ? r[v] : 0.f;
            };
            Raw q[2][HL];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int j = 0; j < HL; ++j) read(q[i][j]);
                if ((i + 1) * HL % E == 0) ra += skew;
            }
            for (int s = 0; s < nsub; ++s) {
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    static_assert(NB % 2 == 0, "the two line sets alternate");
#pragma unroll
                    for (int j = 0; j < HL; ++j) line(q[i & 1][j]);
                    if ((i + 1) * HL % E == 0) rh += skew_h;
                    __builtin_amdgcn_sched_barrier(0);
                    if (i + 2 < NB || s + 1 < nsub) {
#pragma unroll
                        for (int j = 0; j < HL; ++j) read(q[i & 1][j]);
                        if ((i + 3) * HL % E == 0) ra += skew;
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    }

    __device__ __forceinline__ void run(int dir, int first_line) {
        const FwdParams& p = a.p;
        constexpr int ax = HORZ ? 1 : 0;
        d = dir;
        rev = BWD ? !(d & 1) : (d & 1);
        part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        H = p.H; W = p.W; HW = H * W;
        lo = first_line; lines = min(a.range[ax], (HORZ ? W : H) - lo);
        S = HORZ ? (lines + E - 1) / E * E : lines; L = HORZ ? H : W;
        K = a.K[ax]; pitch = a.pitch[ax]; skew = a.skew[ax]; parts = a.parts[ax];
        nthr = (int)blockDim.x - parts * 64;                     // the first `parts` waves scan, the others load
        tid = (int)threadIdx.x - parts * 64;
        const size_t planes = (size_t)p.B * p.C, groups = (size_t)p.B * p.G;
        const size_t pc = (size_t)plane * HW;
        const size_t slot_c = p.shared ? 0 : (size_t)d * planes * HW;
        const size_t slot_w = p.shared ? 0 : (size_t)d * groups * 3 * HW;
        const size_t back = bg == 0 ? 0 : (size_t)HW;             // the neighbouring plane a window may reach into
        X = (const char*)((const T*)p.x + pc - back);
        LAM = (const char*)((const T*)p.lam + slot_c + pc - back);
        W0 = (const char*)((const T*)p.w + slot_w + (size_t)bg * 3 * HW - back);
        W1 = W0 + (size_t)HW * sizeof(T);
        W2 = W1 + (size_t)HW * sizeof(T);
        HS = HSAVE ? (char*)((T*)p.hs + (size_t)d * planes * HW + pc) : nullptr;
        PT = PART ? a.part + (size_t)d * planes * HW + pc : nullptr;
        LO = (BWD && sizeof(T) == 2) ? (char*)((T*)a.hs_lo + (size_t)d * planes * HW + pc) : nullptr;
        at_ends = bg == 0 || bg == (int)groups - 1;
        top = ((int)back + (bg == (int)groups - 1 ? HW : 2 * HW) - E) * (int)sizeof(T);
        next_buf = a.chunk[ax];
        edge = (float*)(lds + a.edge_off[ax]);
        nchunks = (S + K - 1) / K;
        if (part < parts) {
            __builtin_amdgcn_s_setprio(3);       // the chain the others wait for
            if (p.kchunk > 0 && lines > p.kchunk) scan_all<true>();
            else scan_all<false>();
            __builtin_amdgcn_s_setprio(0);
        } else {
            if (__builtin_amdgcn_readfirstlane(tid) >= granules()) {                            // (the same for the whole wave)
                // a loading wave without a granule: the barriers of the others
                for (int n = a.nbuf == 2 ? nchunks + 2 : 1 + 2 * nchunks; n > 0; --n) lds_barrier();
                return;
            }
            const bool two = granules() > nthr;                     // granules of a chunk per thread
            if (a.nbuf == 2) {
                if (two) move_ahead<2, 1>(); else move_ahead<1, 2>();
            } else {
                if (two) move_in_turn<2>(); else move_in_turn<1>();
            }
        }
    }

    __device__ __forceinline__ int subs(int k) const { return (min(K, S - k * K) + AP_SUB - 1) / AP_SUB; }
    // A scanning wave's part of a pass: the barriers below are the ones of move_ahead / move_in_turn.
    template <bool LOCAL>
    __device__ __forceinline__ void scan_all() {
        float h[NV];
#pragma unroll
        for (int v = 0; v < NV; ++v) h[v] = 0.f;
        // scan steps to the next stretch: cuts lie before image lines 0, kchunk, 2 * kchunk, ..
        int until = 1 << 30;
        if (LOCAL) until = rev && S % a.p.kchunk ? S % a.p.kchunk : a.p.kchunk;
        const bool ahead = a.nbuf == 2;
        // this wave's window of the line: its own positions and, of a line that others share, K of its neighbours' on either side,
        // so that the K steps of a chunk need nothing from outside; the states at the end of a chunk pass through `edge`
        const int start = part == 0 ? 0 : part * a.own[HORZ] - K;
        const int pos = start + ((int)threadIdx.x & 63) * NV, own = part * a.own[HORZ];
        lds_barrier();
        for (int k = 0; k < nchunks; ++k) {
            scan<LOCAL>(k, subs(k), start, h, until);
            if (LOCAL) for (until -= subs(k) * AP_SUB; until <= 0;) until += a.p.kchunk;
            if (parts > 1 && pos >= own && pos < min(L, own + a.own[HORZ])) {
                float* const to = edge + (k & 1) * a.edge_len[HORZ];
#pragma unroll
                for (int v = 0; v < NV; ++v) to[pos + v] = h[v];
            }
            if (!ahead) lds_barrier();
            lds_barrier();
            if (parts > 1 && pos < L) {
                const float* const from = edge + (k & 1) * a.edge_len[HORZ];
#pragma unroll
                for (int v = 0; v < NV; ++v) h[v] = pos + v < L ? from[pos + v] : 0.f;
            }
        }
        if (ahead) lds_barrier();
    }

    // A loading wave's part with two chunks in LDS: while chunk k is scanned, chunk k - 1 is finished, chunk k + 1 takes its
    // place and the requests of chunk k + 1 + DEPTH go out.  A thread reads and writes its own granules' places there, so nothing but
    // the end of the scan is waited for.  R: granules of a chunk per thread; DEPTH: chunks in flight, two where a thread's one granule
    // leaves the registers, which hides a memory latency longer than a chunk's scan.
    template <int R, int DEPTH>
    __device__ __forceinline__ void move_ahead() {
        Regs q[DEPTH][R];
        Gran g[R];
        Out out[R];
#pragma unroll
        for (int r = 0; r < R; ++r) g[r] = place(r);
#pragma unroll
        for (int i = 0; i < DEPTH; ++i)
#pragma unroll
            for (int r = 0; r < R; ++r) load(i, g[r], q[i][r]);
#pragma unroll
        for (int r = 0; r < R; ++r) stage(0, g[r], q[0][r]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int r = 0; r < R; ++r) load(DEPTH, g[r], q[0][r]);
        lds_barrier();
        auto chunk = [&](int k, Regs (&next)[R]) {
            if (k > 0) {
#pragma unroll
                for (int r = 0; r < R; ++r) finish(k - 1, g[r], out[r]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < R; ++r) stage(k + 1, g[r], next[r]);
            __builtin_amdgcn_sched_barrier(0);
            if (k > 0) {
#pragma unroll
                for (int r = 0; r < R; ++r) store(k - 1, g[r], out[r]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < R; ++r) load(k + 1 + DEPTH, g[r], next[r]);
            __builtin_amdgcn_sched_barrier(0);
            lds_barrier();
        };
        for (int k = 0; k <= nchunks; k += DEPTH) {
            chunk(k, q[1 % DEPTH]);
            if constexpr (DEPTH == 2) {
                if (k + 1 <= nchunks) chunk(k + 1, q[0]);
            }
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
            for (int r = 0; r < R; ++r) load(k + 1, g[r], q[r]);
            __builtin_amdgcn_sched_barrier(0);
            lds_barrier();
#pragma unroll
            for (int r = 0; r < R; ++r) finish(k, g[r], out[r]);
#pragma unroll
            for (int r = 0; r < R; ++r) stage(k + 1, g[r], q[r]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int r = 0; r < R; ++r) store(k, g[r], out[r]);
            lds_barrier();
        }
    }
};

template <typename T, int MODE, bool LOGITS, int NV>
__global__ void __launch_bounds__(1024) apart_kernel(ApartArgs a) {
    extern __shared__ __attribute__((aligned(16))) char ap_lds[];
    const FwdParams& p = a.p;
    // neighbouring planes on one XCD, so that the channels of a group meet in one L2 with the weights of their direction, and every
    // XCD works on all directions, whose scans differ in length
    const int planes = p.B * p.C;
    const bool eighths = planes % 8 == 0;
    const int per = eighths ? planes / 8 : planes, at = eighths ? (int)(blockIdx.x >> 3) : (int)xcd_contiguous_item(blockIdx.x, gridDim.x);
    int q = at / per;
    const int plane = at - q * per + (eighths ? (int)(blockIdx.x & 7) * per : 0);
    const int b = plane / p.C, bg = b * p.G + (plane - b * p.C) / p.cpg;
    const int nv = 2 * a.nrange[0];
    const bool horz = q >= nv;
    if (horz) q -= nv;
    const int di = q / a.nrange[horz], first = (q - di * a.nrange[horz]) * a.range[horz];
    const int d = di + 2 * horz;
    if (horz) {
        ApartPass<T, MODE, LOGITS, NV, true> v(a, ap_lds);
        v.plane = plane; v.bg = bg;
        v.run(d, first);
    } else {
        ApartPass<T, MODE, LOGITS, NV, false> v(a, ap_lds);
        v.plane = plane; v.bg = bg;
        v.run(d, first);
    }
}

template <typename T, int MODE, bool LOGITS>
hipError_t launch_apart_one(const ApartArgs& a, int threads, int nv, size_t lds, hipStream_t s) {
    const int items = 2 * (a.nrange[0] + a.nrange[1]);
    const dim3 grid((unsigned)((size_t)a.p.B * a.p.C * items)), block(threads);
    void (*k)(ApartArgs) = nv == 1 ? apart_kernel<T, MODE, LOGITS, 1> : nv == 2 ? apart_kernel<T, MODE, LOGITS, 2> : apart_kernel<T, MODE, LOGITS, 4>;
    const hipError_t e = allow_dynamic_lds((const void*)k, 160 * 1024);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, grid, block, lds, s, a);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_apart_type(const ApartArgs& a, bool reverse, int threads, int nv, size_t lds, hipStream_t s) {
    if (reverse) return a.p.logits ? launch_apart_one<T, AP_BWD, true>(a, threads, nv, lds, s) : launch_apart_one<T, AP_BWD, false>(a, threads, nv, lds, s);
    if (a.p.hs) return a.p.logits ? launch_apart_one<T, AP_SAVE, true>(a, threads, nv, lds, s) : launch_apart_one<T, AP_SAVE, false>(a, threads, nv, lds, s);
    if constexpr (sizeof(T) == 4) return hipErrorInvalidValue;
    else return a.p.logits ? launch_apart_one<T, AP_FWD, true>(a, threads, nv, lds, s) : launch_apart_one<T, AP_FWD, false>(a, threads, nv, lds, s);
}

}  // namespace
}  // namespace gspn
