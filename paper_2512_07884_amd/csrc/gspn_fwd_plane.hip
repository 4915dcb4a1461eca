// Forward GSPN scan for small feature maps (lines of at most 64 positions, planes of at most 8 KB in
// storage precision: 56x56 bf16, 28x28 fp32, ...): every tensor is read from global memory exactly
// once per use as flat, fully coalesced 16 B-per-lane plane copies, and the scans run out of LDS.
//
// Per (channel, direction) the recurrence of Eq. 1 (Sec. 3.2)
//     h_s[j] = w0_s[j] h_{s-1}[j-1] + w1_s[j] h_{s-1}[j] + w2_s[j] h_{s-1}[j+1] + lam_s[j] x_s[j]
// is walked by one wave: lane = position j on the line (two channels side by side when a line fits
// in 32 lanes), the previous line's neighbours come from DPP whole-wave shifts, and the per-step
// operands a = lam*x, w0, w1, w2 are read from fp32 planes in LDS through an address walk whose stride
// encodes the direction (+-pitch for the vertical scans, +-1 for the horizontal ones), so that one
// code path serves all four directions.  h overwrites a in place; afterwards the plane is read back
// in the flat layout for y += u*h (Eq. 2 and the sum merge of the four passes, accumulated in
// registers and rounded once) and, when asked for, h_save.
//
// What this saves over line-by-line loading: x is loaded once for all directions and stays in
// registers; with channel-shared weights (Sec. 4.2) the three weight planes of a direction are
// loaded ONCE per workgroup into LDS and read by all its channels; every request is a complete
// cache line.  Rows in LDS have an odd pitch so that both access orientations are conflict-free.
//
// Maps whose rows are not whole 16 B chunks (7x7, 14x14, 28x28 bf16: the later stages of a classifier), and small
// maps whose rows are, take the FLAT variant: LDS planes without padding, so that a chunk's place in LDS is its place in memory and
// chunks may run over row and channel ends; 2, 4 or 8 channels side by side in a wave (32, 16 or 8 lanes
// each) so that the wave's channels together are whole chunks; weights fetched in the widest pieces their
// alignment allows.
#include "gspn_tile_common.hpp"
#include <stdlib.h>

namespace gspn {

namespace {

typedef float pf32a __attribute__((may_alias));
typedef __attribute__((address_space(3))) pf32a plds_f32;
extern __shared__ float plane_lds[];

__device__ __forceinline__ uint32_t plds_base() {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)plane_lds;
}
__device__ __forceinline__ float plds_ld(uint32_t a) { return *(const plds_f32*)(uintptr_t)a; }
__device__ __forceinline__ void plds_st(uint32_t a, float v) { *(plds_f32*)(uintptr_t)a = v; }
typedef float pf32x4a __attribute__((ext_vector_type(4), may_alias));
typedef __attribute__((address_space(3))) pf32x4a plds_f32x4;
__device__ __forceinline__ pf32x4a plds_ld4(uint32_t a) { return *(const plds_f32x4*)(uintptr_t)a; }
typedef uint32_t pu32x2a __attribute__((ext_vector_type(2), may_alias));
typedef __attribute__((address_space(3))) pu32x2a plds_u32x2;
__device__ __forceinline__ u32x2 plds_ld2(uint32_t a) { const pu32x2a v = *(const plds_u32x2*)(uintptr_t)a; return u32x2{v.x, v.y}; }
__device__ __forceinline__ void plds_st2(uint32_t a, uint32_t x, uint32_t y) { *(plds_u32x2*)(uintptr_t)a = pu32x2a{x, y}; }
__device__ __forceinline__ void plds_st4(uint32_t a, pf32x4a v) { *(plds_f32x4*)(uintptr_t)a = v; }

// element e of a 16 B chunk of storage, widened to fp32
template <typename T> __device__ __forceinline__ float chunk_elem(const u32x4& c, int e) {
    if constexpr (sizeof(T) == 4) return __uint_as_float(c[e]);
    else return (e & 1) ? word_hi<T>(c[e >> 1]) : word_lo<T>(c[e >> 1]);
}
template <typename T> __device__ __forceinline__ u32x4 chunk_pack(const float* v) {
    u32x4 c;
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] = __float_as_uint(v[e]);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] = pack_word<T>(v[2 * e], v[2 * e + 1]);
    }
    return c;
}

}  // namespace

struct FwdPlaneArgs {
    FwdParams p;
    int K;        // channels per workgroup
    int cpw;      // channels per wave (1, 2, 4 or 8): each takes 64 / cpw lanes
    int lsh;      // log2 of the lanes per channel
    int nwaves;
    int pitch;    // LDS row pitch in floats (odd; W in the flat variant)
    int wlw;      // flat variant, shared weights: bytes per weight request (16, 8, 4 or 2)
    uint64_t seg[4];   // per direction: bit r set <=> image line r of the scan axis starts a stretch in scan order
};

// WPRE (shared weights): the workgroup has enough threads to hold a direction's weights in registers
// (WSH chunks per thread), so they are requested a direction ahead; otherwise they are fetched in place.
// FLAT: planes in LDS are unpadded and the wave's channels contiguous (see the head of the file).
// LOCAL: GSPN-local (Sec. 3.2), on instantiations of its own so that the global scan carries none of it.
// BWD: the reverse sweep of the backward pass (first pass of the two-pass backward scan) on the same machinery: the
// caller passes gy as x, u as lam, lam as u, gx as y and the buffer that receives e as hs; every direction is walked
// against its scan order, and a position multiplies its state by the taps of the line swept before and hands the
// products to the positions those taps read from (e_t = u_t*gy_t + T_{t+1}^T e_{t+1}).  The taps that are stored as 0
// (out-of-line neighbours, GSPN-local: lines that start a stretch) are the ones that must pass nothing on here too.
// W16: a group's weights in LDS as {w0, w1} in 16 bits and w2 in fp32, 8 bytes per position instead of 16, so that a CU holds eight waves in two
// or more workgroups where it held six in one, which all waited for the memory at once: 6144 planes 56x56 bf16 (cpg 12) 141 -> 106 us, with
// h_save and backward 512 -> 457, 48x48 f16 113 -> 84, 17280 of 36x32 176 -> 166; 0.86 in the mean of 1080 calls.
// NCHT: 16 B chunks per lane the register arrays are sized for (8: the wave's channels hold at most 8 KB; 4: small maps
// with weights of each channel's own, and those of the flat variant, which then has the registers to give its LDS planes an odd pitch too -- every element's place is
// tracked through two bit masks per chunk)
// (fp32 planes of the flat variant with eight chunks per lane need 167 to 171 registers as the compiler lays them out; 168 are what three waves
// per SIMD may have: 1872 planes 38x38 fp32 with logits and stretches, h_save, 59 us with three, 86 with two)
template <typename T, bool SAVE, bool SHARED, bool WPRE, bool FLAT, bool LOCAL, bool BWD = false, int NCHT = 8, bool W16 = false>
__global__ void __launch_bounds__(SHARED ? 512 : 256, sizeof(T) == 4 && FLAT && NCHT == 8 ? 3 : SHARED ? 2 : 1) fwd_plane_kernel(FwdPlaneArgs a) {
    static_assert(!(FLAT && WPRE), "the flat variant fetches its weights in place");
    static_assert(NCHT == 8 || (NCHT == 4 && (FLAT || !SHARED)), "the short register arrays are for small maps of the flat variant and with weights of each channel's own");
    constexpr bool WAHEAD = !SHARED && !FLAT && NCHT == 4;        // at most 4 KB of channels per wave, their weights requested a direction ahead
    constexpr bool PADFLAT = FLAT && NCHT == 4;    // flat variant with padded LDS planes
    static_assert(!BWD || SAVE, "the reverse sweep saves its state");
    constexpr int E = 16 / (int)sizeof(T);        // elements per 16 B chunk
    constexpr int NCH = NCHT;                     // chunks per lane
    static_assert(!W16 || (sizeof(T) == 2 && WPRE && !LOCAL), "16-bit weights in LDS: the prefetching variant's, normalised, global scan");
    constexpr int WSH = W16 ? 6 : 4;              // weight chunks per thread (shared weights; W16: the same chunk of the three taps, twice)
    constexpr uint32_t WPOS = W16 ? 8 : 16;       // bytes per position of the weights in LDS
    const FwdParams& p = a.p;
    const int H = p.H, W = p.W, HW = H * W, P = a.pitch;
    const int HP = (FLAT && !PADFLAT) ? HW : (H * P + 3) & ~3;   // floats per plane region in LDS (16 B granules when padded)
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int cpw = a.cpw;
    const int half = lane >> a.lsh;                    // which of the wave's channels this lane works on
    const int i = lane & ((1 << a.lsh) - 1);           // position on the line
    const int wgs_per_image = p.C / a.K;
    const unsigned item = xcd_contiguous_item(blockIdx.x, gridDim.x);
    const int b = item / wgs_per_image;
    const int c_first = (item - b * wgs_per_image) * a.K;
    const int c0 = c_first + wave * cpw;                               // first channel of this wave
    const size_t planes = (size_t)p.B * p.C, groups = (size_t)p.B * p.G;
    const size_t pc = ((size_t)b * p.C + c0) * HW;
    const int n16 = cpw * HW / E;                                      // 16 B chunks of the wave's channels
    const int n16p = HW / E;                                           // ... of one plane

    // LDS (floats).  Weights are kept interleaved, [H][P][4] = (w0, w1, w2, unused) per position, so that a scan
    // step fetches its three taps with one 16 B read (W16: {w0, w1} in 16 bits, w2 in fp32, 8 bytes).  Shared weights: one such region for the direction,
    // then per wave [cpw][H][P] a/h.  Per-channel weights: per wave [cpw] weight regions, then [cpw][H][P] a/h.
    const uint32_t base = plds_base();
    const uint32_t wreg = SHARED ? base : base + 4u * (uint32_t)(wave * cpw * 5 * HP);
    const uint32_t ahreg = SHARED ? base + 4u * (uint32_t)((W16 ? 2 : 4) * HP + wave * cpw * HP)
                                  : wreg + 4u * (uint32_t)(cpw * 4 * HP);

    // flat layout: chunk q = k*64 + lane covers elements [q*E, q*E + E) of the wave's channels
    bool vq[NCH];
    int rc[NCH];          // row*P + col of the chunk's first element (padded flat variant: plus its channel's region)
    int ch[NCH];          // channel of the wave (0 / 1) the chunk belongs to
    int row0[NCH], col0[NCH];
    // padded flat variant: a chunk may run over the end of a row and of a channel: bit e set <=> element e of the chunk is
    // the last of its row / of its channel, i.e. the next element's place in LDS is further by the row / region padding
    uint32_t rowend[NCH], chend[NCH];
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
        const int q = k * 64 + lane;
        vq[k] = q < n16;
        const int idx0 = vq[k] ? q * E : 0;
        rowend[k] = 0; chend[k] = 0;
        if constexpr (PADFLAT) {
            const int c = idx0 / HW, rem = idx0 - c * HW;
            int row = rem / W, col = rem - row * W;
            ch[k] = 0; rc[k] = c * HP + row * P + col; row0[k] = 0; col0[k] = 0;
#pragma unroll
            for (int e = 0; e < E; ++e) {
                if (++col == W) {
                    col = 0; rowend[k] |= 1u << e;
                    if (++row == H) { row = 0; chend[k] |= 1u << e; }
                }
            }
        } else if constexpr (FLAT) {
            ch[k] = 0; rc[k] = idx0; row0[k] = 0; col0[k] = 0;     // LDS offset = offset in memory
        } else {
            ch[k] = idx0 >= HW ? 1 : 0;
            const int rem = idx0 - ch[k] * HW;
            const int row = rem / W;
            rc[k] = row * P + (rem - row * W);
            row0[k] = row; col0[k] = rem - row * W;
        }
    }
    const uint32_t flat = (uint32_t)lane * 16u;
    const uint32_t row_pad4 = 4u * (uint32_t)(P - W), ch_pad4 = 4u * (uint32_t)(HP - H * P);   // padded flat variant: bytes skipped at a row / channel end
    auto ldg = [&](rsrc_t rs, uint32_t vo, int so) -> u32x4 { return __builtin_amdgcn_raw_buffer_load_b128(rs, vo, so, 0); };
    // x, lam, u: each line is asked for once by the whole launch (CP_STREAM: the caches give it up first)
    auto load_planes = [&](const T* basep, u32x4 (&st)[NCH]) {
        const rsrc_t rs = make_rsrc(basep);
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            u32x4 v = {0, 0, 0, 0};
            if (vq[k]) v = __builtin_amdgcn_raw_buffer_load_b128(rs, flat, k * 1024, CP_STREAM);
            st[k] = v;
        }
    };

    // shared weights: the three planes of a direction are 3*n16p chunks, dealt round-robin to the threads
    const int nthreads = blockDim.x;
    bool wv[WSH];
    int wl[WSH];          // LDS float offset of the chunk's first element in the weight region (tap included)
    int wrow[WSH], wcol[WSH], wtap[WSH];
    uint32_t wgo[WSH];    // byte offset of the chunk from the group's first weight plane
    if constexpr (SHARED && WPRE) {
#pragma unroll
        for (int j = 0; j < WSH; ++j) {
            const int c = (int)threadIdx.x + (W16 ? j / 3 : j) * nthreads;
            wv[j] = c < (W16 ? 1 : 3) * n16p;
            const int cc = wv[j] ? c : 0;
            const int tap = W16 ? j % 3 : cc / n16p;
            const int idx0 = (W16 ? cc : cc - tap * n16p) * E;
            const int row = idx0 / W;
            wl[j] = 4 * (row * P + (idx0 - row * W)) + tap;
            wrow[j] = row; wcol[j] = idx0 - row * W; wtap[j] = tap;
            wgo[j] = (uint32_t)((tap * HW + idx0) * (int)sizeof(T));
        }
    }
    auto load_wshare = [&](const T* wbase, u32x4 (&st)[WSH]) {
        const rsrc_t rs = make_rsrc(wbase);
#pragma unroll
        for (int j = 0; j < WSH; ++j) {
            u32x4 v = {0, 0, 0, 0};
            if (wv[j]) v = ldg(rs, wgo[j], 0);
            st[j] = v;
        }
    };

    u32x4 xs[NCH];
    load_planes((const T*)p.x + pc, xs);
    float y[NCH][E];
#pragma unroll
    for (int k = 0; k < NCH; ++k)
#pragma unroll
        for (int e = 0; e < E; ++e) y[k][e] = 0.f;

    // directions in scan order; operands of the first one are requested here, later ones a direction ahead
    int d = 0;
    while (d < 4 && !((p.mask >> d) & 1u)) ++d;
    const int g = c_first / p.cpg;                                     // shared weights: the workgroup's group
    auto slot_c = [&](int dd) { return p.shared ? (size_t)0 : (size_t)dd * planes * HW; };
    auto wptr = [&](int dd, int grp) {
        return (const T*)p.w + (p.shared ? (size_t)0 : (size_t)dd * groups * 3 * HW) + ((size_t)b * p.G + grp) * 3 * HW;
    };
    u32x4 ls[NCH], us[NCH], wsh[WSH], wa[WAHEAD ? 3 : 1][NCH];
    auto load_wahead = [&](int dd) {
#pragma unroll
        for (int t = 0; t < (WAHEAD ? 3 : 0); ++t) {
            const rsrc_t rs = make_rsrc(wptr(dd, c0) + (size_t)t * HW);
#pragma unroll
            for (int k = 0; k < NCH; ++k) {
                u32x4 v = {0, 0, 0, 0};
                if (vq[k]) v = __builtin_amdgcn_raw_buffer_load_b128(rs, flat + (uint32_t)(ch[k] * 2 * HW * (int)sizeof(T)), k * 1024, CP_STREAM);
                wa[t][k] = v;
            }
        }
    };
    if (d < 4) {
        load_planes((const T*)p.lam + slot_c(d) + pc, ls);
        if constexpr (SHARED && WPRE) load_wshare(wptr(d, g), wsh);
        if constexpr (WAHEAD) load_wahead(d);
    }

    while (d < 4) {
        int dn = d + 1;
        while (dn < 4 && !((p.mask >> dn) & 1u)) ++dn;
        // element (position j, scan step s) of a plane sits at float offset j*ps + s0 + s*ss
        const bool vert = d < 2, rev = ((d & 1) != 0) != BWD;       // (the reverse sweep walks against the scan order)
        const int S = vert ? H : W, L = vert ? W : H;
        const int ps = vert ? 1 : P;
        const int ss4 = 4 * (vert ? (rev ? -P : P) : (rev ? -1 : 1));
        const int s0 = vert ? (rev ? (H - 1) * P : 0) : (rev ? W - 1 : 0);
        const bool active = i < L;
        const int ic = active ? i : L - 1;
        const bool first = i == 0, last = i == L - 1;
        const int tpos = ic * ps + s0;
        // GSPN-local (Sec. 3.2): a line that starts a stretch has no predecessor, so its three taps are stored as 0
        // like the out-of-line ones, and the sweep restarts from lam*x there without knowing about stretches.
        // The prefetching variant has no registers to spare for the test where the weights are written: it clears
        // those lines in a pass of its own afterwards.
        constexpr bool LOCAL_PASS = LOCAL && WPRE;
        // weights given as logits: a tap that takes no part is stored as -inf and the three are normalised in LDS
        const float masked = p.logits ? -__builtin_huge_valf() : 0.f;
        const uint64_t starts = LOCAL ? a.seg[d] : 0ull;
        auto no_pred = [&](int row, int col) { return LOCAL && !LOCAL_PASS && ((starts >> (vert ? row : col)) & 1ull) != 0; };

        // ---- operands into LDS
        if constexpr (FLAT) {
            if constexpr (SHARED) lds_barrier();           // every wave is done with the previous direction's weights
            // The block to bring in: the group's three planes (the threads of the workgroup share the work) or
            // the three planes of each of the wave's channels, which are contiguous in memory.  A request may run
            // over the end of a row, a plane or a channel: the place of every element is tracked on its own.
            const int nel = SHARED ? 3 * HW : cpw * 3 * HW;
            const int lw = SHARED ? a.wlw : 16;
            const int ew = lw / (int)sizeof(T);            // elements per request; divides nel (host)
            const int t0 = SHARED ? (int)threadIdx.x : lane, tn = SHARED ? nthreads : 64;
            const rsrc_t rs = make_rsrc(wptr(d, SHARED ? g : c0));
            // Weights of the wave's own channels four pieces at a time: piece by piece it waited for the memory up to 24 times per
            // direction (11136 planes 16x14 fp32 92 -> 78 us).  A group's are few pieces per thread, and the registers cost more there (9216
            // planes 14x14 f16 20 -> 30).
            if constexpr (SHARED) {
                for (int c = t0; c * ew < nel; c += tn) {
                    const int idx0 = c * ew;
                    const uint32_t bo = (uint32_t)(idx0 * (int)sizeof(T));
                    u32x4 v = {0, 0, 0, 0};
                    if (lw == 16) v = ldg(rs, bo, 0);
                    else if (lw == 8) { const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(rs, bo, 0, 0); v[0] = t.x; v[1] = t.y; }
                    else if (lw == 4) v[0] = __builtin_amdgcn_raw_buffer_load_b32(rs, bo, 0, 0);
                    else v[0] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, bo, 0, 0);
                    int chn = idx0 / (3 * HW);
                    int r = idx0 - chn * 3 * HW;
                    int tap = r / HW;
                    r -= tap * HW;
                    int row = r / W, col = r - row * W;
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        if (e < ew) {
                            // a tap that points outside the line is stored as 0, whatever the tensor holds there
                            const int pos = vert ? col : row;
                            const bool outside = (tap == 0 && pos == 0) || (tap == 2 && pos == L - 1) || no_pred(row, col);
                            plds_st(wreg + 4u * (uint32_t)(chn * 4 * HP + 4 * (row * P + col) + tap),
                                    outside ? masked : chunk_elem<T>(v, e));
                            if (++col == W) { col = 0; if (++row == H) { row = 0; if (++tap == 3) { tap = 0; ++chn; } } }
                        }
                    }
                }
            } else {
                constexpr int WB = 4;
                for (int cb = t0; cb * ew < nel; cb += WB * tn) {
                    u32x4 wv4[WB];
#pragma unroll
                    for (int j = 0; j < WB; ++j) {
                        const int c = cb + j * tn;
                        const uint32_t bo = (uint32_t)(c * lw);
                        u32x4 v = {0, 0, 0, 0};
                        if (c * ew < nel) {
                            if (lw == 16) v = ldg(rs, bo, 0);
                            else if (lw == 8) { const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(rs, bo, 0, 0); v[0] = t.x; v[1] = t.y; }
                            else if (lw == 4) v[0] = __builtin_amdgcn_raw_buffer_load_b32(rs, bo, 0, 0);
                            else v[0] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rs, bo, 0, 0);
                        }
                        wv4[j] = v;
                    }
#pragma unroll
                    for (int j = 0; j < WB; ++j) {
                        const int c = cb + j * tn, idx0 = c * ew;
                        if (idx0 >= nel) break;
                        int chn = idx0 / (3 * HW);
                        int r = idx0 - chn * 3 * HW;
                        int tap = r / HW;
                        r -= tap * HW;
                        int row = r / W, col = r - row * W;
#pragma unroll
                        for (int e = 0; e < E; ++e) {
                            if (e < ew) {
                                // a tap that points outside the line is stored as 0, whatever the tensor holds there
                                const int pos = vert ? col : row;
                                const bool outside = (tap == 0 && pos == 0) || (tap == 2 && pos == L - 1) || no_pred(row, col);
                                plds_st(wreg + 4u * (uint32_t)(chn * 4 * HP + 4 * (row * P + col) + tap),
                                        outside ? masked : chunk_elem<T>(wv4[j], e));
                                if (++col == W) { col = 0; if (++row == H) { row = 0; if (++tap == 3) { tap = 0; ++chn; } } }
                            }
                        }
                    }
                }
            }
        } else if constexpr (SHARED) {
            lds_barrier();                                 // every wave is done with the previous direction's weights
            if constexpr (W16) {
#pragma unroll
                for (int j = 0; j < WSH; j += 3) {
                    if (wv[j]) {
                        // a tap that points outside the line is stored as 0, whatever the tensor holds there
                        const uint32_t o = wreg + 2u * (uint32_t)wl[j];
                        const bool all0 = !vert && wrow[j] == 0, all2 = !vert && wrow[j] == L - 1;
#pragma unroll
                        for (int e = 0; e < E; ++e) {
                            const int pos = wcol[j] + e;
                            const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;
                            uint32_t w01 = __builtin_amdgcn_perm(wsh[j + 1][e >> 1], wsh[j][e >> 1], sel);
                            float w2 = chunk_elem<T>(wsh[j + 2], e);
                            w01 &= all0 || (vert && pos == 0) ? 0xffff0000u : 0xffffffffu;
                            w2 = all2 || (vert && pos == L - 1) ? 0.f : w2;
                            plds_st2(o + 8u * e, w01, __float_as_uint(w2));
                        }
                    }
                }
            } else if constexpr (WPRE) {
#pragma unroll
                for (int j = 0; j < WSH; ++j) {
                    if (wv[j]) {
#pragma unroll
                        for (int e = 0; e < E; ++e) {
                            // a tap that points outside the line is stored as 0, whatever the tensor holds there
                            const int pos = vert ? wcol[j] + e : wrow[j];
                            const bool outside = (wtap[j] == 0 && pos == 0) || (wtap[j] == 2 && pos == L - 1) ||
                                                 no_pred(wrow[j], wcol[j] + e);
                            plds_st(wreg + 4u * (uint32_t)(wl[j] + 4 * e), outside ? masked : chunk_elem<T>(wsh[j], e));
                        }
                    }
                }
            } else {
                // small workgroups: fetched here, without the head start
                const rsrc_t rs = make_rsrc(wptr(d, g));
                for (int c = (int)threadIdx.x; c < 3 * n16p; c += nthreads) {
                    const int tap = c / n16p;
                    const int idx0 = (c - tap * n16p) * E;
                    const int row = idx0 / W, col = idx0 - row * W;
                    const u32x4 v = ldg(rs, (uint32_t)((tap * HW + idx0) * (int)sizeof(T)), 0);
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const int pos = vert ? col + e : row;
                        const bool outside = (tap == 0 && pos == 0) || (tap == 2 && pos == L - 1) || no_pred(row, col + e);
                        plds_st(wreg + 4u * (uint32_t)(4 * (row * P + col + e) + tap), outside ? masked : chunk_elem<T>(v, e));
                    }
                }
            }
        } else {
            // the wave's own channels: three planes each, 3*HW elements apart per channel
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const rsrc_t rs = make_rsrc(wptr(d, c0) + (size_t)t * HW);
                u32x4 wt[NCH];
#pragma unroll
                for (int k = 0; k < NCH; ++k) {
                    u32x4 v = {0, 0, 0, 0};
                    if constexpr (WAHEAD) v = wa[t][k];
                    else if (vq[k]) v = ldg(rs, (uint32_t)(((ch[k] * 2 * HW) + (k * 64 + lane) * E) * (int)sizeof(T)), 0);
                    wt[k] = v;
                }
#pragma unroll
                for (int k = 0; k < NCH; ++k) {
                    if (vq[k]) {
                        const uint32_t o = wreg + 4u * (uint32_t)(ch[k] * 4 * HP + 4 * rc[k] + t);
#pragma unroll
                        for (int e = 0; e < E; ++e) {
                            const int pos = vert ? col0[k] + e : row0[k];
                            const bool outside = (t == 0 && pos == 0) || (t == 2 && pos == L - 1) || no_pred(row0[k], col0[k] + e);
                            plds_st(o + 16u * e, outside ? masked : chunk_elem<T>(wt[k], e));
                        }
                    }
                }
            }
        }
        // a = lam * x
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            if (vq[k]) {
                uint32_t o = ahreg + 4u * (uint32_t)(ch[k] * HP + rc[k]);
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    if constexpr (PADFLAT) {
                        plds_st(o, chunk_elem<T>(ls[k], e) * chunk_elem<T>(xs[k], e));
                        o += 4u + (((rowend[k] >> e) & 1u) ? row_pad4 : 0u) + (((chend[k] >> e) & 1u) ? ch_pad4 : 0u);
                    } else {
                        plds_st(o + 4u * e, chunk_elem<T>(ls[k], e) * chunk_elem<T>(xs[k], e));
                    }
                }
            }
        }
        // requests for after the sweep (u) and for the next direction (lam, shared weights)
        load_planes((const T*)p.u + slot_c(d) + pc, us);
        if (dn < 4) {
            load_planes((const T*)p.lam + slot_c(dn) + pc, ls);
            if constexpr (SHARED && WPRE) load_wshare(wptr(dn, g), wsh);
            if constexpr (WAHEAD) load_wahead(dn);
        }
        if constexpr (SHARED) lds_barrier();               // weights of this direction are in place (LDS only: the
                                                           // requests above stay in flight across the barrier)

        if (p.logits) {
            // Sec. 3.2 normalisation: softmax over the taps of a position that take part (the others hold -inf);
            // a line without predecessor (GSPN-local: first line of a stretch) gets three zeros
            const int nreg = SHARED ? 1 : cpw;             // weight regions: the group's, or the wave's own
            const int t0 = SHARED ? (int)threadIdx.x : lane, tn = SHARED ? nthreads : 64;
            // (padding positions are normalised like the rest: what they hold is never read)
            const float inv_hp = 1.0f / (float)HP, inv_p = 1.0f / (float)P;
            for (int idx = t0; idx < nreg * HP; idx += tn) {
                const uint32_t o = wreg + 16u * (uint32_t)idx;
                pf32x4a z = plds_ld4(o);
                const float m = fmaxf(z.y, fmaxf(z.x, z.z));
                bool none = m == -__builtin_huge_valf();
                if constexpr (LOCAL) {
                    // (row, column) of the position; the float quotients are exact at these sizes (idx < 2^16, P <= 65)
                    const int chn = (int)(((float)idx + 0.5f) * inv_hp), pos = idx - chn * HP;
                    const int row = (int)(((float)pos + 0.5f) * inv_p), col = pos - row * P;
                    none = none || ((starts >> ((vert ? row : col) & 63)) & 1ull) != 0;
                }
                const float e0 = __expf(z.x - m), e1 = __expf(z.y - m), e2 = __expf(z.z - m);
                const float r = 1.0f / (e0 + e1 + e2);
                z.x = none ? 0.f : e0 * r; z.y = none ? 0.f : e1 * r; z.z = none ? 0.f : e2 * r; z.w = 0.f;
                plds_st4(o, z);
            }
            if constexpr (SHARED) lds_barrier();
        } else if constexpr (LOCAL_PASS) {
            for (int r = 0; r < S; ++r) {
                if (!((starts >> r) & 1ull)) continue;
                for (int j = (int)threadIdx.x; j < L; j += nthreads) {
                    const uint32_t o = wreg + 16u * (uint32_t)(vert ? r * P + j : j * P + r);
                    plds_st(o, 0.f); plds_st(o + 4u, 0.f); plds_st(o + 8u, 0.f);
                }
            }
            lds_barrier();
        }

        // ---- the scan: h overwrites a
        {
            uint32_t aad = ahreg + 4u * (uint32_t)(half * HP + tpos);
            uint32_t wad = wreg + WPOS * (uint32_t)((SHARED ? 0 : half * HP) + tpos);
            float h = plds_ld(aad);                        // scan step 0: no previous line, its weights are never read
            auto taps = [&]() {
                if constexpr (W16) {
                    const u32x2 q = plds_ld2(wad);
                    return pf32x4a{word_lo<T>(q[0]), word_hi<T>(q[0]), __uint_as_float(q[1]), 0.f};
                } else {
                    return plds_ld4(wad);
                }
            };
            pf32x4a wp = taps();                           // BWD: taps of the line swept before
            // lanes past the end of the line walk the last position's operands; what they compute is never
            // stored, and the selects below keep it out of the line
            auto step = [&]() {
                aad += (uint32_t)ss4; wad += (uint32_t)((int)WPOS / 4 * ss4);
                const float av = plds_ld(aad);
                const pf32x4a w = taps();
                if constexpr (BWD) {
                    float lin = from_lane_below(wp.z * h), rin = from_lane_above(wp.x * h);
                    lin = first ? 0.f : lin;
                    rin = last ? 0.f : rin;
                    h = fmaf(wp.y, h, av) + (lin + rin);
                    wp = w;
                } else {
                    float hl = from_lane_below(h), hr = from_lane_above(h);
                    hl = first ? 0.f : hl;                 // no neighbour outside the line (its weight is stored as 0)
                    hr = last ? 0.f : hr;
                    h = fmaf(w.x, hl, fmaf(w.y, h, fmaf(w.z, hr, av)));
                }
                if (active) plds_st(aad, h);
            };
            // four steps per trip: their operand reads do not depend on h and are issued together
            int s = 1;
            for (; s + 7 < S; s += 8) { step(); step(); step(); step(); step(); step(); step(); step(); }
            for (; s + 3 < S; s += 4) { step(); step(); step(); step(); }
            for (; s < S; ++s) step();
        }

        // ---- back in the flat layout: y += u*h, optional h_save
        {
            const rsrc_t hb = make_rsrc(SAVE ? (T*)p.hs + (size_t)d * planes * HW + pc : (T*)p.y);
#pragma unroll
            for (int k = 0; k < NCH; ++k) {
                if (vq[k]) {
                    uint32_t o = ahreg + 4u * (uint32_t)(ch[k] * HP + rc[k]);
                    float hv[E];
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        if constexpr (PADFLAT) {
                            hv[e] = plds_ld(o);
                            o += 4u + (((rowend[k] >> e) & 1u) ? row_pad4 : 0u) + (((chend[k] >> e) & 1u) ? ch_pad4 : 0u);
                        } else {
                            hv[e] = plds_ld(o + 4u * e);
                        }
                        y[k][e] = fmaf(chunk_elem<T>(us[k], e), hv[e], y[k][e]);
                    }
                    if constexpr (SAVE) st_b128<CP_STREAM>(hb, flat + k * 1024, chunk_pack<T>(hv));
                }
            }
        }
        d = dn;
    }

    // merged output, rounded once
    {
        const rsrc_t yb = make_rsrc((T*)p.y + pc);
#pragma unroll
        for (int k = 0; k < NCH; ++k)
            if (vq[k]) st_b128<CP_STREAM>(yb, flat + k * 1024, chunk_pack<T>(y[k]));
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
static constexpr int FPLANE_LDS_BUDGET = 160 * 1024;

// on_cu: channels that a CU holds at a time
struct FwdPlanePlan { bool ok, flat, small, w16; int es, most_waves, most_shared, K, cpw, lsh, nwaves, pitch, shared_group, wlw, on_cu; size_t lds; };

// how often the chip is filled until a call's planes are through, `on_cu` of them on each of its 256 CUs
static long plane_rounds(const FwdParams& p, int on_cu) { return ((long)p.B * p.C + 256l * on_cu - 1) / (256l * on_cu); }

// waves per workgroup and LDS bytes, given the channels per wave and the bytes of one fp32 plane region
static bool plan_fwd_plane_waves(const FwdParams& p, FwdPlanePlan& t, size_t hp) {
    if (p.cpg == 1) {
        t.shared_group = 0;
        // per wave: cpw * (4 weight + 1 a/h) planes; of up to 4 waves per workgroup the number with which the most fit on a CU (LDS comes
        // in pieces of 1280 bytes), the larger of equals.  24576 planes of 16x16: 4 waves of 87 KB, or twice 3 of 65 KB
        const size_t wave = (size_t)t.cpw * 5 * hp;
        int best = 0;
        for (int nw = 4; nw >= 1; --nw) {
            if (p.C % (nw * t.cpw) || nw * wave > (size_t)FPLANE_LDS_BUDGET) continue;
            const int fit = (int)((size_t)FPLANE_LDS_BUDGET / ((nw * wave + 1279) / 1280 * 1280)), waves = (fit < 1 ? 1 : fit) * nw;
            const int on_cu = waves < t.most_waves ? waves : t.most_waves;
            if (on_cu > best) { best = on_cu; t.nwaves = nw; }
        }
        if (!best) return false;
        t.on_cu = best * t.cpw;
        t.K = t.nwaves * t.cpw;
        t.lds = t.nwaves * wave;
    } else {
        t.shared_group = 1;
        // The number of waves (up to 8) whose channels divide the group and of which the most fit on a CU, a smaller one only for a quarter more of
        // them (its workgroups each bring in the weights: 9216 planes 16x16 fp32 with logits, 3 waves -> 1, 22 -> 31 us) and, in fp32, where the chip
        // is then filled less often, or three times and more (1303 random calls that had the choice: 0.82 in the mean there, 1.01 elsewhere; 17280 planes
        // 14x14 with logits 39 -> 53 us, 1080 of 20x23 with h_save 53 -> 73); the flat variant's not five in six's place, which spread unevenly over
        // the four SIMDs (nine calls 1.06, 7200 planes 12x63 90 -> 113 us); weights that the largest could request a
        // direction ahead stay so.  In fp32 (flat: small maps) and with 16-bit weights in LDS; else the most waves, whose share of the weights is
        // the smallest.  Most waves -> this: 49920 planes 7x7 fp32 40 -> 30 us, 5x5 35 -> 26, 18432 of 28x28 134 -> 119; where it
        // stays: 15360 of 36x36 f16 with logits 207 -> 286, 29952 of 10x10 f16 56 -> 69.
        const int es = t.es, chunks = p.H * p.W * es / 16;
        auto ahead = [&](int nw) { return t.w16 ? chunks <= 2 * 64 * nw : 3 * chunks <= 4 * 64 * nw; };
        for (int w16 = t.w16; w16 >= 0; --w16) {
            t.w16 = w16 != 0;
            int best = 0;
            bool was_ahead = false;
            for (int nw = 8; nw >= 1; --nw) {
                const size_t lds = ((t.w16 ? 2 : 4) + (size_t)nw * t.cpw) * hp;
                if ((p.cpg / t.cpw) % nw || lds > (size_t)FPLANE_LDS_BUDGET || (t.w16 && !ahead(nw))) continue;
                if (was_ahead && !t.flat && !ahead(nw)) continue;
                const int by_lds = (int)((size_t)FPLANE_LDS_BUDGET / ((lds + 1279) / 1280 * 1280)), by_regs = t.most_shared / nw;
                const int waves = (by_lds < 1 ? 1 : by_regs < 1 ? 1 : by_lds < by_regs ? by_lds : by_regs) * nw;
                if (best && (es == 2 ? !t.w16 : t.flat && !t.small)) break;
                const bool fewer = es == 2 || !best || ((!t.flat || nw <= 4) && (plane_rounds(p, best * t.cpw) > 2 || plane_rounds(p, best * t.cpw) > plane_rounds(p, waves * t.cpw)));
                if (!best || (fewer && 4 * waves >= 5 * best)) { best = waves; t.nwaves = nw; t.K = nw * t.cpw; t.lds = lds; was_ahead = !t.flat && ahead(nw); }
            }
            if (best) { t.on_cu = best * t.cpw; break; }
            if (!w16) return false;
        }
    }
    return (size_t)p.B * (p.C / t.K) <= 0x7fffffffull;
}

// padded planes (rows of whole 16-byte chunks), one or two channels per wave
static FwdPlanePlan plan_fwd_plane_padded(const FwdParams& p, int es) {
    FwdPlanePlan t = {};
    const int HW = p.H * p.W, m = p.H > p.W ? p.H : p.W;
    t.cpw = m <= 32 ? 2 : 1;
    // Weights of each channel's own: the channels that four chunks per lane hold.  The registers then hold their weights a direction ahead, where eight
    // chunks per lane waited for the memory three times per direction, on four waves per CU.  6144 planes 28x28 fp32 100 -> 80 us (with
    // logits 134 -> 96), 8448 of 36x32 f16 (backward) 393 -> 260, 32256 of 19x16 f16 344 -> 128; 0.60 in the mean of 1110 calls.
    t.small = p.cpg == 1 && HW * es <= 4096;
    if (t.small && 2 * HW * es > 4096) t.cpw = 1;
    if ((size_t)t.cpw * HW * es > 8192) {
        if (t.cpw == 2 && (size_t)HW * es <= 8192) t.cpw = 1; else return t;
    }
    if (p.cpg == 1 ? p.C % t.cpw : p.cpg % t.cpw) t.cpw = 1;
    t.lsh = t.cpw == 2 ? 5 : 6;
    t.pitch = p.W | 1;
    t.most_waves = es == 4 ? (t.small ? 12 : 8) : t.small ? 8 : 4;      // (registers, weights of each channel's own)
    const size_t hp = (((size_t)p.H * t.pitch + 3) & ~(size_t)3) * sizeof(float);   // one plane region in LDS
    // 16-bit weights that the scan takes as they are stay 16-bit in LDS
    t.es = es; t.most_shared = 8;
    t.w16 = es == 2 && p.cpg > 1 && p.kchunk <= 0 && !p.logits;
    t.ok = plan_fwd_plane_waves(p, t, hp);
    return t;
}
// flat planes: the most channels per wave (each on 64 / cpw lanes) that are whole 16 B chunks together
static FwdPlanePlan plan_fwd_plane_flat(const FwdParams& p, int es) {
    FwdPlanePlan t = {};
    const int HW = p.H * p.W, m = p.H > p.W ? p.H : p.W;
    t.flat = true;
    int lsh = 3;
    while ((1 << lsh) < m) ++lsh;
    for (; lsh <= 6; ++lsh) {
        const int cpw = 64 >> lsh;
        if ((size_t)cpw * HW * es % 16 || (size_t)cpw * HW * es > 8192) continue;
        if (p.cpg == 1 ? p.C % cpw : p.cpg % cpw) continue;
        t.cpw = cpw; t.lsh = lsh;
        break;
    }
    if (!t.cpw) return t;
    // small maps (at most four 16 B chunks per lane) get an odd pitch like the padded variant; larger ones keep rows packed
    t.small = (size_t)t.cpw * HW * es <= 4 * 64 * 16;
    t.pitch = t.small ? (p.W | 1) : p.W;
    t.most_waves = !t.small ? 8 : es == 4 ? 16 : 12;
    t.es = es; t.most_shared = t.most_waves;
    // shared weights: the widest request that divides a group's block (its start is a multiple of its size)
    const size_t wblock = (size_t)3 * HW * es;
    t.wlw = wblock % 16 == 0 ? 16 : wblock % 8 == 0 ? 8 : wblock % 4 == 0 ? 4 : 2;
    t.ok = plan_fwd_plane_waves(p, t, t.small ? (((size_t)p.H * t.pitch + 3) & ~(size_t)3) * sizeof(float) : (size_t)HW * sizeof(float));
    return t;
}

// Rows of whole chunks take the padded variant, but for small maps, whose lines leave most lanes of its waves idle (up to 16 positions: two channels
// per wave where four or eight have their place) or, in fp32 with shared weights, whose chunks need half of its registers, in calls that
// fill the chip with it more often than with the flat one: what that gains is channels per CU, and what it costs is that the weights are
// waited for in each direction.  Both timed on 1480 random calls: 0.78 in the mean where the chip is filled less often, 1.13 where as
// often (up to 4096 planes of two channels per wave; 2048 planes 20x20 fp32 17.6 against 25 us, 2624 of 16x16 f16 13.5 against 21.6).
// us: 36864 planes 8x8 bf16, forward 103 -> 44, 45312 of 11x8 fp32 134 -> 49, 73728 of 16x16 bf16 with logits 248 -> 167.  Workgroups of
// five and more waves, which wait for each other, in place of such as need not, 1.03 (5120 planes 9x4 fp32 25 against 21); a wave that
// fetches a group's weights by itself, beyond 340 pixels 1.04 (8896 planes 25x20 fp32 60 against 76).
// Beyond the lines: 24x24 f16 48 -> 60, 25x28 fp32 63 -> 76.  Weights of each channel's own: up to 128 pixels in 16 bits (5x8 36 us for 105,
// 16x8 26 for 32; 13x16 60 for 46, 15x16 30 for 14), 80 in fp32 (10x8 71 for 78; 12x12 28 for 24.5, with stretches 36 for 42).
static FwdPlanePlan plan_fwd_plane(const FwdParams& p, int dtype) {
    const int es = dtype == 0 ? 4 : 2, m = p.H > p.W ? p.H : p.W;
    if (p.H < 2 || p.W < 2 || p.H > 64 || p.W > 64) return FwdPlanePlan{};
    if (p.xt) return FwdPlanePlan{};                       // transposed-horizontal layout: tile and generic kernels
    if (p.W % (16 / es)) return plan_fwd_plane_flat(p, es);
    const bool shared_f32 = dtype == 0 && p.cpg > 1;
    const FwdPlanePlan padded = plan_fwd_plane_padded(p, es);
    if (m <= 16 || shared_f32) {
        const FwdPlanePlan t = plan_fwd_plane_flat(p, es);
        const bool size = t.ok && t.small && (t.cpw > 2 || (shared_f32 && t.cpw == 2)) && (p.cpg > 1 || p.H * p.W <= (es == 2 ? 128 : p.kchunk > 0 ? 144 : 80));
        const bool waits = size && p.cpg > 1 && (t.nwaves == 1 ? p.H * p.W > 340 : t.nwaves >= 5 && padded.nwaves <= (es == 2 ? 2 : 1));
        if (size && padded.ok && !waits && plane_rounds(p, t.on_cu) < plane_rounds(p, padded.on_cu)) return t;
    }
    return padded;
}

bool fwd_plane_applicable(const FwdParams& p, int dtype) { return plan_fwd_plane(p, dtype).ok; }

template <typename T, bool SAVE, bool SHARED, bool WPRE, bool FLAT, bool LOCAL, bool BWD, int NCH, bool W16 = false>
static hipError_t launch_fplane_kn(const FwdPlaneArgs& a, const FwdPlanePlan& t, hipStream_t s) {
    auto k = fwd_plane_kernel<T, SAVE, SHARED, WPRE, FLAT, LOCAL, BWD, NCH, W16>;
    hipError_t e = allow_dynamic_lds((const void*)k, FPLANE_LDS_BUDGET);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)((size_t)a.p.B * (a.p.C / a.K))), block(64 * a.nwaves);
    hipLaunchKernelGGL(k, grid, block, t.lds, s, a);
    return hipGetLastError();
}

template <typename T, bool SAVE, bool SHARED, bool WPRE, bool FLAT, bool LOCAL, bool BWD = false>
static hipError_t launch_fplane_kl(const FwdPlaneArgs& a, const FwdPlanePlan& t, hipStream_t s) {
    if constexpr (WPRE && !LOCAL && sizeof(T) == 2) {
        if (t.w16) return launch_fplane_kn<T, SAVE, SHARED, WPRE, FLAT, LOCAL, BWD, 8, true>(a, t, s);
    }
    if constexpr (FLAT || !SHARED) {
        if (t.small) return launch_fplane_kn<T, SAVE, SHARED, WPRE, FLAT, LOCAL, BWD, 4>(a, t, s);
    }
    return launch_fplane_kn<T, SAVE, SHARED, WPRE, FLAT, LOCAL, BWD, 8>(a, t, s);
}

template <typename T, bool SAVE, bool SHARED, bool WPRE, bool FLAT>
static hipError_t launch_fplane_k(const FwdPlaneArgs& a, const FwdPlanePlan& t, hipStream_t s) {
    return a.p.kchunk > 0 ? launch_fplane_kl<T, SAVE, SHARED, WPRE, FLAT, true>(a, t, s)
                          : launch_fplane_kl<T, SAVE, SHARED, WPRE, FLAT, false>(a, t, s);
}

template <typename T, bool SAVE, bool SHARED>
static hipError_t launch_fplane(const FwdPlaneArgs& a, const FwdPlanePlan& t, hipStream_t s) {
    if (t.flat) return launch_fplane_k<T, SAVE, SHARED, false, true>(a, t, s);
    if constexpr (SHARED) {
        const int E = 16 / (int)sizeof(T);
        const bool wpre = t.w16 || 3 * (a.p.H * a.p.W / E) <= 4 * 64 * a.nwaves;   // WSH chunks per thread
        return wpre ? launch_fplane_k<T, SAVE, true, true, false>(a, t, s)
                    : launch_fplane_k<T, SAVE, true, false, false>(a, t, s);
    } else {
        return launch_fplane_k<T, SAVE, false, false, false>(a, t, s);
    }
}

template <typename T>
static hipError_t launch_fplane_t(const FwdPlaneArgs& a, const FwdPlanePlan& t, hipStream_t s) {
    if (a.p.hs) return t.shared_group ? launch_fplane<T, true, true>(a, t, s) : launch_fplane<T, true, false>(a, t, s);
    return t.shared_group ? launch_fplane<T, false, true>(a, t, s) : launch_fplane<T, false, false>(a, t, s);
}

// reverse sweep (first pass of the two-pass backward scan): the same choice of variant, state always saved
template <typename T, bool SHARED, bool WPRE, bool FLAT>
static hipError_t launch_fplane_rev_k(const FwdPlaneArgs& a, const FwdPlanePlan& t, hipStream_t s) {
    return a.p.kchunk > 0 ? launch_fplane_kl<T, true, SHARED, WPRE, FLAT, true, true>(a, t, s)
                          : launch_fplane_kl<T, true, SHARED, WPRE, FLAT, false, true>(a, t, s);
}
template <typename T, bool SHARED>
static hipError_t launch_fplane_rev(const FwdPlaneArgs& a, const FwdPlanePlan& t, hipStream_t s) {
    if (t.flat) return launch_fplane_rev_k<T, SHARED, false, true>(a, t, s);
    if constexpr (SHARED) {
        const int E = 16 / (int)sizeof(T);
        const bool wpre = t.w16 || 3 * (a.p.H * a.p.W / E) <= 4 * 64 * a.nwaves;   // WSH chunks per thread
        return wpre ? launch_fplane_rev_k<T, true, true, false>(a, t, s) : launch_fplane_rev_k<T, true, false, false>(a, t, s);
    } else {
        return launch_fplane_rev_k<T, false, false, false>(a, t, s);
    }
}

bool reverse_sweep_plane_applicable(const FwdParams& p, int dtype) { return plan_fwd_plane(p, dtype).ok; }

// p holds gy as x, u as lam, lam as u, gx as y and the buffer that receives e as hs
hipError_t launch_reverse_sweep_plane(const FwdParams& p, int dtype, hipStream_t s) {
    const FwdPlanePlan t = plan_fwd_plane(p, dtype);
    if (!t.ok || !p.hs) return hipErrorInvalidValue;
    FwdPlaneArgs a;
    a.p = p; a.K = t.K; a.cpw = t.cpw; a.lsh = t.lsh; a.nwaves = t.nwaves; a.pitch = t.pitch; a.wlw = t.wlw;
    for (int d = 0; d < 4; ++d) a.seg[d] = stretch_start_bits(d < 2 ? p.H : p.W, d & 1, p.kchunk, false);
    if (dtype == 0) return t.shared_group ? launch_fplane_rev<float, true>(a, t, s) : launch_fplane_rev<float, false>(a, t, s);
    if (dtype == 2) return t.shared_group ? launch_fplane_rev<f16_t, true>(a, t, s) : launch_fplane_rev<f16_t, false>(a, t, s);
    return t.shared_group ? launch_fplane_rev<bf16_t, true>(a, t, s) : launch_fplane_rev<bf16_t, false>(a, t, s);
}

hipError_t launch_fwd_plane(const FwdParams& p, int dtype, hipStream_t s) {
    const FwdPlanePlan t = plan_fwd_plane(p, dtype);
    if (!t.ok) return hipErrorInvalidValue;
    FwdPlaneArgs a;
    a.p = p; a.K = t.K; a.cpw = t.cpw; a.lsh = t.lsh; a.nwaves = t.nwaves; a.pitch = t.pitch; a.wlw = t.wlw;
    for (int d = 0; d < 4; ++d) a.seg[d] = stretch_start_bits(d < 2 ? p.H : p.W, d & 1, p.kchunk, false);
    if (dtype == 2) return launch_fplane_t<f16_t>(a, t, s);
    return dtype == 0 ? launch_fplane_t<float>(a, t, s) : launch_fplane_t<bf16_t>(a, t, s);
}

}  // namespace gspn

// For the tests, not part of the ABI: {flat variant, channels per wave, waves per workgroup, channels on a CU at a time} of the plane kernel's
// forward call, 0 where it does not take the shape.
extern "C" int gspn_plane_shape(int B, int C, int H, int W, int G, int kchunk, int logits, int dtype, int* shape) {
    gspn::FwdParams p = {};
    p.B = B; p.C = C; p.H = H; p.W = W; p.G = G; p.cpg = C / G; p.mask = 15; p.kchunk = kchunk; p.logits = logits;
    const gspn::FwdPlanePlan t = gspn::plan_fwd_plane(p, dtype);
    shape[0] = t.flat; shape[1] = t.cpw; shape[2] = t.nwaves; shape[3] = t.on_cu;
    return t.ok;
}
