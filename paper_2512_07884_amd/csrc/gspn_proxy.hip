// Compressive proxy projections (Sec. 4.2, "Compressive Proxy Dimension"): the 1x1 convolutions over the channel
// axis that take x from C channels down to C_proxy before the scan and back up to C after it,
//
//     out[b][m][n] = sum_k P[m][k] * in[b][k][n]        n = pixel (h*W + w), contiguous
//
// i.e. per image a dense [M x K] by [K x N] product with N = H*W: down-projection M = C_proxy, K = C; back up
// M = C, K = C_proxy.  This is the one dense contraction around the scan, so it runs on the matrix cores in bf16
// (v_mfma_f32_32x32x16_bf16, or 32x32x8 when K is not a multiple of 16; fp32 accumulation); with C_proxy << C it moves far more bytes than it computes and
// is bound by reading `in` (down) or writing `out` (up) once.
//
// Mapping: one wave owns a tile of 32 output channels x 256 pixels.  The MFMA wants both operands packed along
// k, while `in` is contiguous along n: each lane loads, for its k-rows (lanes 0-31 the first half of the k-step,
// lanes 32-63 the second), 16 B = 8 consecutive pixels (a wave reads whole 512 B row segments), and regroups them in registers
// with byte permutes into eight k-packed B operands, one per pixel of its eight.  Eight MFMAs per k-step then give
// each lane, per output row it holds, eight consecutive pixels: the result leaves as 16 B stores of whole segments.
// Where that leaves too few waves (1152 -> 144 channels on two 64x64 images: 160 waves of 72 dependent k-steps) the four
// waves of a workgroup take every fourth k-step of a narrower tile (128 pixels) and add their sums through LDS in wave order.
// N not a multiple of 8: the same kernels with requests at element alignment; the last lane of a row takes its last eight
// (four) pixels, some of them a second time (same sum, same bytes stored).
// What the MFMA path does not take (fp32 storage, K not a multiple of 8, fewer than 8 pixels) runs a plain FMA kernel.
#include "gspn_unaligned.hpp"

namespace gspn {

namespace {

typedef short bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef _Float16 f16x4_t __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));

// one 32x32 matrix-core step over 8 / 16 k values of 16-bit operands (T = bf16_t or f16_t; the two formats share the
// operand layout), fp32 accumulation
template <typename T> __device__ __forceinline__ f32x16_t mfma_k8(const u32x2& a, const u32x2& b, const f32x16_t& c) {
    if constexpr (__is_same(T, f16_t)) return __builtin_amdgcn_mfma_f32_32x32x8f16(__builtin_bit_cast(f16x4_t, a), __builtin_bit_cast(f16x4_t, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(__builtin_bit_cast(bf16x4_t, a), __builtin_bit_cast(bf16x4_t, b), c, 0, 0, 0);
}
template <typename T> __device__ __forceinline__ f32x16_t mfma_k16(const u32x4& a, const u32x4& b, const f32x16_t& c) {
    if constexpr (__is_same(T, f16_t)) return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// NB bytes (16 or 8) of a row at p: ANY = p is aligned to its element only
template <typename T, int NB, bool ANY> __device__ __forceinline__ void ld_row(const T* p, uint32_t* r) {
    if constexpr (NB == 16) {
        u32x4 v;
        if constexpr (ANY) v = rg_load(p); else v = *(const u32x4*)p;
        r[0] = v[0]; r[1] = v[1]; r[2] = v[2]; r[3] = v[3];
    } else {
        typedef uint32_t any8 __attribute__((ext_vector_type(2), aligned(2)));
        u32x2 v;
        if constexpr (ANY) v = *(const any8*)p; else v = *(const u32x2*)p;
        r[0] = v.x; r[1] = v.y;
    }
}
template <typename T, int NB, bool ANY> __device__ __forceinline__ void st_row(T* p, const uint32_t* r) {
    if constexpr (NB == 16) {
        const u32x4 v = {r[0], r[1], r[2], r[3]};
        if constexpr (ANY) rg_store(p, v); else *(u32x4*)p = v;
    } else {
        typedef uint32_t any8 __attribute__((ext_vector_type(2), aligned(2)));
        const u32x2 v = {r[0], r[1]};
        if constexpr (ANY) *(any8*)p = v; else *(u32x2*)p = v;
    }
}

// one 16x16 step over 32 k values (the small tiles of the weight gradient)
typedef float f32x4_t __attribute__((ext_vector_type(4)));
template <typename T> __device__ __forceinline__ f32x4_t mfma16_k32(const u32x4& a, const u32x4& b, const f32x4_t& c) {
    if constexpr (__is_same(T, f16_t)) return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// KS = k values per MFMA: 8 (v_mfma_f32_32x32x8_bf16_1k) or 16 (v_mfma_f32_32x32x16_bf16, K a multiple of 16).
// A lane feeds KS/2 consecutive k: lanes 0-31 the first half of the k-step, lanes 32-63 the second.
// PT: the matrix is applied transposed, out[b][m][n] = sum_k P[k][m] * in[b][k][n] with P stored [K][M] (the gradient of
// the projection w.r.t. its input): a lane then gathers its KS/2 values of P with 2-byte loads a row apart (P is small
// and stays in cache).
// SPLIT = 1: a wave owns 32 rows x 256 pixels.  SPLIT = 4: a workgroup owns 32 rows x 128 pixels, its waves every fourth
// k-step (1152 -> 144 on two 64x64 images 58 -> 18 us).  MT = 2 (SPLIT = 4): two row tiles of the same pixels, `in` requested and
// regrouped once for both, P^T a pair of rows per request (17 -> 14, P^T 18 -> 12; same sums, bit for bit).  ANY: rows of `in` / `out`
// start at any element.  BUF: buffer requests and stores with 32-bit offsets; lanes beyond the row request nothing.
template <typename T, int KS, bool PT, int SPLIT, int MT, bool ANY, bool BUF>
__global__ void __launch_bounds__(256) proxy_mfma_kernel(const T* __restrict__ in, const T* __restrict__ P,
                                                         T* __restrict__ out, int B, int K, int M, int N,
                                                         int ntiles, int mtiles) {
    constexpr int KL = KS / 2;                                 // k-rows per lane and k-step
    constexpr int PX = SPLIT == 1 ? 8 : 4;                     // pixels per lane
    constexpr int NB = PX * 2;
    constexpr int DEPTH = SPLIT == 1 ? 1 : 3;                  // k-steps requested ahead
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // work item -> (image, pixel tile, row tile), row tile fastest: the waves of a workgroup (SPLIT = 4: neighbouring
    // workgroups) take the row tiles of one pixel tile (they read the same `in`, which then comes out of the caches) or,
    // with a single row tile, neighbouring pixel tiles
    const long item = SPLIT == 1 ? (long)blockIdx.x * 4 + wave : (long)xcd_contiguous_item(blockIdx.x, gridDim.x);
    const long per_image = (long)ntiles * mtiles;
    if (item >= (long)B * per_image) return;                   // (whole waves; whole workgroups where the waves meet)
    const int b = (int)(item / per_image);
    const int rem = (int)(item - (long)b * per_image);
    const int nt = rem / mtiles, mt = rem - nt * mtiles;
    const int jl = lane & 31, kh = lane >> 5;                  // pixel group of the lane, which half of the k-step
    const int n_raw = nt * (32 * PX) + jl * PX;                // first of the lane's pixels
    const bool n_ok = n_raw < N;
    const int n_lane = n_ok ? min(n_raw, N - PX) : 0;          // a row's last lane: its last PX pixels
    // row of P this lane feeds as the A operand; MT = 2: and the 32nd after it, or (PT: one request for both) the next
    constexpr int MY = MT == 2 && PT ? 1 : 32, MJ = MT == 2 && PT ? 2 : 1;
    const int m_lane = mt * (32 * MT) + MJ * jl;

    static_assert(!BUF || (SPLIT == 1 && !ANY), "buffer requests: whole rows, a wave per tile");
    const T* src = in + (size_t)b * K * N + n_lane;
    const rsrc_t inb = make_rsrc(in + (size_t)b * K * N), ob = make_rsrc(out + (size_t)b * M * N);
    const rsrc_t pb = make_rsrc(P);
    f32x16_t acc[MT][PX];
#pragma unroll
    for (int y = 0; y < MT; ++y)
#pragma unroll
        for (int v = 0; v < PX; ++v)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[y][v][r] = 0.f;

    struct Step { uint32_t q[KL][NB / 4]; uint32_t pa[MT][KL / 2]; };         // the lane's k-rows of `in`; P[m_lane][its k values]
    auto fetch = [&](int k0, Step& t) {
        const int kr = k0 + KL * kh;
#pragma unroll
        for (int kk = 0; kk < KL; ++kk) {
            if constexpr (BUF) {
                u32x4 v = {0, 0, 0, 0};
                if (n_ok) v = __builtin_amdgcn_raw_buffer_load_b128(inb, (uint32_t)(((size_t)(kr + kk) * N + n_lane) * 2), 0, 0);
                t.q[kk][0] = v.x; t.q[kk][1] = v.y; t.q[kk][2] = v.z; t.q[kk][3] = v.w;
            } else {
                ld_row<T, NB, ANY>(src + (size_t)(kr + kk) * N, t.q[kk]);      // (spare lanes: pixel 0)
            }
        }
        if constexpr (MT == 2 && PT) {                         // (M is even)
#pragma unroll
            for (int i = 0; i < KL / 2; ++i) {
                uint32_t lo = 0, hi = 0;
                if (m_lane < M) {
                    lo = __builtin_amdgcn_raw_buffer_load_b32(pb, (uint32_t)(((size_t)(kr + 2 * i) * M + m_lane) * 2), 0, 0);
                    hi = __builtin_amdgcn_raw_buffer_load_b32(pb, (uint32_t)(((size_t)(kr + 2 * i + 1) * M + m_lane) * 2), 0, 0);
                }
                t.pa[0][i] = lo; t.pa[MT - 1][i] = hi;         // (taken apart where they are multiplied)
            }
            return;
        }
#pragma unroll
        for (int y = 0; y < MT; ++y) {
            const int m = m_lane + MY * y;
#pragma unroll
            for (int i = 0; i < KL / 2; ++i) t.pa[y][i] = 0;
            if (m < M && PT) {
#pragma unroll
                for (int i = 0; i < KL / 2; ++i) {
                    const uint32_t lo = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(pb, (uint32_t)(((size_t)(kr + 2 * i) * M + m) * 2), 0, 0);
                    const uint32_t hi = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(pb, (uint32_t)(((size_t)(kr + 2 * i + 1) * M + m) * 2), 0, 0);
                    t.pa[y][i] = (lo & 0xffffu) | (hi << 16);
                }
            } else if (m < M) {
                const uint32_t po = (uint32_t)(((size_t)m * K + kr) * 2);
                if constexpr (KS == 8) { const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(pb, po, 0, 0); t.pa[y][0] = v.x; t.pa[y][1] = v.y; }
                else { const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(pb, po, 0, 0); t.pa[y][0] = v.x; t.pa[y][1] = v.y; t.pa[y][2] = v.z; t.pa[y][3] = v.w; }
            }
        }
    };
    auto multiply = [&](Step& t) {
        if constexpr (MT == 2 && PT) {
#pragma unroll
            for (int i = 0; i < KL / 2; ++i) {
                const uint32_t lo = t.pa[0][i], hi = t.pa[MT - 1][i];
                t.pa[0][i] = __builtin_amdgcn_perm(hi, lo, 0x05040100u); t.pa[MT - 1][i] = __builtin_amdgcn_perm(hi, lo, 0x07060302u);
            }
        }
#pragma unroll
        for (int v = 0; v < PX; ++v) {
            // pixel v of the lane's, its k values packed in pairs: element v sits in word v/2, half v%2
            const uint32_t sel = (v & 1) ? 0x07060302u : 0x05040100u;
            uint32_t bb[KL / 2];
#pragma unroll
            for (int i = 0; i < KL / 2; ++i) bb[i] = __builtin_amdgcn_perm(t.q[2 * i + 1][v >> 1], t.q[2 * i][v >> 1], sel);
#pragma unroll
            for (int y = 0; y < MT; ++y) {
                if constexpr (KS == 8) {
                    const u32x2 av = {t.pa[y][0], t.pa[y][1]}, bv = {bb[0], bb[1]};
                    acc[y][v] = mfma_k8<T>(av, bv, acc[y][v]);
                } else {
                    const u32x4 av = {t.pa[y][0], t.pa[y][1], t.pa[y][2], t.pa[y][3]}, bv = {bb[0], bb[1], bb[2], bb[3]};
                    acc[y][v] = mfma_k16<T>(av, bv, acc[y][v]);
                }
            }
        }
    };
    // the operands of the next k-steps are requested before the current one is multiplied (past the end the last
    // step is requested again: redundant, in bounds, never multiplied)
    const int last = K - KS;
    const int k_first = SPLIT == 1 ? 0 : wave * KS;
    constexpr int HOP = KS * SPLIT;
    if constexpr (DEPTH == 1) {
        Step cur, nxt;
        fetch(0, cur);
        for (int k0 = 0; k0 < K; k0 += KS) {
            fetch(min(k0 + KS, last), nxt);
            multiply(cur);
            cur = nxt;
        }
    } else {
        Step s0, s1, s2;
        fetch(min(k_first, last), s0);
        fetch(min(k_first + HOP, last), s1);
        for (int k0 = k_first; k0 < K; k0 += 3 * HOP) {
            fetch(min(k0 + 2 * HOP, last), s2);
            multiply(s0);
            fetch(min(k0 + 3 * HOP, last), s0);
            if (k0 + HOP < K) multiply(s1);
            fetch(min(k0 + 4 * HOP, last), s1);
            if (k0 + 2 * HOP < K) multiply(s2);
        }
    }

    // accumulator register r of a lane: output row 8*(r/4) + 4*(lane/32) + r%4 of the tile, column = the lane's pixel
    T* dst = out + (size_t)b * M * N + n_lane;
    if constexpr (SPLIT == 1) {
        if (!n_ok) return;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int m = mt * 32 + 8 * (r >> 2) + 4 * kh + (r & 3);
            if (m < M) {
                const uint32_t o[4] = {pack_word<T>(acc[0][0][r], acc[0][1][r]), pack_word<T>(acc[0][2][r], acc[0][3][r]),
                                       pack_word<T>(acc[0][4][r], acc[0][5][r]), pack_word<T>(acc[0][6][r], acc[0][7][r])};
                if constexpr (BUF) st_b128(ob, (uint32_t)(((size_t)m * N + n_lane) * 2), u32x4{o[0], o[1], o[2], o[3]});
                else st_row<T, NB, ANY>(dst + (size_t)m * N, o);
            }
        }
    } else {
        __shared__ float red[SPLIT][16][PX][64];
#pragma unroll
        for (int y = 0; y < MT; ++y) {
            if (y) __syncthreads();                            // the row tile before has been read
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int v = 0; v < PX; ++v) red[wave][r][v][lane] = acc[y][v][r];
            __syncthreads();
            // each wave adds and stores a quarter of the rows
#pragma unroll
            for (int i = 0; i < 16 / SPLIT; ++i) {
                const int r = wave * (16 / SPLIT) + i;
                const int m = mt * (32 * MT) + MY * y + MJ * (8 * (r >> 2) + 4 * kh + (r & 3));
                if (m < M && n_ok) {
                    float t[PX];
#pragma unroll
                    for (int v = 0; v < PX; ++v) {
                        t[v] = red[0][r][v][lane];
#pragma unroll
                        for (int w = 1; w < SPLIT; ++w) t[v] += red[w][r][v][lane];
                    }
                    const uint32_t o[2] = {pack_word<T>(t[0], t[1]), pack_word<T>(t[2], t[3])};
                    st_row<T, NB, ANY>(dst + (size_t)m * N, o);
                }
            }
        }
    }
}

// any shape, any storage type: one thread per pixel, eight output channels at a time
template <typename T, bool PT = false>
__global__ void __launch_bounds__(256) proxy_fma_kernel(const T* __restrict__ in, const T* __restrict__ P, T* __restrict__ out,
                                                        int B, int K, int M, int N) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long)B * N) return;
    const int b = (int)(idx / N), n = (int)(idx - (long)b * N);
    const T* x = in + (size_t)b * K * N + n;
    T* y = out + (size_t)b * M * N + n;
    for (int m0 = 0; m0 < M; m0 += 8) {
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int k = 0; k < K; ++k) {
            const float xv = ldf(x + (size_t)k * N);
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (m0 + j < M) acc[j] = fmaf(ldf(PT ? P + (size_t)k * M + (m0 + j) : P + (size_t)(m0 + j) * K + k), xv, acc[j]);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (m0 + j < M) stf(y + (size_t)(m0 + j) * N, acc[j]);
    }
}

// ---- gradient w.r.t. the matrix: gP[m][k] = sum over b, n of gout[b][m][n] * in[b][k][n] ----------------------------
// Both operands are contiguous along the contraction axis n, which is what the matrix cores want.  One workgroup per
// (image, 32 x 32 tile of gP); its NW waves take interleaved 16-pixel steps of n and add their accumulators through
// LDS in wave order; the per-image sums go to the caller's workspace and a small kernel adds the images in order, so the
// result does not depend on scheduling.  NW = 8 where four waves per tile would leave the chip short of loads in flight.
// Whole rows: buffer requests, rows past the end request nothing.  ANY: rows start at any element; a
// wave takes four neighbouring steps (whole 128-byte lines of the rows) and the step that crosses the end of the rows takes
// the last eight pixels and moves them down, zeros behind them.  (Neighbouring steps and global requests on whole rows were
// measured slower: 1152 -> 288 on four 96x96 images 171 -> 185 us.)  For short rows and few tiles (launch_gradw_as).
template <typename T, int NW, bool ANY>
__global__ void __launch_bounds__(64 * NW) proxy_gradw_mfma_kernel(const T* __restrict__ gout, const T* __restrict__ in,
                                                               float* __restrict__ partial, int K, int M, int N,
                                                               int mtiles, int ktiles) {
    __shared__ float red[NW][16][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int per_image = mtiles * ktiles;
    const int b = blockIdx.x / per_image;
    const int rem = blockIdx.x - b * per_image;
    const int mt = rem / ktiles, kt = rem - mt * ktiles;
    const int jl = lane & 31, nh = lane >> 5;                  // row of the operand this lane feeds; which 8 of the 16 pixels
    const int m_lane = mt * 32 + jl, k_lane = kt * 32 + jl;
    const rsrc_t gb = make_rsrc(gout + ((size_t)b * M + mt * 32) * N);           // the tile's rows of gout / of in
    const rsrc_t xb = make_rsrc(in + ((size_t)b * K + kt * 32) * N);
    const uint32_t row_off = (uint32_t)((size_t)jl * N * 2);
    // (ANY: rows past the end are read as the last row, their sums are not stored)
    const T* ga = gout + ((size_t)b * M + min(m_lane, M - 1)) * N;
    const T* ib = in + ((size_t)b * K + min(k_lane, K - 1)) * N;
    f32x16_t acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    // four 16-pixel steps per trip: their loads are requested together (steps past the end load nothing and multiply zeros)
    constexpr int HOP = ANY ? 16 : 16 * NW;
    for (int n0 = wave * (ANY ? 64 : 16); n0 < N; n0 += 64 * NW) {
        u32x4 av[4], bv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int n = n0 + HOP * q + 8 * nh;
            av[q] = u32x4{0, 0, 0, 0}; bv[q] = u32x4{0, 0, 0, 0};
            if constexpr (!ANY) {
                const uint32_t off = row_off + (uint32_t)(n * 2);
                if (m_lane < M && n < N) av[q] = __builtin_amdgcn_raw_buffer_load_b128(gb, off, 0, 0);
                if (k_lane < K && n < N) bv[q] = __builtin_amdgcn_raw_buffer_load_b128(xb, off, 0, 0);
            } else if (n < N) {
                const int nl = min(n, N - 8);
                ld_row<T, 16, true>(ga + nl, (uint32_t*)&av[q]);
                ld_row<T, 16, true>(ib + nl, (uint32_t*)&bv[q]);
            }
        }
        if (ANY && n0 + 64 > N) {                              // the end of the rows (a uniform branch)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + 16 * q + 8 * nh;
                const int sh = n < N ? max(n - (N - 8), 0) : 0;
                av[q] = rg_realign<T>(av[q], sh);
                bv[q] = rg_realign<T>(bv[q], sh);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) acc = mfma_k16<T>(av[q], bv[q], acc);
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[r];
    __syncthreads();
    // accumulator register r of a lane: row 8*(r/4) + 4*(lane/32) + r%4 of the tile (m), column lane%32 (k)
    for (int idx = threadIdx.x; idx < 16 * 64; idx += 64 * NW) {
        const int r = idx >> 6, l = idx & 63;
        float v = red[0][r][l];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += red[w][r][l];
        const int m = mt * 32 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3), k = kt * 32 + (l & 31);
        if (m < M && k < K) partial[((size_t)b * M + m) * K + k] = v;
    }
}

// The same with the rows through LDS.  A matrix-core operand is 16 bytes of each of 32 rows: asked for as it is multiplied, a request
// touches 32 lines for a quarter of each.  Here a request is eight rows of whole 128-byte lines; 128 pixels of the tile's rows make a
// stage, the stages after it are on their way in registers, and each of the eight waves multiplies every eighth step of 16 pixels, in
// the order of the kernel above with eight waves (on whole rows its sums, bit for bit; launches of 512 tiles and more have four there).
// 1152 x 144 on two 64x64 images 30 -> 18 us, on 16 of 28x28 32.7 -> 29.5 (in stages of 256 pixels 37).  Every tile of the longer side is read by as many workgroups as the
// shorter side has tiles, and each XCD has an L2 of its own: an XCD takes neighbouring tiles of the longer side with all of the
// shorter one's.
template <typename T, bool ANY>
__global__ void __launch_bounds__(512) proxy_gradw_tile_kernel(const T* __restrict__ gout, const T* __restrict__ in,
                                                              float* __restrict__ partial, int K, int M, int N,
                                                              int mtiles, int ktiles) {
    constexpr int ROWS = 64, PITCH = 256 + 16, AHEAD = 3;
    __shared__ __attribute__((aligned(16))) char stage[2 * ROWS * PITCH];                // (the sums of the waves pass through it at the end)
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int per_image = mtiles * ktiles, item = (int)xcd_contiguous_item(blockIdx.x, gridDim.x);
    const int b = item / per_image, rem = item - b * per_image;
    const int mt = mtiles <= ktiles ? rem % mtiles : rem / ktiles, kt = mtiles <= ktiles ? rem / mtiles : rem % ktiles;
    // this thread's pieces: row threadIdx / 16 of every 32, pixels 8 * (threadIdx % 16) of the stage (rows past the end are read as the
    // last row, their sums are not stored)
    const int r0 = threadIdx.x >> 4, c0 = (threadIdx.x & 15) * 8;
    const T* const gr = gout + ((size_t)b * M + min(mt * 32 + r0, M - 1)) * N;
    const T* const xr = in + ((size_t)b * K + min(kt * 32 + r0, K - 1)) * N;
    struct Piece { u32x4 g, x; };
    const int nstages = (N + 127) / 128;
    auto fetch = [&](int s, Piece& p) {
        const int n = min(s, nstages - 1) * 128 + c0, nl = min(n, N - 8);        // (beyond the rows' end: their last eight pixels)
        ld_row<T, 16, ANY>(gr + nl, (uint32_t*)&p.g);
        ld_row<T, 16, ANY>(xr + nl, (uint32_t*)&p.x);
    };
    char* const place = stage + r0 * PITCH + c0 * 2;
    auto put = [&](int s, Piece& p) {
        const int n = s * 128 + c0;
        if (s == nstages - 1) {                                                  // (uniform) what lies beyond the rows counts as 0
            const int sh = min(max(n - (N - 8), 0), 8);
            if constexpr (ANY) { p.g = rg_realign<T>(p.g, sh); p.x = rg_realign<T>(p.x, sh); }
            if (sh >= 8) p.g = p.x = u32x4{0, 0, 0, 0};
        }
        *(u32x4*)(place + (s & 1) * ROWS * PITCH) = p.g;
        *(u32x4*)(place + ((s & 1) * ROWS + 32) * PITCH) = p.x;
    };
    f32x16_t acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    const char* const from = stage + (lane & 31) * PITCH + wave * 32 + (lane >> 5) * 16;
    auto multiply = [&](int s) {
        const char* f = from + (s & 1) * ROWS * PITCH;
        acc = mfma_k16<T>(*(const u32x4*)f, *(const u32x4*)(f + 32 * PITCH), acc);
    };
    Piece p[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) fetch(i, p[i]);
    put(0, p[0]);
    fetch(AHEAD, p[0]);
    lds_barrier();
    for (int s0 = 0; s0 < nstages; s0 += AHEAD) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int s = s0 + i;
            if (s < nstages) {
                if (s + 1 < nstages) put(s + 1, p[(i + 1) % AHEAD]);
                fetch(s + 1 + AHEAD, p[(i + 1) % AHEAD]);
                multiply(s);
                lds_barrier();
            }
        }
    }
    float (*const red)[16][64] = (float (*)[16][64])stage;
    static_assert(sizeof(float) * 8 * 16 * 64 <= sizeof(stage), "");
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[r];
    __syncthreads();
    for (int idx = threadIdx.x; idx < 16 * 64; idx += 512) {
        const int r = idx >> 6, l = idx & 63;
        float v = red[0][r][l];
#pragma unroll
        for (int w = 1; w < 8; ++w) v += red[w][r][l];
        const int m = mt * 32 + 8 * (r >> 2) + 4 * (l >> 5) + (r & 3), k = kt * 32 + (l & 31);
        if (m < M && k < K) partial[((size_t)b * M + m) * K + k] = v;
    }
}

// The same with the rows through LDS, in tiles of 16 MT x 16 KT (v_mfma_f32_16x16x32).  A matrix-core operand is 16 bytes of each of 16
// rows: asked for as it is multiplied, a request touches 16 lines for a part of each.  Here a request is two rows of 512 bytes, whole lines;
// 256 pixels of the tile's rows make a stage, the stages after it are on their way in registers (three or four: 96 to 144 KB per CU, which is
// what a CU's rate goes by), and each of the eight waves multiplies the whole tile over every eighth step of 32 pixels.  Bound by what a
// CU takes in: 50 to 60 KB per us, of some 75 that its L1 passes on.  1152 x 144 on two 64x64 images 24 -> 15.5 us, on one 128x128 70 -> 23.5, 48 x 768
// on two of 44x101 22.0 -> 15.8 (with 32 x 32 tiles, stages of 128 pixels and two fewer of them on their way: the figures before).
// Every tile of the longer side is read by as many workgroups as the shorter side has tiles, and each XCD has an L2 of its own: an XCD takes
// neighbouring tiles of the longer side with all of the shorter one's.
// ranges = 2: two workgroups per tile and image, the second of which leaves its half of the pixels' sums in gP.
template <typename T, bool ANY, int MT, int KT>
__global__ void __launch_bounds__(512, MT + KT <= 4 ? 4 : 2) proxy_gradw_lds_kernel(const T* __restrict__ gout, const T* __restrict__ in,
                                                              float* __restrict__ partial, float* __restrict__ gP, int K, int M, int N,
                                                              int mtiles, int ktiles, int ranges) {
    constexpr int NP = MT + KT, ROWS = 16 * NP, PX = 256, PITCH = PX * 2 + 16, AHEAD = NP <= 4 ? 3 : 4;
    extern __shared__ __attribute__((aligned(16))) char stage[];                         // (the sums of the waves pass through it at the end)
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int per_image = mtiles * ktiles;
    int rem = (int)xcd_contiguous_item(blockIdx.x, gridDim.x);
    const int br = rem / per_image;                            // image and range of its pixels
    rem -= br * per_image;
    const int b = br / ranges, range = br - b * ranges;
    const int mt = mtiles <= ktiles ? rem % mtiles : rem / ktiles, kt = mtiles <= ktiles ? rem / mtiles : rem % ktiles;
    const int nstages = (N + PX - 1) / PX, s_begin = range * nstages / ranges, s_end = (range + 1) * nstages / ranges;
    // this thread's pieces: row threadIdx / 32 of every 16, pixels 8 * (threadIdx % 32) of the stage (rows past the end are read as the
    // last row, their sums are not stored)
    const int r0 = threadIdx.x >> 5, c0 = (threadIdx.x & 31) * 8;
    const T* row[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        if (i < MT) row[i] = gout + ((size_t)b * M + min((mt * MT + i) * 16 + r0, M - 1)) * N;
        else row[i] = in + ((size_t)b * K + min((kt * KT + i - MT) * 16 + r0, K - 1)) * N;
    }
    struct Piece { u32x4 v[NP]; };
    auto fetch = [&](int s, Piece& p) {
        const int nl = min(min(s, s_end - 1) * PX + c0, N - 8);                  // (beyond the rows' end: their last eight pixels)
#pragma unroll
        for (int i = 0; i < NP; ++i) ld_row<T, 16, ANY>(row[i] + nl, (uint32_t*)&p.v[i]);
    };
    char* const place = stage + r0 * PITCH + c0 * 2;
    auto put = [&](int s, Piece& p) {
        if (s == nstages - 1) {                                                  // (uniform) what lies beyond the rows counts as 0
            const int sh = min(max(s * PX + c0 - (N - 8), 0), 8);
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                if constexpr (ANY) p.v[i] = rg_realign<T>(p.v[i], sh);
                if (sh >= 8) p.v[i] = u32x4{0, 0, 0, 0};
            }
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) *(u32x4*)(place + ((s & 1) * ROWS + 16 * i) * PITCH) = p.v[i];
    };
    f32x4_t acc[MT][KT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int k = 0; k < KT; ++k) acc[m][k] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const char* const from = stage + (lane & 15) * PITCH + wave * 64 + (lane >> 4) * 16;
    auto multiply = [&](int s) {
        const char* const f = from + (s & 1) * ROWS * PITCH;
        u32x4 v[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) v[i] = *(const u32x4*)(f + 16 * i * PITCH);
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int k = 0; k < KT; ++k) acc[m][k] = mfma16_k32<T>(v[m], v[MT + k], acc[m][k]);
    };
    Piece p[AHEAD];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) fetch(s_begin + i, p[i]);
    put(s_begin, p[0]);
    fetch(s_begin + AHEAD, p[0]);
    lds_barrier();
    for (int s0 = s_begin; s0 < s_end; s0 += AHEAD) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int s = s0 + i;
            if (s < s_end) {
                if (s + 1 < s_end) put(s + 1, p[(i + 1) % AHEAD]);
                fetch(s + 1 + AHEAD, p[(i + 1) % AHEAD]);
                multiply(s);
                lds_barrier();
            }
        }
    }
    float (*const red)[MT * KT * 4][64] = (float (*)[MT * KT * 4][64])stage;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int k = 0; k < KT; ++k)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[wave][(m * KT + k) * 4 + r][lane] = acc[m][k][r];
    __syncthreads();
    float* const to = range == 0 ? partial + (size_t)b * M * K : gP;
    for (int idx = threadIdx.x; idx < MT * KT * 256; idx += 512) {
        const int r = idx >> 6, l = idx & 63, t = r >> 2;
        float v = red[0][r][l];
#pragma unroll
        for (int w = 1; w < 8; ++w) v += red[w][r][l];
        const int m = (mt * MT + t / KT) * 16 + 4 * (l >> 4) + (r & 3), k = (kt * KT + t % KT) * 16 + (l & 15);
        if (m < M && k < K) to[(size_t)m * K + k] = v;
    }
}

// The same in tiles of 16 x 16 (v_mfma_f32_16x16x32: 32 pixels per step, lane l feeds row l % 16 and pixels 8 * (l / 16) ..),
// sixteen waves each, for calls whose 32 x 32 tiles are fewer than a quarter of the CUs: a tile's rows are read by one CU,
// whose request rate is then what bounds the call (24 <- 96 channels on two 78x117 images: 6 tiles, 44 us -> 24 tiles, 19 us).
template <typename T, bool ANY>
__global__ void __launch_bounds__(1024) proxy_gradw_small_kernel(const T* __restrict__ gout, const T* __restrict__ in,
                                                                 float* __restrict__ partial, int K, int M, int N,
                                                                 int mtiles, int ktiles) {
    constexpr int NW = 16;
    __shared__ float red[NW][4][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int per_image = mtiles * ktiles;
    const int b = blockIdx.x / per_image;
    const int rem = blockIdx.x - b * per_image;
    const int mt = rem / ktiles, kt = rem - mt * ktiles;
    const int jl = lane & 15, nq = lane >> 4;
    // rows past the end are read as the last row (their sums are not stored)
    const T* ga = gout + ((size_t)b * M + min(mt * 16 + jl, M - 1)) * N;
    const T* ib = in + ((size_t)b * K + min(kt * 16 + jl, K - 1)) * N;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    for (int n0 = wave * 128; n0 < N; n0 += 128 * NW) {
        u32x4 av[4], bv[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int n = n0 + 32 * q + 8 * nq;
            av[q] = u32x4{0, 0, 0, 0}; bv[q] = u32x4{0, 0, 0, 0};
            if (n < N) {
                const int nl = ANY ? min(n, N - 8) : n;
                ld_row<T, 16, ANY>(ga + nl, (uint32_t*)&av[q]);
                ld_row<T, 16, ANY>(ib + nl, (uint32_t*)&bv[q]);
            }
        }
        if (ANY && n0 + 128 > N) {                             // the end of the rows (a uniform branch)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + 32 * q + 8 * nq;
                const int sh = n < N ? max(n - (N - 8), 0) : 0;
                av[q] = rg_realign<T>(av[q], sh);
                bv[q] = rg_realign<T>(bv[q], sh);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) acc = mfma16_k32<T>(av[q], bv[q], acc);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wave][r][lane] = acc[r];
    __syncthreads();
    // accumulator register r of a lane: row 4*(lane/16) + r of the tile (m), column lane%16 (k)
    if (threadIdx.x < 256) {
        const int r = threadIdx.x >> 6, l = threadIdx.x & 63;
        float v = red[0][r][l];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += red[w][r][l];
        const int m = mt * 16 + 4 * (l >> 4) + r, k = kt * 16 + (l & 15);
        if (m < M && k < K) partial[((size_t)b * M + m) * K + k] = v;
    }
}

// any shape, any storage type: a workgroup owns 8 rows x 32 columns of gP for one image and walks n in chunks of 64
// staged through LDS (coalesced loads along n; pitch 65 keeps the per-thread walks conflict-free)
template <typename T>
__global__ void __launch_bounds__(256) proxy_gradw_fma_kernel(const T* __restrict__ gout, const T* __restrict__ in,
                                                              float* __restrict__ partial, int K, int M, int N,
                                                              int mtiles, int ktiles) {
    __shared__ float gs[8][65], xs[32][65];
    const int per_image = mtiles * ktiles;
    const int b = blockIdx.x / per_image;
    const int rem = blockIdx.x - b * per_image;
    const int mt = rem / ktiles, kt = rem - mt * ktiles;
    const int tm = threadIdx.x >> 5, tk = threadIdx.x & 31;    // this thread's element of the tile
    const int col = threadIdx.x & 63, row4 = threadIdx.x >> 6; // loader: pixel inside the chunk, row group
    float acc = 0.f;
    for (int n0 = 0; n0 < N; n0 += 64) {
        const int n = n0 + col;
#pragma unroll
        for (int r = row4; r < 8; r += 4) {
            const int m = mt * 8 + r;
            gs[r][col] = (m < M && n < N) ? ldf(gout + ((size_t)b * M + m) * N + n) : 0.f;
        }
#pragma unroll
        for (int r = row4; r < 32; r += 4) {
            const int k = kt * 32 + r;
            xs[r][col] = (k < K && n < N) ? ldf(in + ((size_t)b * K + k) * N + n) : 0.f;
        }
        __syncthreads();
#pragma unroll 8
        for (int j = 0; j < 64; ++j) acc = fmaf(gs[tm][j], xs[tk][j], acc);
        __syncthreads();
    }
    const int m = mt * 8 + tm, k = kt * 32 + tk;
    if (m < M && k < K) partial[((size_t)b * M + m) * K + k] = acc;
}

// gP = the per-image sums added in image order
__global__ void __launch_bounds__(256) proxy_gradw_sum_kernel(const float* __restrict__ partial, float* __restrict__ gP, int B, int MK) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= MK) return;
    float v = 0.f;
    // sixteen images requested at a time (the loads do not depend on the sum), then added in order
    for (int b0 = 0; b0 < B; b0 += 16) {
        float t[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) t[j] = b0 + j < B ? partial[(size_t)(b0 + j) * MK + i] : 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) if (b0 + j < B) v += t[j];
    }
    gP[i] = v;
}
// ... of one image, the sums of whose second half of pixels are in gP
__global__ void __launch_bounds__(256) proxy_gradw_halves_kernel(float* __restrict__ partial, float* __restrict__ gP, int MK) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= MK) return;
    const float v = partial[i] + gP[i];
    partial[i] = v; gP[i] = v;
}

}  // namespace

// 16-bit rows of any length from eight pixels up (those that are not a multiple of eight with requests at element alignment:
// 24 <- 96 channels on two 78x117 images, FMA kernels -> these: forward 165 -> 11, input gradient 141 -> 11, weight gradient
// 492 -> 19 us); 32-bit byte offsets inside P
bool proxy_mfma_applicable(int K, int M, int N, int dtype) {
    return dtype != 0 && K % 8 == 0 && N >= 8 && (size_t)M * K * 2 < (1ull << 31);
}

template <typename T, int KS, bool PT, int SPLIT, int MT = 1>
static hipError_t launch_project_mfma(const void* in, const void* P, void* out, int B, int K, int M, int N, hipStream_t s) {
    constexpr int tile = SPLIT == 1 ? 256 : 128;
    const int ntiles = (N + tile - 1) / tile, mtiles = (M + 32 * MT - 1) / (32 * MT);
    const long items = (long)B * ntiles * mtiles, blocks = SPLIT == 1 ? (items + 3) / 4 : items;
    if (blocks > 0x7fffffffl) return hipErrorInvalidValue;
    void (*k)(const T*, const T*, T*, int, int, int, int, int, int);
    if (N % 8 != 0) k = proxy_mfma_kernel<T, KS, PT, SPLIT, MT, true, false>;
    else k = proxy_mfma_kernel<T, KS, PT, SPLIT, MT, false, false>;
    if constexpr (SPLIT == 1) {
        // Whole rows: buffer requests for P^T (with global ones 18 -> 20 us at 24 -> 1152 channels on two 128x128 images), for
        // steps of 8 (8 -> 1152 there 14.6 -> 15.8) and from four waves per CU on (from memory: 144 -> 192 on 64 images 28x28
        // 21.1 -> 22.3, 288 -> 768 on 64 of 32x32 84 -> 88).  With fewer waves the lanes' own addresses serve better (144 -> 192
        // on eight 64x64 images 17.0 -> 14.8, 288 -> 1152 on two 56x56 24.8 -> 20.6), and they reach images beyond 2^31 bytes.
        const bool fits = (size_t)K * N * 2 < (1ull << 31) && (size_t)M * N * 2 < (1ull << 31);
        if (N % 8 == 0 && fits && (PT || KS == 8 || items >= 1024)) k = proxy_mfma_kernel<T, KS, PT, 1, 1, false, true>;
    }
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(256), 0, s, (const T*)in, (const T*)P, (T*)out, B, K, M, N, ntiles, mtiles);
    return hipGetLastError();
}

// out = P in (PT = false) or P^T in (PT = true: the gradient w.r.t. the projection's input) in storage type T
template <typename T, bool PT>
static hipError_t launch_project_as(const void* in, const void* P, void* out, int B, int K, int M, int N, bool mfma, hipStream_t s) {
    // a launch counts its threads in 32 bits (what is beyond is cut off without an error): very many images go in several
    const unsigned long long image = mfma ? 64ull * ((N + 255) / 256) * ((M + 31) / 32) : (unsigned long long)N;
    const unsigned long long most = ((1ull << 32) - 512) / image;
    if ((unsigned long long)B > most) {
        if (most < 1) return hipErrorInvalidValue;
        for (long b0 = 0; b0 < B; b0 += (long)most) {
            const int n = (int)(B - b0 < (long)most ? B - b0 : (long)most);
            const hipError_t e = launch_project_as<T, PT>((const T*)in + (size_t)b0 * K * N, P, (T*)out + (size_t)b0 * M * N, n, K, M, N, mfma, s);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    if constexpr (sizeof(T) == 2) {
        if (mfma) {
            // The waves of a workgroup share the k-steps where one wave per tile would leave the chip short of waves and the
            // chain is long: the longer the chain, the more waves that takes.  Measured, plain -> shared: 1152 -> 144 on two
            // 64x64 images (160 waves, 72 steps) 58 -> 18 us; 288 -> 384 on eight 28x28 (384 waves, 18 steps) 15.0 -> 11.4;
            // 1152 -> 288 on four 64x64 (576, 72) 61 -> 45.  Beyond the lines sharing loses: 384 -> 24 on eight 128x128 (512,
            // 24) from memory 42 -> 46; 288 -> 768 on 32 images 14x14 (768, 18) 16.7 -> 22.7; 768 -> 8 on 64 images 56x56 (832,
            // 48) from memory 118 -> 122; 768 -> 96 on 32 images 64x64 (1536, 48) 56 -> 65; 144 -> 192 on eight 56x56 (624, 9)
            // 11 -> 15.
            const long waves = (long)B * ((N + 255) / 256) * ((M + 31) / 32);
            const int steps = K / (K % 16 == 0 ? 16 : 8);
            const bool split = (waves <= 448 && steps >= 16) || (waves <= 768 && steps >= 48);
            // A workgroup of pairs of row tiles reads `in` once for 64 rows, a compute unit holds one of them (registers) and two of the
            // others: pairs where they take fewer turns of 256 workgroups.  1152 -> 144 on two 64x64 images (192 for 320) 16.9 -> 13.9 us,
            // P^T 18.1 -> 12.4; 768 -> 144 on three of 60x60 (261 for 435: two turns either way) 12.9 -> 13.8, 13.7 -> 16.9.  More
            // than one turn pays for P^T only, whose requests they halve as well: 1152 -> 144 on one 128x128 (384 for 640) 29.3 ->
            // 21.9, 1152 -> 288 on four 64x64 (640 for 1152) 43.3 -> 31.9; P 24.1 -> 25.5, 36.6 -> 36.4.
            const long ntiles = (long)B * ((N + 127) / 128), single = ntiles * ((M + 31) / 32), pairs = ntiles * ((M + 63) / 64);
            const bool paired = split && (PT ? M % 2 == 0 : pairs <= 256) && (pairs + 255) / 256 < (single + 255) / 256;
            if (paired) return K % 16 == 0 ? launch_project_mfma<T, 16, PT, 4, 2>(in, P, out, B, K, M, N, s) : launch_project_mfma<T, 8, PT, 4, 2>(in, P, out, B, K, M, N, s);
            if (K % 16 == 0) return split ? launch_project_mfma<T, 16, PT, 4>(in, P, out, B, K, M, N, s) : launch_project_mfma<T, 16, PT, 1>(in, P, out, B, K, M, N, s);
            return split ? launch_project_mfma<T, 8, PT, 4>(in, P, out, B, K, M, N, s) : launch_project_mfma<T, 8, PT, 1>(in, P, out, B, K, M, N, s);
        }
    }
    const long threads = (long)B * N;
    if ((threads + 255) / 256 > 0x7fffffffl) return hipErrorInvalidValue;
    const dim3 grid((unsigned)((threads + 255) / 256)), block(256);
    hipLaunchKernelGGL((proxy_fma_kernel<T, PT>), grid, block, 0, s, (const T*)in, (const T*)P, (T*)out, B, K, M, N);
    return hipGetLastError();
}

hipError_t launch_proxy_project(const void* in, const void* P, void* out, int B, int K, int M, int N, int dtype,
                                hipStream_t s) {
    const bool mfma = proxy_mfma_applicable(K, M, N, dtype);
    if (dtype == 0) return launch_project_as<float, false>(in, P, out, B, K, M, N, false, s);
    if (dtype == 1) return launch_project_as<bf16_t, false>(in, P, out, B, K, M, N, mfma, s);
    return launch_project_as<f16_t, false>(in, P, out, B, K, M, N, mfma, s);
}

template <typename T, int MT, int KT>
static hipError_t launch_gradw_lds(const void* gout, const void* in, float* partial, float* gP, int B, int K, int M, int N, int ranges, hipStream_t s) {
    const int mt = (M + 16 * MT - 1) / (16 * MT), kt = (K + 16 * KT - 1) / (16 * KT);
    constexpr int stages = 2 * 16 * (MT + KT) * (256 * 2 + 16), sums = 8 * MT * KT * 256 * 4, lds = stages > sums ? stages : sums;
    void (*k)(const T*, const T*, float*, float*, int, int, int, int, int, int) = N % 8 ? proxy_gradw_lds_kernel<T, true, MT, KT> : proxy_gradw_lds_kernel<T, false, MT, KT>;
    const hipError_t e = allow_dynamic_lds((const void*)k, 160 * 1024);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((unsigned)((long)B * ranges * mt * kt)), dim3(512), lds, s, (const T*)gout, (const T*)in, partial, gP, K, M, N, mt, kt, ranges);
    return hipGetLastError();
}

// The weight gradient's kernel for 16-bit storage: its tile in units of 16 rows and the ranges of pixels that are summed apart.
// apart: `partial` and gP share no memory.
enum GradwKernel { GRADW_PLAIN = 0, GRADW_SMALL = 1, GRADW_LDS = 2, GRADW_TILE = 3 };
struct GradwPlan { GradwKernel kernel; int mt, kt, ranges; };

// The tile of the kernel with stages of 256 pixels: what a CU takes in, rows per tile times turns of 256 workgroups, is what the time goes
// by.  32 x 32 has two workgroups on a CU, which hide each other's start and end (0.75 of that); 64 x 64 nearly runs out of registers (1.15).
// us with 32 x 32, 48 x 32, 48 x 48, 64 x 64: 144 x 1152 on two 64x64 images 18.3 15.3 17.6 22.6; 48 x 1152 on 14 images 72x81
// 66 56 65 48, on six of 105x48 22.4 18.8 21.3 27.2; 144 x 768 on four of 118x18 18.7 25.2 17.7 22.3.  Rows of less than
// eight stages are not worth a second start.  One image leaves `partial` a single place: its second half's sums go to gP on the way
// (144 x 1152 channels on 128x128 32.7 -> 28.6 us, 24 <- 192 on 123x49 23.2 -> 16.3), unless that is the same place.
static GradwPlan gradw_stages(int B, int K, int M, int N, bool apart, long* wgs) {
    GradwPlan p = {GRADW_LDS, 2, 2, B == 1 && apart ? 2 : 1};
    const int shapes[][2] = {{2, 2}, {3, 2}, {2, 3}, {3, 3}, {4, 4}};
    long best = -1;
    for (const auto& t : shapes) {
        const long n = (long)B * p.ranges * ((M + 16 * t[0] - 1) / (16 * t[0])) * ((K + 16 * t[1] - 1) / (16 * t[1])), turns = (n + 255) / 256;
        const bool pair = t[0] == 2 && t[1] == 2;
        if (!pair && turns > 1 && N < 2048) continue;
        const long cost = turns * (t[0] + t[1]) * (pair && turns > 1 ? 75 : t[0] == 4 ? 115 : 100);
        if (best < 0 || cost < best) { best = cost; p.mt = t[0]; p.kt = t[1]; *wgs = n; }
    }
    return p;
}

// Where the rows are long they pass through LDS in stages of 256 pixels, elsewhere by the kernel that the products had before it.  The four
// timed on 19 600 random products of 512 pixels and more (2 to 1400 channels, 1 to 64 images; graph replays): what it takes 0.80 of the time of the
// kernel in its place in the mean, 1 in a hundred above 1.05; the others would take 1.13, 1.02 and 1.04 with it.
//   In place of the 16 x 16 tiles (there where 32 x 32 ones are fewer than a quarter of the CUs and the rows are long: two images, 8 <- 96 channels on
// 96x96 26.8 -> 17.0 us; below 4096 pixels no gain in the mean and up to 7 % lost: 48 <- 96 on 56x56 16.1 -> 17.2; rows at any element from
// 1024 pixels on 0.94): odd rows, half of whose requests fall between 32-bit words and are worked off in twice the time (24 <- 192 on four
// images 89x111 52 -> 32 us), from 3072 pixels on with more than ten channels on the smaller side (0.71), 5120 with more than 16 on the larger (0.88;
// up to 16 1.1, shorter rows 1.2); of one image sooner.  Whole words: of one image only (0.80; several 1.3 to 1.5).
//   In place of the 32 x 32 tiles with stages of 128 pixels, four of which a CU holds (2048 pixels and 16 tiles, 1024 and 64, 512 and 256; a single tile
// on one side rows at any element from 1024 pixels on, whole ones from 4096 and 256 tiles on; timed against the kernel without LDS on 4900
// products, 0.6 to 0.83): fewer and longer stages lose where the rows are short or many workgroups queue.  Granules: one turn of the CUs 0.75,
// more from 2560 pixels on with a larger tile (0.81), 4096 with 32 x 32 (0.95; below 1.1: 144 x 1152 on 16 images 28x28 29.5 against 37 us).  Other even
// rows: from 2560 pixels on (one turn 0.84), 3072 with a larger tile (0.81), 5632 with 32 x 32 (0.93; below 1.1 to 1.3).  Odd rows: from 2560 on
// with a larger tile (0.78), 8192 with 32 x 32 (0.95; below 1.0 to 1.4).  Of one image from 2048 pixels on, with whole granules any.
//   In place of the kernel without LDS: from 2049 pixels on with more than 16 channels on the smaller side (0.67), 64 workgroups or one image (0.78;
// others 1.09); shorter rows of more than 16 channels from 1409 pixels on (0.86), odd ones from 833 (0.83; shorter ones 1.06 to 1.2).
static GradwPlan gradw_plan(int B, int K, int M, int N, bool apart) {
    GradwPlan p = {GRADW_PLAIN, 2, 2, 1};
    const int mtiles = (M + 31) / 32, ktiles = (K + 31) / 32, fewer = M < K ? M : K, more = M < K ? K : M;
    const long tiles = (long)B * mtiles * ktiles;
    if (N < 512 || tiles > 0x7fffff) return p;                 // (a launch counts its threads in 32 bits)
    const bool odd = N % 2 != 0, granules = N % 8 == 0;
    long wgs = 0;
    const GradwPlan stages = gradw_stages(B, K, M, N, apart, &wgs);
    const bool pair = stages.mt == 2 && stages.kt == 2;
    bool take;
    if (tiles < 64 && N >= (granules ? 4096 : 1024)) {
        p.kernel = GRADW_SMALL; p.mt = p.kt = 1;
        take = B == 1 ? (odd ? N > 3072 || fewer > 16 : N > 5120 && fewer > 16) : odd && more > 16 && ((fewer > 10 && N > 3072) || N > 5120);
    } else if (mtiles > 1 && ktiles > 1 ? (N >= 2048 && tiles >= 16) || (N >= 1024 && tiles >= 64) || tiles >= 256
                                        : granules ? N >= 4096 && tiles >= 256 : N >= 1024) {
        p.kernel = GRADW_TILE;
        take = N >= (B == 1 ? (granules ? 0 : 2048)
                   : granules ? (wgs <= 256 ? 0 : pair ? 4096 : 2560)
                   : odd ? (pair ? 8192 : 2560) : wgs <= 256 ? 2560 : pair ? 5632 : 3072);
    } else {
        take = N > 2048 ? fewer > 16 || wgs > 64 || B == 1 : fewer > 16 && (N > 1408 || (odd && N > 832));
    }
    return take && tiles <= 0x3fffff ? stages : p;
}

// per-image sums of gout in^T into `partial` (B*M*K floats), storage type T; halves: of one image, the sums of its second half into gP
template <typename T>
static hipError_t launch_gradw_as(const void* gout, const void* in, float* partial, float* gP, bool* halves, int B, int K, int M, int N, hipStream_t s) {
    const bool mfma = sizeof(T) == 2 && N >= 8;
    const int mtiles = mfma ? (M + 31) / 32 : (M + 7) / 8;
    const int ktiles = (K + 31) / 32;
    if constexpr (sizeof(T) == 2) {
        const size_t MK = (size_t)M * K;
        const GradwPlan t = gradw_plan(B, K, M, N, gP + MK <= partial || partial + MK <= gP);
        if (t.kernel == GRADW_SMALL) {
            const int mt = (M + 15) / 16, kt = (K + 15) / 16;
            void (*k)(const T*, const T*, float*, int, int, int, int, int) = N % 8 ? proxy_gradw_small_kernel<T, true> : proxy_gradw_small_kernel<T, false>;
            hipLaunchKernelGGL(k, dim3((unsigned)((long)B * mt * kt)), dim3(1024), 0, s, (const T*)gout, (const T*)in, partial, K, M, N, mt, kt);
            return hipGetLastError();
        }
        if (t.kernel == GRADW_TILE) {
            void (*k)(const T*, const T*, float*, int, int, int, int, int) = N % 8 ? proxy_gradw_tile_kernel<T, true> : proxy_gradw_tile_kernel<T, false>;
            hipLaunchKernelGGL(k, dim3((unsigned)((long)B * mtiles * ktiles)), dim3(512), 0, s, (const T*)gout, (const T*)in, partial, K, M, N, mtiles, ktiles);
            return hipGetLastError();
        }
        if (t.kernel == GRADW_LDS) {
            *halves = t.ranges == 2;
            const int ranges = t.ranges;
            return t.mt == 4 ? launch_gradw_lds<T, 4, 4>(gout, in, partial, gP, B, K, M, N, ranges, s)
                 : t.mt == 3 ? (t.kt == 3 ? launch_gradw_lds<T, 3, 3>(gout, in, partial, gP, B, K, M, N, ranges, s) : launch_gradw_lds<T, 3, 2>(gout, in, partial, gP, B, K, M, N, ranges, s))
                             : (t.kt == 3 ? launch_gradw_lds<T, 2, 3>(gout, in, partial, gP, B, K, M, N, ranges, s) : launch_gradw_lds<T, 2, 2>(gout, in, partial, gP, B, K, M, N, ranges, s));
        }
    }
    const long blocks = (long)B * mtiles * ktiles;
    if (blocks > 0x7fffffffl) return hipErrorInvalidValue;
    const bool wide = blocks * 4 < 2048;     // eight waves per tile while four would leave a compute unit under eight
    if constexpr (sizeof(T) == 2) {
        if (mfma) {
            const bool any = N % 8 != 0 || (size_t)N * 2 * 64 >= (1ull << 31);         // (whole rows: 32-bit offsets within a tile's rows)
            void (*k)(const T*, const T*, float*, int, int, int, int, int) =
                wide ? (any ? proxy_gradw_mfma_kernel<T, 8, true> : proxy_gradw_mfma_kernel<T, 8, false>)
                     : (any ? proxy_gradw_mfma_kernel<T, 4, true> : proxy_gradw_mfma_kernel<T, 4, false>);
            hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(wide ? 512 : 256), 0, s, (const T*)gout, (const T*)in, partial, K, M, N, mtiles, ktiles);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL(proxy_gradw_fma_kernel<T>, dim3((unsigned)blocks), dim3(256), 0, s, (const T*)gout, (const T*)in,
                       partial, K, M, N, mtiles, ktiles);
    return hipGetLastError();
}

// Gradients of the projection (chain rule on the sum above): gin = P^T gout per pixel (storage type, may be NULL) and
// gP = sum over images and pixels of gout in^T (fp32 [M, K], may be NULL; `partial` = B*M*K floats of the caller's).
hipError_t launch_proxy_project_bwd(const void* gout, const void* in, const void* P, void* gin, float* gP, float* partial,
                                    int B, int K, int M, int N, int dtype, hipStream_t s) {
    if (gin) {
        // the forward kernels with the matrix read transposed: K output channels, contraction over the M channels of gout
        const bool mfma = proxy_mfma_applicable(M, K, N, dtype);
        const hipError_t e = dtype == 0 ? launch_project_as<float, true>(gout, P, gin, B, M, K, N, false, s)
                           : dtype == 1 ? launch_project_as<bf16_t, true>(gout, P, gin, B, M, K, N, mfma, s)
                                        : launch_project_as<f16_t, true>(gout, P, gin, B, M, K, N, mfma, s);
        if (e != hipSuccess) return e;
    }
    if (gP) {
        if (!partial) return hipErrorInvalidValue;
        bool halves = false;
        hipError_t e = dtype == 0 ? launch_gradw_as<float>(gout, in, partial, gP, &halves, B, K, M, N, s)
                     : dtype == 1 ? launch_gradw_as<bf16_t>(gout, in, partial, gP, &halves, B, K, M, N, s)
                                  : launch_gradw_as<f16_t>(gout, in, partial, gP, &halves, B, K, M, N, s);
        if (e != hipSuccess) return e;
        const int MK = M * K;
        if (halves) hipLaunchKernelGGL(proxy_gradw_halves_kernel, dim3((unsigned)((MK + 255) / 256)), dim3(256), 0, s, partial, gP, MK);
        else hipLaunchKernelGGL(proxy_gradw_sum_kernel, dim3((unsigned)((MK + 255) / 256)), dim3(256), 0, s, partial, gP, B, MK);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ---- the same call for callers that cannot allocate (HIP graph capture, serving loops): the per-image sums go to a
// static device array instead of a workspace of the caller's.  Each GPU the library runs on holds its own copy of the
// array at its own address; the array's name is only a host-side handle, so the address is looked up once per device
// and that pointer is what the kernels get.
static __device__ __align__(256) float scratch[PROXY_SCRATCH_FLOATS];

static hipError_t scratch_address(float** out) {
    constexpr int MAX_DEVICES = 64;
    static float* per_device[MAX_DEVICES] = {};
    static std::mutex mu;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(mu);
    if (!per_device[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));      // with device `dev` current: this device's copy
        if (e != hipSuccess) return e;
        per_device[dev] = (float*)p;
    }
    *out = per_device[dev];
    return hipSuccess;
}

// Every element [b][m][k] of the workspace is overwritten by the first kernel before the second reads it, so the array
// needs no clearing between calls; calls that overlap on one GPU (two streams) would race on it.
hipError_t launch_proxy_project_bwd_static(const void* gout, const void* in, const void* P, void* gin, float* gP,
                                           int B, int K, int M, int N, int dtype, hipStream_t s) {
    float* partial = nullptr;
    if (gP) {
        if ((size_t)B * M * K > PROXY_SCRATCH_FLOATS) return hipErrorInvalidValue;     // checked by the caller
        const hipError_t e = scratch_address(&partial);
        if (e != hipSuccess) return e;
    }
    return launch_proxy_project_bwd(gout, in, P, gin, gP, partial, B, K, M, N, dtype, s);
}

}  // namespace gspn

// For the tests, not part of the ABI: the kernel (0 rows from memory, 1 16 x 16 tiles, 2 and 3 rows through LDS in stages of 256 and 128 pixels), the rows and columns of its tile
// and the ranges of pixels of the weight gradient in 16-bit storage; apart: `partial` and gP share no memory.
extern "C" void gspn_proxy_gradw_shape(int B, int K, int M, int H, int W, int apart, int* shape) {
    const gspn::GradwPlan t = gspn::gradw_plan(B, K, M, H * W, apart != 0);
    shape[0] = t.kernel; shape[1] = 16 * t.mt; shape[2] = 16 * t.kt; shape[3] = t.ranges;
}
