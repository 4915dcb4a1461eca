// 16-byte requests at element alignment, for tensors whose rows start anywhere (odd widths).  gfx950's memory pipe takes
// them as they are: a vertical scan of 100 x 168 rows costs 16 % less than one of 100 x 167.
#pragma once
#include "gspn_tile_common.hpp"

namespace gspn {

template <typename T> struct ElemAligned16 {
    typedef uint32_t type __attribute__((ext_vector_type(4), aligned(2)));     // 16 bytes at element alignment
};
template <> struct ElemAligned16<float> {
    typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4)));
};
template <typename T> __device__ __forceinline__ u32x4 rg_load(const T* p) {
    return *(const typename ElemAligned16<T>::type*)p;
}
template <typename T> __device__ __forceinline__ void rg_store(T* p, u32x4 v) {
    *(typename ElemAligned16<T>::type*)p = v;
}
// A 16-byte granule whose 16-byte window was moved into the tensor by s elements (first or last granule of a tensor only):
// element e of the granule is at index e + s of what was loaded.  Elements outside the tensor are never used.
template <typename T> __device__ __forceinline__ u32x4 rg_realign(u32x4 v, int s) {
#pragma unroll 1
    for (int i = 0; i < 16 / (int)sizeof(T) - 1; ++i) {
        u32x4 r = v, l = v;
        if constexpr (sizeof(T) == 4) {
            r = u32x4{v[1], v[2], v[3], 0u};
            l = u32x4{0u, v[0], v[1], v[2]};
        } else {
            r = u32x4{(v[0] >> 16) | (v[1] << 16), (v[1] >> 16) | (v[2] << 16), (v[2] >> 16) | (v[3] << 16), v[3] >> 16};
            l = u32x4{v[0] << 16, (v[0] >> 16) | (v[1] << 16), (v[1] >> 16) | (v[2] << 16), (v[2] >> 16) | (v[3] << 16)};
        }
        const bool right = s > i, left = -s > i;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = right ? r[k] : (left ? l[k] : v[k]);
    }
    return v;
}

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

}  // namespace gspn
