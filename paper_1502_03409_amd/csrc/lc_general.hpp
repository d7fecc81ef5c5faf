// What the general kernels (lc_forward_general.hip, lc_backward_data_general.hip, lc_backward_weights_general.hip)
// share.  They take any geometry: no alignment of patch rows, strides, filters or batch.  A wave owns an output tile and
// fetches its own operands, four consecutive values per lane, straight from global memory into the MFMA operands; there
// are no barriers in the main loop, and several waves can split one tile's contraction and add up through LDS.
#pragma once
#include "lc_common.hpp"

namespace lc {

typedef const __attribute__((address_space(1))) char *gbytes;

// four consecutive elements at any element-aligned address (unaligned vector loads are one instruction on this chip)
template <typename T> struct Quad;
template <> struct Quad<float> { typedef f32x4 V; };
template <> struct Quad<bf16_t> { typedef u32x2 V; };

template <typename T>
__device__ __forceinline__ typename Quad<T>::V load_quad(gbytes base, unsigned off) {
    typedef __attribute__((address_space(1), aligned(sizeof(T)))) typename Quad<T>::V GV;
    return *(const GV *)(base + off);
}

// N consecutive elements (a vector of three has no type of its own: clang pads it to four)
template <typename T, int N>
struct Run {
    typename RawVec<T, N>::V v;
    __device__ __forceinline__ void load(gbytes base, unsigned off) {
        typedef __attribute__((address_space(1), aligned(sizeof(T)))) typename RawVec<T, N>::V GV;
        v = *(const GV *)(base + off);
    }
    __device__ __forceinline__ float get(int i) const { return raw_get<T, N>(v, i); }
};
template <>
struct Run<float, 3> {
    struct __attribute__((packed, aligned(4))) P { float a, b, c; };
    float a, b, c;
    __device__ __forceinline__ void load(gbytes base, unsigned off) {
        const __attribute__((address_space(1))) P *p = (const __attribute__((address_space(1))) P *)(base + off);
        a = p->a; b = p->b; c = p->c;
    }
    __device__ __forceinline__ float get(int i) const { return i == 0 ? a : i == 1 ? b : c; }
};

// the low / high halves of two packed pairs as one pair (a in the low half)
__device__ __forceinline__ unsigned pair_lo(unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ unsigned pair_hi(unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// Four bf16 rows of N columns, as loaded, transposed: column u as four consecutive contraction indices.
template <int N>
__device__ __forceinline__ u32x2 column4(const Run<bf16_t, N> (&r)[4], int u) {
    if constexpr (N == 1) {
        return (u32x2){(unsigned)r[0].v | ((unsigned)r[1].v << 16), (unsigned)r[2].v | ((unsigned)r[3].v << 16)};
    } else if constexpr (N == 2) {
        return (u & 1) ? (u32x2){pair_hi(r[0].v, r[1].v), pair_hi(r[2].v, r[3].v)}
                       : (u32x2){pair_lo(r[0].v, r[1].v), pair_lo(r[2].v, r[3].v)};
    } else {
        const int h = u >> 1;
        return (u & 1) ? (u32x2){pair_hi(r[0].v[h], r[1].v[h]), pair_hi(r[2].v[h], r[3].v[h])}
                       : (u32x2){pair_lo(r[0].v[h], r[1].v[h]), pair_lo(r[2].v[h], r[3].v[h])};
    }
}

// the packed pair with the elements below `skip` (0..4, counted from the quad's first) set to zero
__device__ __forceinline__ u32x2 clear_below(u32x2 v, int skip) {
    const unsigned lo = skip >= 2 ? 0u : skip == 1 ? 0xffff0000u : 0xffffffffu;
    const unsigned hi = skip >= 4 ? 0u : skip == 3 ? 0xffff0000u : 0xffffffffu;
    return (u32x2){v[0] & lo, v[1] & hi};
}

// Sum of a tile over the `ks` waves (a power of two) that split its contraction: wave 0 of them ends up with it.  Pairs
// are added in a fixed order, so the result does not depend on timing.  buf: one slot of NACC*64 vectors per group of
// waves and per half of them.  Every wave of the workgroup calls it.
template <int NACC>
__device__ __forceinline__ void add_slices(f32x4 *acc, f32x4 *buf, int group, int slice, int ks) {
    const int lane = threadIdx.x & 63;
    for (int h = ks >> 1; h >= 1; h >>= 1) {
        f32x4 *slot = buf + ((size_t)group * (ks >> 1) + (slice & (h - 1))) * (NACC * 64) + lane;
        if (slice >= h && slice < 2 * h) {
#pragma unroll
            for (int q = 0; q < NACC; ++q) slot[q * 64] = acc[q];
        }
        __syncthreads();
        if (slice < h) {
#pragma unroll
            for (int q = 0; q < NACC; ++q) acc[q] += slot[q * 64];
        }
        __syncthreads();
    }
}

}  // namespace lc
