// What the general kernels (lc_forward_general.hip, lc_backward_data_general.hip, lc_backward_weights_general.hip)
// share.  They take any geometry: no alignment of patch rows, strides, filters or batch.  A wave owns an output tile and
// fetches its own operands, four consecutive values per lane, straight from global memory into the MFMA operands; there
// are no barriers in the main loop, and several waves can split one tile's contraction and add up through LDS.
#pragma once
#include <string.h>

#include "lc_common.hpp"

namespace lc {

constexpr long long kMostTasks = 1LL << 30;   // tasks are numbered in 32 bits, with room for the last workgroup's

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

// the packed elements with those below `skip` (counted from the first) set to zero
template <int N>
__device__ __forceinline__ void clear_below(unsigned (&v)[N], int skip) {
#pragma unroll
    for (int q = 0; q < N; ++q) v[q] &= skip >= 2 * q + 2 ? 0u : skip == 2 * q + 1 ? 0xffff0000u : 0xffffffffu;
}
__device__ __forceinline__ u32x2 clear_below(u32x2 v, int skip) {
    unsigned d[2] = {v[0], v[1]};
    clear_below<2>(d, skip);
    return (u32x2){d[0], d[1]};
}

// v_mfma_f32_16x16x32_bf16: lane l supplies the eight consecutive contraction indices 8*(l/16).. of row or column l%16
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f32x4 mfma32_bf16(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ u32x4 clear_below(u32x4 v, int skip) {
    unsigned d[4] = {v[0], v[1], v[2], v[3]};
    clear_below<4>(d, skip);
    return (u32x4){d[0], d[1], d[2], d[3]};
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

// The tile picked for a geometry, remembered per thread: picking is a pure function of the sizes that weighs up some
// hundred candidates, a few microseconds that a launch-bound caller would pay on every call.  64 entries, each replaced
// by the next geometry that falls on it.
template <typename V>
class TileMemo {
  public:
    template <typename Pick>
    const V &get(const Geom &g, int es, Pick pick) {
        const int key[8] = {g.B, g.H, g.W, g.C, g.R, g.S, g.F, es};
        unsigned h = 2166136261u;
        for (int k : key) h = (h ^ (unsigned)k) * 16777619u;
        Entry &e = entries_[(h ^ (h >> 16)) & 63u];
        if (!e.set || memcmp(e.key, key, sizeof(key)) != 0) {
            e.tile = pick(g, es);
            memcpy(e.key, key, sizeof(key));
            e.set = true;
        }
        return e.tile;
    }

  private:
    struct Entry { int key[8]; V tile; bool set; };
    Entry entries_[64] = {};
};

}  // namespace lc
