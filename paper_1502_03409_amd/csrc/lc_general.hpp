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

// Division of 0 <= n < 2^31 by a constant of the launch: a product and a shift, scalar where n is (the compiler's own division
// by a variable is some thirty vector instructions, and a kernel's task takes half a dozen of them in a row).
struct Divisor {
    unsigned m, sh, d;
    __host__ __device__ __forceinline__ int over(int n) const { return (int)(((unsigned long long)(unsigned)n * m) >> sh); }
};
inline Divisor divisor(int d) {
    unsigned s = 0;
    while ((1u << s) < (unsigned)d) ++s;
    // m d = 2^(31+s) + e with 0 < e <= d <= 2^s, so that n e < 2^(31+s)
    return {(unsigned)((1ull << (31 + s)) / (unsigned)d + 1), 31 + s, (unsigned)d};
}

// a wave's base address the compiler takes as it is
__device__ __forceinline__ gbytes opaque(gbytes p) {
    asm("" : "+s"(p));
    return p;
}
// a lane's offset likewise (the variable itself, so that no copy is made)
__device__ __forceinline__ unsigned opaque(unsigned &v) {
    asm("" : "+v"(v));
    return v;
}

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
    __device__ __forceinline__ void blank(bool z) { v = z ? typename RawVec<T, N>::V{} : v; }
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
    __device__ __forceinline__ void blank(bool z) { a = z ? 0.f : a; b = z ? 0.f : b; c = z ? 0.f : c; }
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
__device__ __forceinline__ f32x4 clear_below(f32x4 v, int skip) {
    return (f32x4){skip > 0 ? 0.f : v[0], skip > 1 ? 0.f : v[1], skip > 2 ? 0.f : v[2], skip > 3 ? 0.f : v[3]};
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

// fp32 products on the bf16 matrix units.  An fp32 MFMA holds the vector ALU's own multipliers, 33 clocks for 2048 flop
// and nothing beside it (a wave of 12 of them and 24 vector instructions takes 450 clocks of a SIMD, 390 without; the bf16
// MFMA runs beside them).  A value is the exact sum of three bf16 (8 of its 24 bits each, rounded to nearest: a part is at
// most 2^-8 of the one before it), and the product of two values is the six partial products down to 2^-16 of it; the three
// left out are at most 2^-24 of it together.  The six of 32 products take 96 clocks on the matrix unit, fp32 MFMAs 264.
// An infinite, NaN or overflowing operand makes every sum it meets non-finite, and an operand below 2^-110 can have bits
// below bf16's least value (2^-133): the kernels form tiles that meet either again in fp32.
struct Parts { u32x4 p[3]; };
__device__ __forceinline__ unsigned cvt_pk_bf16(float a, float b) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, __builtin_convertvector(((f32x2){a, b}), bf16x2));
}
// Gathers what two values' third parts are rounded from: 7 bits at most, so that the lower half of the word is zero unless bits
// lie below what bf16 holds.  (Here and now: left to the end, the compiler keeps all of them in registers until then.)
__device__ __forceinline__ void gather_low(unsigned &low, float a, float b) {
    low |= __builtin_bit_cast(unsigned, a) | __builtin_bit_cast(unsigned, b);
    opaque(low);
}
// whether an operand was more than the sum of its parts
__device__ __forceinline__ bool inexact(unsigned low) { return (low & 0xffffu) != 0; }
// eight consecutive contraction indices of a row or column
__device__ __forceinline__ Parts split8(const float (&x)[8], unsigned &low) {
    Parts s;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float a = x[2 * q], b = x[2 * q + 1];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const unsigned v = cvt_pk_bf16(a, b);
            s.p[i][q] = v;
            if (i < 2) {
                a -= bf16_lo(v);
                b -= bf16_hi(v);
            } else {
                gather_low(low, a, b);
            }
        }
    }
    return s;
}
// acc[m][n] += the products of 32 contraction indices of M rows and N columns.  The partial products, smallest first, add up
// from zero and meet the sum in one addition: a matrix instruction that adds to the sum itself rounds it each time (layers of
// 2000 products: 4.1e-7 of the result against 2.4e-7 in fp32 MFMAs; 1.1e-7 this way).  The M N chains of
// six run side by side: with two a wave waits for its own results (four instead of two in the workgroup-tiled kernels: one
// field of 62 x 62 x 24, 192 images, 4096 filters backwards 940 -> 918 us).
template <int M, int N>
__device__ __forceinline__ void mfma_split_rows(const Parts (&a)[M], const Parts (&b)[N], f32x4 (*acc)[N]) {
    constexpr int order[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
    f32x4 t[M][N];
#pragma unroll
    for (int o = 0; o < 6; ++o)
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int n = 0; n < N; ++n)
                t[m][n] = mfma32_bf16(a[m].p[order[o][0]], b[n].p[order[o][1]], o == 0 ? (f32x4){0.f, 0.f, 0.f, 0.f} : t[m][n]);
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
        for (int n = 0; n < N; ++n) acc[m][n] += t[m][n];
}
template <int N>
__device__ __forceinline__ void mfma_split(const Parts &a, const Parts (&b)[N], f32x4 (&acc)[N]) {
    mfma_split_rows(reinterpret_cast<const Parts(&)[1]>(a), b, &acc);
}
template <int M, int N>
__device__ __forceinline__ void mfma_split(const Parts (&a)[M], const Parts (&b)[N], f32x4 (&acc)[M][N]) {
#pragma unroll
    for (int m = 0; m < M; ++m) mfma_split(a[m], b, acc[m]);
}
// whether every value is finite
template <int N>
__device__ __forceinline__ bool all_finite(const f32x4 *v) {
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < N; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) s += v[q][r] * 0.f;
    return s == 0.f;
}

// whether every column n (lanes n, n + 16, n + 32, n + 48) has a lane set
__device__ __forceinline__ bool every_column(unsigned long long m) {
    m |= m >> 32;
    m |= m >> 16;
    return (m & 0xffffull) == 0xffffull;
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

// A forward pass's tile: image and filter blocks of a wave, then waves of a workgroup (blocks of filters, tasks, slices)
struct ForwardTile { int mt, nt, nfw, tasks, ks; };

// lc_forward_turned.hip: whether it takes a layer the general forward kernel supports, and its launches; `direct` is the
// direct form's tile
bool forward_turned_takes(const Geom &g, int es, const ForwardTile &direct);
double forward_turned_clocks(const Geom &g, const ForwardTile &direct);   // estimate of an fp32 launch
int launch_forward_turned(const Geom &g, const float *x, const float *w, const float *bias, float alpha, const float *alpha_dev,
                          float *y, const ForwardTile &direct, hipStream_t s);
int launch_forward_turned(const Geom &g, const bf16_t *x, const bf16_t *w, const float *bias, float alpha,
                          const float *alpha_dev, float *y, const ForwardTile &direct, hipStream_t s);

// Backward data's: image and value blocks of a wave, tasks and slices of a workgroup, strides of a pixel block each way
struct DataTile { int mt, nt, tasks, ks, qr, qc; };

// Fields that touch a block of q strides, summed over the blocks along an image side of n pixels with most fields, and
// their largest number.
inline void fields_across(const Geom &g, int q, int n, int most, double *sum, int *largest) {
    *sum = 0;
    *largest = 0;
    for (int r0 = 0; r0 < n; r0 += q * g.S) {
        const int lo = r0 < g.R ? 0 : (r0 - g.R + g.S) / g.S, hi = (r0 + q * g.S - 1) / g.S;
        const int c = (hi < most ? hi : most - 1) - lo + 1;
        if (c > 0) *sum += c;
        if (c > *largest) *largest = c;
    }
}

// lc_backward_data_turned.hip: whether it takes a layer the general backward-data kernel supports, and its launches; `direct`
// and VW are the direct form's tile and vector width
bool backward_data_turned_takes(const Geom &g, int es);
int launch_backward_data_turned(const Geom &g, const float *dy, const float *w, float *dx, const DataTile &direct, int VW,
                                hipStream_t s);
int launch_backward_data_turned(const Geom &g, const bf16_t *dy, const bf16_t *w, float *dx, const DataTile &direct, int VW,
                                hipStream_t s);

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
