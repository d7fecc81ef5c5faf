// Variants of the local contrast normalisation applied after each layer (Sec. 3.1 names LCN without defining it):
// statistics per channel instead of pooled over the channels, zero-padded instead of renormalised borders, and
// the two-stage form (subtract the local mean, then divide by the local root mean square of the result).
//
// Pooled statistics run in the channel-reduction kernels of the default form (pool_lcn.hip).  This file holds the
// per-channel kernels: two that walk down the rows of maps large enough for them, one that walks both stages of the two-stage
// form at once, and a tile kernel that takes every window, channel count and map size.  There every element has its own statistics, so a workgroup stages an 8x16 pixel
// tile, its halo and up to 32 channels of the quantity under the window in LDS (as float4 where C % 4 == 0), and each thread forms
// the Gaussian window sums for one pixel and four channels at a time.  Bandwidth-bound: the forward passes read
// the tile once (the centre value is taken from LDS), the halo ring comes from L2.
#include <mutex>

#include "lc_common.hpp"

namespace lc {
namespace {

constexpr int kTileH = 8, kTileW = 16;
constexpr int kMaxK = 15;
// Kernels that walk down the rows: waves per compute unit they aim at (segments are as short as that takes, but at least
// twice the rows they re-read) and below which the tile kernel stays, whose workgroups wait for memory once and not once a
// row (7 x 7 windows on [60,19,19,48], 1.7 waves: 21 against 22 us forward, 3.8 waves with the idle lanes of a half-filled
// chunk: 18 against 24 us backward; 5 x 5 on [157,18,18,48], 6 waves and more: 34 against 19 and 25 against 17 us).
constexpr int kStreamWaves = 16, kFewestWaves = 3, kRowsWaves = 12, kRowsFewest = 5;
constexpr int kRowThreads = 512;
constexpr int kLdsTarget = 32 * 1024;   // per workgroup: several workgroups per compute unit hide the load latency

struct Taps { float g[kMaxK]; };

enum : int {
    kFwdOne,    // x -> mu, rstd, y (one stage)
    kMean,      // x -> mu
    kDivide,    // x, mu -> rstd, y = (x - mu) rstd with the window mean of the neighbours' own (x - mu)^2
    kBwdOne,    // one-stage gradient
    kBwdTwoA,   // two-stage gradient up to dv (written to dx) and field = dv / normaliser
    kBwdTwoB    // dx = dv - window sum of field
};

struct Args {
    const float *x, *dy, *mu_in, *rstd_in;
    float *out, *mu_out, *rstd_out, *field;
    int H, W, C, CB, ks, zpad, tiles_w, tiles_per_img, nchunk;
    float eps;
    Taps taps;
};

__device__ __forceinline__ float taps_inside(const Taps &t, int p, int n, int r) {
    float z = 0.f;
    for (int d = -r; d <= r; ++d)
        if (p + d >= 0 && p + d < n) z += t.g[d + r];
    return z;
}

template <int V> struct Pack { float v[V]; };

template <int V> __device__ __forceinline__ Pack<V> load(const float *p) {
    Pack<V> r;
    if constexpr (V == 4) {
        const float4 t = *(const float4 *)p;
        r.v[0] = t.x; r.v[1] = t.y; r.v[2] = t.z; r.v[3] = t.w;
    } else {
        r.v[0] = *p;
    }
    return r;
}

template <int V> __device__ __forceinline__ void store(float *p, const Pack<V> &r) {
    if constexpr (V == 4) *(float4 *)p = make_float4(r.v[0], r.v[1], r.v[2], r.v[3]);
    else *p = r.v[0];
}

// V channels per work item (4 where C % 4 == 0); a.CB channels per workgroup, a multiple of V.
template <int OP, int V>
__global__ __launch_bounds__(256) void lcn_channel_kernel(Args a) {
    extern __shared__ __align__(16) float lds[];
    constexpr bool kTwoMaps = OP == kBwdOne;
    const int r = (a.ks - 1) / 2, hh = kTileH + 2 * r, hw = kTileW + 2 * r, H = a.H, W = a.W, C = a.C;
    const int CBV = a.CB / V;
    float *m1 = lds, *m2 = lds + hh * hw * a.CB;
    const int tid = threadIdx.x;
    int blk = remap_xcd(blockIdx.x, gridDim.x);   // an image's tiles, whose halos overlap, stay in one XCD's L2
    const int chunk = blk % a.nchunk;
    blk /= a.nchunk;
    const int b = blk / a.tiles_per_img, tile = blk - b * a.tiles_per_img;
    const int ti = (tile / a.tiles_w) * kTileH, tj = (tile % a.tiles_w) * kTileW;
    const int c0 = chunk * a.CB, ncv = min(CBV, (C - c0) / V);
    const size_t img = (size_t)b * H * W;
    // window normalisers of the staged rows and columns, once per workgroup (an element's is their product)
    __shared__ float zr[kTileH + kMaxK - 1], zc[kTileW + kMaxK - 1];
    if (tid < hh) zr[tid] = a.zpad ? 1.f : taps_inside(a.taps, ti - r + tid, H, r);
    else if (tid >= 64 && tid < 64 + hw) zc[tid - 64] = a.zpad ? 1.f : taps_inside(a.taps, tj - r + tid - 64, W, r);
    if (OP == kBwdOne || OP == kBwdTwoA) __syncthreads();   // the other passes first use them after phase 1's barrier
    auto norm_at = [&](int row, int col) { return zr[row - ti + r] * zc[col - tj + r]; };

    // phase 1: the quantity under the window for the tile and its halo; zeros outside the image
    for (int idx = tid; idx < hh * hw * CBV; idx += 256) {
        const int hp = idx / CBV, cv = idx - hp * CBV;
        const int hi = hp / hw, hj = hp - hi * hw;
        const int row = ti - r + hi, col = tj - r + hj;
        Pack<V> p1, p2;
#pragma unroll
        for (int k = 0; k < V; ++k) p1.v[k] = p2.v[k] = 0.f;
        if (cv < ncv && row >= 0 && row < H && col >= 0 && col < W) {
            const size_t e = (img + (size_t)row * W + col) * C + c0 + cv * V;
            if (OP == kBwdTwoB) {
                p1 = load<V>(a.field + e);
            } else if (OP == kFwdOne || OP == kMean) {
                p1 = load<V>(a.x + e);
            } else if (OP == kDivide) {
                const Pack<V> xv = load<V>(a.x + e), m = load<V>(a.mu_in + e);
#pragma unroll
                for (int k = 0; k < V; ++k) p1.v[k] = xv.v[k] - m.v[k];
            } else {
                const Pack<V> xv = load<V>(a.x + e), dv = load<V>(a.dy + e), m = load<V>(a.mu_in + e),
                              rs = load<V>(a.rstd_in + e);
                const float iz = 1.f / norm_at(row, col);
#pragma unroll
                for (int k = 0; k < V; ++k) {
                    // gradients of this element's window mean and second moment (or variance), over its normaliser
                    const float bc = rs.v[k] * rs.v[k] * rs.v[k] * dv.v[k] * (xv.v[k] - m.v[k]);
                    if (OP == kBwdOne) {
                        p1.v[k] = (bc * m.v[k] - rs.v[k] * dv.v[k]) * iz;
                        p2.v[k] = bc * iz;
                    } else {
                        p1.v[k] = -0.5f * bc * iz;
                    }
                }
            }
        }
        store<V>(m1 + (size_t)idx * V, p1);
        if (kTwoMaps) store<V>(m2 + (size_t)idx * V, p2);
    }
    __syncthreads();

    // phase 2: window sums for one pixel and V channels, then that element's output
    for (int idx = tid; idx < kTileH * kTileW * CBV; idx += 256) {
        const int op = idx / CBV, cv = idx - op * CBV;
        const int oi = op / kTileW, oj = op - oi * kTileW;
        const int row = ti + oi, col = tj + oj;
        if (cv >= ncv || row >= H || col >= W) continue;
        float s1[V], s2[V];
#pragma unroll
        for (int k = 0; k < V; ++k) s1[k] = s2[k] = 0.f;
        for (int p = 0; p < a.ks; ++p)
            for (int q = 0; q < a.ks; ++q) {
                const float wt = a.taps.g[p] * a.taps.g[q];
                const int h = (((oi + p) * hw + oj + q) * CBV + cv) * V;
                const Pack<V> t = load<V>(m1 + h);
                if (OP == kBwdOne) {
                    const Pack<V> t2 = load<V>(m2 + h);
#pragma unroll
                    for (int k = 0; k < V; ++k) { s1[k] += wt * t.v[k]; s2[k] += wt * t2.v[k]; }
                } else {
#pragma unroll
                    for (int k = 0; k < V; ++k) {
                        if (OP == kDivide) s1[k] += wt * t.v[k] * t.v[k];
                        else s1[k] += wt * t.v[k];
                        if (OP == kFwdOne) s2[k] += wt * t.v[k] * t.v[k];
                    }
                }
            }
        const size_t e = (img + (size_t)row * W + col) * C + c0 + cv * V;
        const float z = norm_at(row, col);
        Pack<V> o;
        if (OP == kFwdOne || OP == kDivide) {
            // the element's own x (or x - mu) is still in LDS
            const Pack<V> ctr = load<V>(m1 + (((oi + r) * hw + oj + r) * CBV + cv) * V);
            Pack<V> m, rs;
#pragma unroll
            for (int k = 0; k < V; ++k) {
                if (OP == kFwdOne) {
                    m.v[k] = s1[k] / z;
                    rs.v[k] = 1.0f / sqrtf(fmaxf(s2[k] / z - m.v[k] * m.v[k], 0.f) + a.eps);
                    o.v[k] = (ctr.v[k] - m.v[k]) * rs.v[k];
                } else {
                    rs.v[k] = 1.0f / sqrtf(s1[k] / z + a.eps);
                    o.v[k] = ctr.v[k] * rs.v[k];
                }
            }
            if (OP == kFwdOne) store<V>(a.mu_out + e, m);
            store<V>(a.rstd_out + e, rs);
            store<V>(a.out + e, o);
        } else if (OP == kMean) {
#pragma unroll
            for (int k = 0; k < V; ++k) o.v[k] = s1[k] / z;
            store<V>(a.mu_out + e, o);
        } else if (OP == kBwdOne) {
            const Pack<V> xv = load<V>(a.x + e), dv = load<V>(a.dy + e), rs = load<V>(a.rstd_in + e);
#pragma unroll
            for (int k = 0; k < V; ++k) o.v[k] = dv.v[k] * rs.v[k] + s1[k] - xv.v[k] * s2[k];
            store<V>(a.out + e, o);
        } else if (OP == kBwdTwoA) {
            const Pack<V> xv = load<V>(a.x + e), dv = load<V>(a.dy + e), m = load<V>(a.mu_in + e),
                          rs = load<V>(a.rstd_in + e);
            Pack<V> f;
#pragma unroll
            for (int k = 0; k < V; ++k) {
                o.v[k] = dv.v[k] * rs.v[k] + 2.f * (xv.v[k] - m.v[k]) * s1[k];
                f.v[k] = o.v[k] / z;
            }
            store<V>(a.out + e, o);
            store<V>(a.field + e, f);
        } else {   // kBwdTwoB
            const Pack<V> dv = load<V>(a.out + e);
#pragma unroll
            for (int k = 0; k < V; ++k) o.v[k] = dv.v[k] - s1[k];
            store<V>(a.out + e, o);
        }
    }
}

// The passes over one array (kFwdOne, kMean, kBwdTwoB) as a stream, for windows of 3, 5, 7 and 9: a work item owns one column and V channels and walks down a
// segment of rows.  Each row it meets gives one horizontal window sum (KS loads whose neighbours in the wave read the same
// lines); the last KS of them stay in registers, so an output costs one new row of loads and KS vertical taps instead of
// KS*KS reads from LDS, and without barriers every wave reads and writes all the time.  Segments of RS rows re-read
// KS-1 rows of their neighbours.  Columns outside the image are read from the item's own column and left out of the sum.
// HBM-bound: one stage on [128,44,44,32] maps, 5 x 5 windows, 45 -> 31 us = 4.1 TB/s of the bytes it cannot do without.
template <int OP, int V, int KS>
__global__ __launch_bounds__(256) void lcn_channel_stream_kernel(Args a, int RS, int nseg, unsigned total) {
    static_assert(OP == kFwdOne || OP == kMean || OP == kBwdTwoB, "passes over one array");
    constexpr bool kTwoMaps = OP == kFwdOne;
    constexpr int r = (KS - 1) / 2;
    const unsigned e = remap_xcd(blockIdx.x, gridDim.x) * 256u + threadIdx.x;
    if (e >= total) return;
    const int H = a.H, W = a.W, CV = a.C / V, per_row = W * CV;
    const unsigned t = e / (unsigned)per_row;
    const int cj = (int)(e - t * (unsigned)per_row), j = cj / CV;
    const int b = (int)(t / (unsigned)nseg), sg = (int)(t - (unsigned)b * nseg);
    const int ro0 = sg * RS, ro1 = min(ro0 + RS, H);
    const size_t base = (size_t)b * H * per_row + cj;          // in vectors of V

    float g[KS];
    int off[KS];
    bool in[KS];
#pragma unroll
    for (int q = 0; q < KS; ++q) {
        const int jj = j + q - r;
        g[q] = a.taps.g[q];
        in[q] = jj >= 0 && jj < W;
        off[q] = in[q] ? (q - r) * CV : 0;
    }
    const float zc = a.zpad ? 1.f : taps_inside(a.taps, j, W, r);
    auto row_norm = [&](int row) -> float {
        if (a.zpad) return 1.f;
        float z = 0.f;
#pragma unroll
        for (int d = 0; d < KS; ++d) z += row + d - r >= 0 && row + d - r < H ? g[d] : 0.f;
        return z;
    };

    Pack<V> h1[KS], h2[kTwoMaps ? KS : 1];                     // horizontal sums of the last KS rows
#pragma unroll
    for (int d = 0; d < KS; ++d)
#pragma unroll
        for (int k = 0; k < V; ++k) {
            h1[d].v[k] = 0.f;
            if (kTwoMaps) h2[d].v[k] = 0.f;
        }
    for (int ir = ro0 - r; ir < ro1 + r; ++ir) {
        Pack<V> n1, n2;
#pragma unroll
        for (int k = 0; k < V; ++k) n1.v[k] = n2.v[k] = 0.f;
        if (ir >= 0 && ir < H) {
            const size_t row = base + (size_t)ir * per_row;
#pragma unroll
            for (int q = 0; q < KS; ++q) {
                const size_t o = (row + off[q]) * V;
                const Pack<V> p = load<V>((OP == kBwdTwoB ? a.field : a.x) + o);
#pragma unroll
                for (int k = 0; k < V; ++k) {
                    const float v = in[q] ? p.v[k] : 0.f;
                    n1.v[k] += g[q] * v;
                    if (kTwoMaps) n2.v[k] += g[q] * v * v;
                }
            }
        }
#pragma unroll
        for (int d = 0; d + 1 < KS; ++d) {
            h1[d] = h1[d + 1];
            if (kTwoMaps) h2[d] = h2[d + 1];
        }
        h1[KS - 1] = n1;
        if (kTwoMaps) h2[kTwoMaps ? KS - 1 : 0] = n2;
        const int ro = ir - r;
        if (ro < ro0) continue;
        float s1[V], s2[V];
#pragma unroll
        for (int k = 0; k < V; ++k) {
            s1[k] = s2[k] = 0.f;
#pragma unroll
            for (int d = 0; d < KS; ++d) {
                s1[k] += g[d] * h1[d].v[k];
                if (kTwoMaps) s2[k] += g[d] * h2[kTwoMaps ? d : 0].v[k];
            }
        }
        const size_t o = (base + (size_t)ro * per_row) * V;
        const float z = row_norm(ro) * zc;
        Pack<V> out;
        if (OP == kMean) {
#pragma unroll
            for (int k = 0; k < V; ++k) out.v[k] = s1[k] / z;
            store<V>(a.mu_out + o, out);
        } else if (OP == kFwdOne) {
            const Pack<V> xv = load<V>(a.x + o);
            Pack<V> m, rs;
#pragma unroll
            for (int k = 0; k < V; ++k) {
                m.v[k] = s1[k] / z;
                rs.v[k] = 1.0f / sqrtf(fmaxf(s2[k] / z - m.v[k] * m.v[k], 0.f) + a.eps);
                out.v[k] = (xv.v[k] - m.v[k]) * rs.v[k];
            }
            store<V>(a.mu_out + o, m);
            store<V>(a.rstd_out + o, rs);
            store<V>(a.out + o, out);
        } else {
            const Pack<V> dv = load<V>(a.out + o);
#pragma unroll
            for (int k = 0; k < V; ++k) out.v[k] = dv.v[k] - s1[k];
            store<V>(a.out + o, out);
        }
    }
}

// The passes whose quantity under the window takes several arrays (kDivide, kBwdOne, kBwdTwoA), C % 4 == 0: forming it KS
// times per element costs more than the window sums, so a workgroup walks down a strip of TO columns (and r on either
// side) by CB channel quads, each thread forms its own element's quantity of a row once and leaves it in LDS, and the
// horizontal sums come from there: one barrier a row, two row buffers in turn.  What the output needs of its own element
// waits r rows in registers, so every array is read once (but for the r columns and rows on a strip's sides).  The next
// row's loads are in flight meanwhile.  On the same maps: one-stage gradient 45 -> 30 us; two stages 74 -> 43 us forward,
// 85 -> 53 us backward.  (Forming the quantity for every neighbour, as the stream above would, took 117 and 84 us backward.)
template <int OP, int KS>
__global__ __launch_bounds__(kRowThreads) void lcn_channel_rows_kernel(Args a, int TO, int CB, int nstrip, int RS, int nseg) {
    static_assert(OP == kDivide || OP == kBwdOne || OP == kBwdTwoA, "passes over several arrays");
    constexpr int r = (KS - 1) / 2;
    constexpr bool kTwoMaps = OP == kBwdOne, kGrad = OP != kDivide;
    typedef float f4 __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) float lds[];
    const int H = a.H, W = a.W, CV = a.C / 4, TC = TO + 2 * r;
    const int ct = threadIdx.x / CB, cq = threadIdx.x - ct * CB;
    int blk = remap_xcd(blockIdx.x, gridDim.x);                // strips and segments of one image stay in one XCD's L2
    const int chunk = blk % a.nchunk; blk /= a.nchunk;
    const int strip = blk % nstrip; blk /= nstrip;
    const int sg = blk % nseg, b = blk / nseg;
    const int j = strip * TO + ct - r, cv = chunk * CB + cq;
    const bool lane = ct < TC && cv < CV, col_in = lane && j >= 0 && j < W;
    const bool owns = col_in && ct >= r && ct < r + TO;        // an output column of this strip
    const int ro0 = sg * RS, ro1 = min(ro0 + RS, H);
    const size_t base = ((size_t)b * H * W + (col_in ? j : 0)) * CV + (lane ? cv : 0), rstride = (size_t)W * CV;
    f4 *row0 = (f4 *)lds + ct * CB + cq;                       // [2 buffers][maps][TC][CB]
    const int map = TC * CB, buf = (kTwoMaps ? 2 : 1) * map;

    float g[KS];
#pragma unroll
    for (int q = 0; q < KS; ++q) g[q] = a.taps.g[q];
    const float zc = a.zpad ? 1.f : taps_inside(a.taps, col_in ? j : 0, W, r);
    auto row_norm = [&](int row) -> float {
        if (a.zpad) return 1.f;
        float z = 0.f;
#pragma unroll
        for (int d = 0; d < KS; ++d) z += row + d - r >= 0 && row + d - r < H ? g[d] : 0.f;
        return z;
    };
    struct Elem { f4 x, m, d, rs; };
    auto fetch = [&](int row, Elem &e) {
        const size_t o = base + (size_t)min(max(row, 0), H - 1) * rstride;
        e.x = ((const f4 *)a.x)[o];
        e.m = ((const f4 *)a.mu_in)[o];
        if constexpr (kGrad) {
            e.d = ((const f4 *)a.dy)[o];
            e.rs = ((const f4 *)a.rstd_in)[o];
        }
    };
    f4 h1[KS], h2[kTwoMaps ? KS : 1], k1[r + 1], k2[kGrad ? r + 1 : 1];
#pragma unroll
    for (int d = 0; d < KS; ++d) {
        h1[d] = (f4)(0.f);
        if (kTwoMaps) h2[kTwoMaps ? d : 0] = (f4)(0.f);
    }
    Elem cur, nxt;
    fetch(ro0 - r, cur);
    for (int ir = ro0 - r; ir < ro1 + r; ++ir) {
        fetch(ir + 1, nxt);
        f4 p1 = (f4)(0.f), p2 = (f4)(0.f);
        const f4 diff = cur.x - cur.m;
        if (col_in && ir >= 0 && ir < H) {
            if constexpr (OP == kDivide) {
                p1 = diff * diff;
            } else {
                // gradients of this element's window mean and second moment (or variance), over its normaliser
                const float iz = 1.f / (row_norm(ir) * zc);
                const f4 bc = cur.rs * cur.rs * cur.rs * cur.d * diff;
                if constexpr (OP == kBwdOne) {
                    p1 = (bc * cur.m - cur.rs * cur.d) * iz;
                    p2 = bc * iz;
                } else {
                    p1 = -0.5f * bc * iz;
                }
            }
        }
        f4 *row = row0 + (ir & 1) * buf;
        if (lane) {
            row[0] = p1;
            if constexpr (kTwoMaps) row[map] = p2;
        }
        // what the output of this row needs of its own element, r rows later
#pragma unroll
        for (int d = 0; d < r; ++d) {
            k1[d] = k1[d + 1];
            if constexpr (kGrad) k2[d] = k2[d + 1];
        }
        if constexpr (OP == kDivide) k1[r] = diff;
        else { k1[r] = cur.d * cur.rs; k2[r] = OP == kBwdOne ? cur.x : diff; }
        __syncthreads();
        f4 n1 = (f4)(0.f), n2 = (f4)(0.f);
        if (owns) {
#pragma unroll
            for (int q = 0; q < KS; ++q) {
                n1 += g[q] * row[(q - r) * CB];
                if constexpr (kTwoMaps) n2 += g[q] * row[map + (q - r) * CB];
            }
        }
#pragma unroll
        for (int d = 0; d + 1 < KS; ++d) {
            h1[d] = h1[d + 1];
            if constexpr (kTwoMaps) h2[d] = h2[d + 1];
        }
        h1[KS - 1] = n1;
        if constexpr (kTwoMaps) h2[KS - 1] = n2;
        const int ro = ir - r;
        cur = nxt;
        if (ro < ro0 || !owns) continue;
        f4 s1 = (f4)(0.f), s2 = (f4)(0.f);
#pragma unroll
        for (int d = 0; d < KS; ++d) {
            s1 += g[d] * h1[d];
            if constexpr (kTwoMaps) s2 += g[d] * h2[d];
        }
        const size_t o = base + (size_t)ro * rstride;
        const float z = row_norm(ro) * zc;
        if constexpr (OP == kDivide) {
            f4 rs;
#pragma unroll
            for (int k = 0; k < 4; ++k) rs[k] = 1.0f / sqrtf(s1[k] / z + a.eps);
            ((f4 *)a.rstd_out)[o] = rs;
            ((f4 *)a.out)[o] = k1[0] * rs;
        } else if constexpr (OP == kBwdOne) {
            ((f4 *)a.out)[o] = k1[0] + s1 - k2[0] * s2;
        } else {
            const f4 dv = k1[0] + 2.f * k2[0] * s1;
            ((f4 *)a.out)[o] = dv;
            ((f4 *)a.field)[o] = dv / z;
        }
    }
}

// Waves per SIMD that the two-stage kernel's registers are kept to; none of them spills under it (with seven the gradient of
// single channels and 7 x 7 spilled four: 60 maps 1.06 times as long as with six, 1.03 in the caches).
constexpr int two_stage_waves(bool grad, int V, int KS) {
    if (V == 4) return grad ? (KS == 3 ? 3 : 2) : (KS == 3 ? 5 : 3);
    if (V == 2) return grad ? (KS == 3 ? 6 : KS == 5 ? 4 : 3) : (KS == 3 ? 8 : KS == 5 ? 5 : 4);
    return grad ? (KS <= 5 ? 8 : KS == 7 ? 6 : 5) : (KS == 3 ? 8 : KS == 5 ? 7 : KS == 7 ? 5 : 4);
}

// Both stages of the two-stage form in one walk, forward (GRAD false: x -> mu, rstd, y) or backward (x, mu, rstd, dy -> dx).
// A workgroup walks down a strip of TO columns, 2r more on either side, by CB work items of V channels; each row it loads
// goes through two rings of KS rows in registers.  A stage sums its ring vertically, leaves the sum in LDS and adds it up
// horizontally from there: the first stage's row is r rows behind the load and gives the quantity under the second window
// (the squared difference from the mean, or dv over its normaliser), the second stage's is r + 1 rows behind that, so one
// barrier a row serves both.  The ring slots are named by the row loop, which is unrolled over KS rows.  Values outside the
// image are zeros.  Every array is read once, but for the 2 r columns and rows at a strip's sides: on [128,44,44,32], 5 x 5, 33
// us forward and 30 backward where the two passes take 45 and 54, which move the mean, dv and its normalised field through memory
// (the arrays alone are 21 and 26 us at 6 TB/s).  The forward walk issues vector instructions in 46 % of its cycles at 2.2 waves
// per SIMD, 3.5 TB/s and no bank conflicts: what is left is the row's chain of load, vertical sum, LDS, horizontal sum twice over.
// The gradient moves 5.8 TB/s.  Maps of tens of microseconds and less wait for launches and that chain, and halve.
template <bool GRAD, int V, int KS>
__global__ __launch_bounds__(kRowThreads, two_stage_waves(GRAD, V, KS)) void lcn_channel_two_stage_kernel(Args a, int TO, int CB, int nstrip, int RS,
                                                                            int nseg) {
    constexpr int r = (KS - 1) / 2;
    typedef typename FVec<V>::T VT;
    extern __shared__ __align__(16) float lds[];
    const int H = a.H, W = a.W, CV = a.C / V, TC = TO + 4 * r;
    const int ct = threadIdx.x / CB, cq = threadIdx.x - ct * CB;
    int blk = remap_xcd(blockIdx.x, gridDim.x);                // strips and segments of one image stay in one XCD's L2
    const int chunk = blk % a.nchunk; blk /= a.nchunk;
    const int strip = blk % nstrip; blk /= nstrip;
    const int sg = blk % nseg, b = blk / nseg;
    const int j = strip * TO + ct - 2 * r, cv = chunk * CB + cq;
    const bool lane = ct < TC && cv < CV, col_in = lane && j >= 0 && j < W;
    const bool inner = col_in && ct >= r && ct < TC - r;       // a column of the first stage
    const bool owns = col_in && ct >= 2 * r && ct < 2 * r + TO;
    const int ro0 = sg * RS, ro1 = min(ro0 + RS, H);
    const size_t base = ((size_t)b * H * W + (col_in ? j : 0)) * CV + (lane ? cv : 0), rstride = (size_t)W * CV;
    VT *row0 = (VT *)lds + ct * CB + cq;                       // [2 buffers][2 stages][TC][CB]
    const int map = TC * CB;

    float g[KS], full = 0.f;
#pragma unroll
    for (int q = 0; q < KS; ++q) { g[q] = a.taps.g[q]; full += g[q]; }
    const float zc = a.zpad ? 1.f : taps_inside(a.taps, col_in ? j : 0, W, r);
    const float whole = 1.f / (full * zc);
    auto inv_norm = [&](int row) -> float {                    // 1 / normaliser of the window around an element of this row
        if (a.zpad) return 1.f;
        if (row >= r && row + r < H) return whole;
        float z = 0.f;
#pragma unroll
        for (int d = 0; d < KS; ++d) z += row + d - r >= 0 && row + d - r < H ? g[d] : 0.f;
        return 1.f / (z * zc);
    };
    constexpr int AHEAD = GRAD || KS < 5 || V * KS > 16 ? 2 : 3;          // rows whose loads are in flight
    struct Elem { VT x, m, d, rs; } e[KS];
    auto fetch = [&](int row, Elem &e) {
        const size_t o = base + (size_t)min(max(row, 0), H - 1) * rstride;
        e.x = ((const VT *)a.x)[o];
        if constexpr (GRAD) {
            e.m = ((const VT *)a.mu_in)[o];
            e.d = ((const VT *)a.dy)[o];
            e.rs = ((const VT *)a.rstd_in)[o];
        }
    };
    // q1: what the first window sums.  q2: what the second one sums; c2: what the output needs of the same element.
    // c1, d1 (GRAD): dy rstd and x - mu of the rows the first stage has not reached
    VT q1[KS], q2[KS], c2[KS], c1[GRAD ? KS : 1], d1[GRAD ? KS : 1];
#pragma unroll
    for (int d = 0; d < KS; ++d) q1[d] = q2[d] = c2[d] = (VT)(0.f);
    if constexpr (GRAD)
#pragma unroll
        for (int d = 0; d < KS; ++d) c1[d] = d1[d] = (VT)(0.f);
    const int first = max(ro0 - 2 * r, 0), last = ro1 + 2 * r;   // rows of the walk; the last one only ends the second stage
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) fetch(first + u, e[u]);
    for (int top = first; top <= last; top += KS) {
#pragma unroll
        for (int u = 0; u < KS; ++u) {
            const int ir = top + u, ra = ir - r, rb = ir - 2 * r - 1;
            if (ir > last) break;
            const bool in = col_in && ir >= 0 && ir < H;
            if constexpr (GRAD) {
                const VT diff = e[u].x - e[u].m;
                d1[u] = diff;
                c1[u] = e[u].d * e[u].rs;
                // gradient of this element's window variance, over its normaliser
                q1[u] = in ? -0.5f * (e[u].rs * e[u].rs * e[u].rs * e[u].d * diff) * inv_norm(ir) : (VT)(0.f);
            } else {
                q1[u] = in ? e[u].x : (VT)(0.f);
            }
            fetch(ir + AHEAD, e[(u + AHEAD) % KS]);
            VT v1 = (VT)(0.f), v2 = (VT)(0.f);
#pragma unroll
            for (int d = 0; d < KS; ++d) {
                v1 += g[d] * q1[(u + 1 + d) % KS];
                v2 += g[d] * q2[(u + d) % KS];
            }
            VT *row = row0 + (u & 1 ? 2 * map : 0);
            if (top - first & 1) row = row0 + (u & 1 ? 0 : 2 * map);   // KS is odd: the buffers change places every trip
            if (lane) {
                row[0] = v1;
                row[map] = v2;
            }
            __syncthreads();
            VT n2 = (VT)(0.f), m2 = (VT)(0.f);
            if (inner && ra >= 0 && ra < H) {
                VT s = (VT)(0.f);
#pragma unroll
                for (int q = 0; q < KS; ++q) s += g[q] * row[(q - r) * CB];
                const float iz = inv_norm(ra);
                if constexpr (GRAD) {
                    m2 = c1[(u + KS - r) % KS] + 2.f * d1[(u + KS - r) % KS] * s;
                    n2 = m2 * iz;
                } else {
                    const VT mu = s * iz;
                    if (owns && ra >= ro0 && ra < ro1) ((VT *)a.mu_out)[base + (size_t)ra * rstride] = mu;
                    m2 = q1[(u + KS - r) % KS] - mu;
                    n2 = m2 * m2;
                }
            }
            if (owns && rb >= ro0) {                           // rb < ro1 by the end of the loop
                VT s = (VT)(0.f);
#pragma unroll
                for (int q = 0; q < KS; ++q) s += g[q] * row[map + (q - r) * CB];
                const size_t o = base + (size_t)rb * rstride;
                const VT c = c2[(u + KS - 1 - r) % KS];
                if constexpr (GRAD) {
                    ((VT *)a.out)[o] = c - s;
                } else {
                    const float iz = inv_norm(rb);
                    VT rs;
                    if constexpr (V > 1) {
#pragma unroll
                        for (int k = 0; k < V; ++k) rs[k] = 1.0f / sqrtf(s[k] * iz + a.eps);
                    } else {
                        rs = 1.0f / sqrtf(s * iz + a.eps);
                    }
                    ((VT *)a.rstd_out)[o] = rs;
                    ((VT *)a.out)[o] = c * rs;
                }
            }
            q2[u] = n2;
            c2[u] = m2;
        }
    }
}

bool make_taps(int ks, float sigma, Taps *t) {
    if (ks < 1 || ks > kMaxK || (ks & 1) == 0 || !(sigma > 0.f)) return false;
    const int r = (ks - 1) / 2;
    double s = 0.0, g[kMaxK];
    for (int p = -r; p <= r; ++p) {
        g[p + r] = exp(-(double)(p * p) / (2.0 * (double)sigma * (double)sigma));
        s += g[p + r];
    }
    for (int p = 0; p < kMaxK; ++p) t->g[p] = p < ks ? (float)(g[p] / s) : 0.f;
    return true;
}

template <int OP, int V, int KS>
int launch_stream(const Args &a, int B, hipStream_t s, const char *where, bool *done) {
    // segments so short that the chip holds about WANT waves per compute unit, but at least twice the rows they re-read
    const long long cols = (long long)B * a.W * (a.C / V), want = (256LL * kStreamWaves * 64 + cols - 1) / cols;
    int RS = (int)((a.H + want - 1) / want);
    if (RS < 2 * (KS - 1)) RS = 2 * (KS - 1);
    const int nseg = (a.H + RS - 1) / RS;
    const long long total = cols * nseg;
    if (total >= (1LL << 31) || total < 256LL * 64 * kFewestWaves) return LC_OK;
    *done = true;
    hipLaunchKernelGGL((lcn_channel_stream_kernel<OP, V, KS>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, a, RS,
                       nseg, (unsigned)total);
    LC_HIP_LAUNCH_CHECK(where);
    return LC_OK;
}

template <int OP, int KS>
int launch_rows(Args a, int B, hipStream_t s, const char *where, bool *done) {
    constexpr int r = (KS - 1) / 2;
    const int CV = a.C / 4;
    // whole 128-byte lines of a pixel per chunk; strips that split the image evenly within a workgroup's threads
    const int CB = CV < 8 ? CV : 8, most = kRowThreads / CB - 2 * r;
    if (most < 1) return LC_OK;
    a.nchunk = (CV + CB - 1) / CB;
    const int nstrip = (a.W + most - 1) / most, TO = (a.W + nstrip - 1) / nstrip, TC = TO + 2 * r;
    // narrow maps of four and eight channels leave most lanes of a wave without work ([210,161,11,4], 7 x 7 windows, two
    // stages: 46 us forward and 41 backward here, 36 and 33 in tiles; [124,259,16,4]: 43 and 40 against 33 and 32; from 17
    // columns on the two are even and, where the last tile is ragged, [112,248,20,4]: 38 and 29 against 39 and 40)
    if (CB <= 2 && TO * CB <= 16) return LC_OK;
    const int nthr = (TC * CB + 63) / 64 * 64;
    const long long strips = (long long)B * nstrip * a.nchunk, want = 256LL * kRowsWaves * 64;
    long long nseg = (want + strips * nthr - 1) / (strips * nthr);
    int RS = (int)((a.H + nseg - 1) / nseg);
    if (RS < 2 * (KS - 1)) RS = 2 * (KS - 1);
    nseg = (a.H + RS - 1) / RS;
    if (strips * nseg > 0x7fffffffLL || strips * nseg * nthr < 256LL * 64 * kRowsFewest) return LC_OK;
    const size_t lds = (size_t)2 * (OP == kBwdOne ? 2 : 1) * TC * CB * 16;
    *done = true;
    hipLaunchKernelGGL((lcn_channel_rows_kernel<OP, KS>), dim3((unsigned)(strips * nseg)), dim3(nthr), lds, s, a, TO, CB, nstrip,
                       RS, (int)nseg);
    LC_HIP_LAUNCH_CHECK(where);
    return LC_OK;
}

// one pass through the streaming kernels where they take the window; *done tells whether one was launched
template <int OP, int V, int KS>
int launch_walk(const Args &a, int B, hipStream_t s, const char *where, bool *done) {
    if constexpr (OP == kDivide || OP == kBwdOne || OP == kBwdTwoA) {
        if constexpr (V == 4) return launch_rows<OP, KS>(a, B, s, where, done);
        else return LC_OK;
    } else {
        return launch_stream<OP, V, KS>(a, B, s, where, done);
    }
}

template <int OP, int V>
int launch_pass_v(Args a, int B, hipStream_t s, const char *where) {
    // (the two-stage form takes these windows in one kernel where C is no multiple of four)
    if constexpr (V == 4 || OP == kFwdOne) {
        bool done = false;
        int rc = LC_OK;
        if (a.ks == 3) rc = launch_walk<OP, V, 3>(a, B, s, where, &done);
        else if (a.ks == 5) rc = launch_walk<OP, V, 5>(a, B, s, where, &done);
        else if (a.ks == 7) rc = launch_walk<OP, V, 7>(a, B, s, where, &done);
        else if (a.ks == 9) rc = launch_walk<OP, V, 9>(a, B, s, where, &done);
        if (done || rc != LC_OK) return rc;
    }
    const int tiles_h = (a.H + kTileH - 1) / kTileH;
    a.tiles_w = (a.W + kTileW - 1) / kTileW;
    a.tiles_per_img = tiles_h * a.tiles_w;
    const int maps = OP == kBwdOne ? 2 : 1;
    const size_t per_channel = (size_t)(kTileH + a.ks - 1) * (kTileW + a.ks - 1) * maps * sizeof(float);
    // whole 128-byte lines of a pixel where LDS allows; never fewer than V channels (at most 10.6 KB then)
    a.CB = a.C < 32 ? a.C : 32;
    while (a.CB > V && a.CB * per_channel > (size_t)kLdsTarget) a.CB = (a.CB / 2 + V - 1) / V * V;
    a.nchunk = (a.C + a.CB - 1) / a.CB;
    const long long nblk = (long long)B * a.tiles_per_img * a.nchunk;
    if (nblk > 0x7fffffffLL) return LC_EUNSUPPORTED;
    const size_t lds = a.CB * per_channel;
    auto kern = lcn_channel_kernel<OP, V>;
    if (int rc = allow_dynamic_lds((const void *)kern, lds, where)) return rc;
    hipLaunchKernelGGL(kern, dim3((unsigned)nblk), dim3(256), lds, s, a);
    LC_HIP_LAUNCH_CHECK(where);
    return LC_OK;
}

template <int OP>
int launch_pass(const Args &a, int B, hipStream_t s, const char *where) {
    return a.C % 4 == 0 ? launch_pass_v<OP, 4>(a, B, s, where) : launch_pass_v<OP, 1>(a, B, s, where);
}

// Both stages in one kernel.  CB work items a pixel side by side and segments of RS rows by estimated time: a compute unit
// walks its workgroups in rounds of as many as the registers hold, a row takes a round 0.2 us per channel of a work item and
// 0.05 us per wave, narrow pieces of a pixel take longer; short segments walk the 4 r rows at their sides for fewer rows of
// their own.  The constants are a fit to 24 maps timed with every CB and 17 numbers of segments: the pick is on average 2 % slower
// than the fastest backward and 5 % forward.  CB is a power of two, or a whole pixel: pieces of 24 or 96 bytes share sectors
// with the next workgroup's.
template <bool GRAD, int V, int KS>
int launch_two_stage(Args a, int B, hipStream_t s, const char *where, bool *done) {
    constexpr int r = (KS - 1) / 2;
    const int CV = a.C / V;
    constexpr int resident = 4 * two_stage_waves(GRAD, V, KS);
    int CB = 0, nstrip = 1, TO = 1, nthr = 64, RS = a.H;
    double least = 1e300;
    for (int cb = 1; cb <= 8 && cb <= CV; ++cb) {
        if ((cb & (cb - 1)) != 0 && cb != CV) continue;
        const int most = kRowThreads / cb - 4 * r, n = (a.W + most - 1) / most, to = (a.W + n - 1) / n;
        const int t = ((to + 4 * r) * cb + 63) / 64 * 64, waves = t / 64, slots = resident / waves > 0 ? resident / waves : 1;
        const long long strips = (long long)B * n * ((CV + cb - 1) / cb);
        for (int seg = 1; seg <= a.H; seg += seg < 8 ? 1 : seg / 4) {
            const int rs = (a.H + seg - 1) / seg;
            const long long per_cu = (strips * seg + 255) / 256;
            const double rows = rs + 2 * r + 1 + (seg > 1 ? 2 * r : 0);
            const double us = rows * (1.0 + 0.4 / cb) *
                              ((double)(per_cu / slots) * (0.2 * V + 0.05 * slots * waves) +
                               (per_cu % slots ? 0.2 * V + 0.05 * (per_cu % slots) * waves : 0.0));
            if (us < least) { least = us; CB = cb; nstrip = n; TO = to; nthr = t; RS = rs; }
        }
    }
    a.nchunk = (CV + CB - 1) / CB;
    const int TC = TO + 4 * r, nseg = (a.H + RS - 1) / RS;
    const long long strips = (long long)B * nstrip * a.nchunk;
    if (strips * nseg > 0x7fffffffLL) return LC_OK;
    const size_t lds = (size_t)4 * TC * CB * V * 4;
    *done = true;
    hipLaunchKernelGGL((lcn_channel_two_stage_kernel<GRAD, V, KS>), dim3((unsigned)(strips * nseg)), dim3(nthr), lds, s, a, TO,
                       CB, nstrip, RS, nseg);
    LC_HIP_LAUNCH_CHECK(where);
    return LC_OK;
}

// Channels per work item: the wider, the fewer loads and index steps; two where four leave the chip too few waves (5 x 5 on
// [2,12,48,64]: 8.6 us with four, 6.9 with two), and two and one where the rings of 7 and 9 rows would take the registers.
// Large maps keep the two passes where those move the rows at the rate of memory and the one kernel re-walks too many: maps
// narrower than the window ([175,62,4,128] 5 x 5: 43 and 44 us against 50 and 49), windows of 7 and 9 beyond 2 million
// values ([25,116,107,32] 7 x 7: 63 and 75 us against 89 and 143; [20,43,97,32], 2.7 million, 40 and 42 against 23 and 20) and
// the forward pass of 5 x 5 beyond 8 million ([78,88,83,32]: 97 us against 109; [132,38,44,48] 72 against 49).  The number of
// values is a coarse line, drawn where no map gets slower by much rather than where most get faster: beyond it the walk would be
// faster on 57 of 81 maps with windows of 7 and 9, by up to 2 times, and slower on 20, down to 0.54; an estimate of the two
// passes beside that of the walk would tell them apart.  The two passes have no vectors where C is no multiple of four and
// are never faster there ([20,20,44,130]: 62 and 65 us against 25 and 35).
template <bool GRAD>
int launch_both_stages(const Args &a, int B, hipStream_t s, const char *where, bool *done) {
    *done = false;
    const long long values = (long long)B * a.H * a.W * a.C;
    const bool pairs = a.C % 2 == 0, quads = a.C % 4 == 0 && values >= (1 << 19);
    if (a.C % 4 == 0 && ((values > (1 << 20) && a.W < a.ks) || (values > (1 << 21) && a.ks >= 7) ||
                         (values > (1 << 23) && a.ks == 5 && !GRAD)))
        return LC_OK;
#define LC_WIDTH(K, V) if (a.ks == K) return launch_two_stage<GRAD, V, K>(a, B, s, where, done)
    if (quads) { LC_WIDTH(3, 4); if constexpr (GRAD) LC_WIDTH(5, 4); }
    if (pairs) { LC_WIDTH(3, 2); LC_WIDTH(5, 2); LC_WIDTH(7, 2); }
    LC_WIDTH(3, 1); LC_WIDTH(5, 1); LC_WIDTH(7, 1); LC_WIDTH(9, 1);
#undef LC_WIDTH
    return LC_OK;
}

}  // namespace

size_t lcn_variant_scratch_bytes(int B, int H, int W, int C, unsigned flags) {
    if (!(flags & LCN_TWO_STAGE)) return 0;
    return (size_t)B * H * W * ((flags & LCN_PER_CHANNEL) ? C : 1) * sizeof(float);
}

int launch_lcn_variant_fwd(const float *x, float *y, float *mu, float *rstd, int B, int H, int W, int C, int ks,
                           float sigma, float eps, unsigned flags, hipStream_t s) {
    const bool pc = flags & LCN_PER_CHANNEL, zp = flags & LCN_ZERO_PAD, two = flags & LCN_TWO_STAGE;
    if (!pc) {
        return launch_lcn(two ? 2 : 0, x, nullptr, y, mu, rstd, B, H, W, C, ks, sigma, eps, s, zp);
    }
    Args a{};
    if (!make_taps(ks, sigma, &a.taps)) return LC_EINVAL;
    a.x = x; a.out = y; a.mu_out = mu; a.rstd_out = rstd; a.mu_in = mu;
    a.H = H; a.W = W; a.C = C; a.ks = ks; a.zpad = zp; a.eps = eps;
    if (!two) return launch_pass<kFwdOne>(a, B, s, "lcn_variant_fwd");
    bool done;
    if (int rc = launch_both_stages<false>(a, B, s, "lcn_variant_fwd (two stages)", &done)) return rc;
    if (done) return LC_OK;
    if (int rc = launch_pass<kMean>(a, B, s, "lcn_variant_fwd (mean)")) return rc;
    return launch_pass<kDivide>(a, B, s, "lcn_variant_fwd (divide)");
}

int launch_lcn_variant_bwd(const float *x, const float *mu, const float *rstd, const float *dy, float *dx, int B, int H,
                           int W, int C, int ks, float sigma, unsigned flags, void *ws, size_t ws_bytes, hipStream_t s) {
    const bool pc = flags & LCN_PER_CHANNEL, zp = flags & LCN_ZERO_PAD, two = flags & LCN_TWO_STAGE;
    if (two && (ws == nullptr || ws_bytes < lcn_variant_scratch_bytes(B, H, W, C, flags))) return LC_EWORKSPACE;
    float *mu_ = const_cast<float *>(mu), *rstd_ = const_cast<float *>(rstd);   // read only in these modes
    if (!pc) {
        return launch_lcn(two ? 3 : 1, x, dy, dx, mu_, rstd_, B, H, W, C, ks, sigma, 0.f, s, zp);
    }
    Args a{};
    if (!make_taps(ks, sigma, &a.taps)) return LC_EINVAL;
    a.x = x; a.dy = dy; a.mu_in = mu; a.rstd_in = rstd; a.out = dx; a.field = (float *)ws;
    a.H = H; a.W = W; a.C = C; a.ks = ks; a.zpad = zp;
    if (!two) return launch_pass<kBwdOne>(a, B, s, "lcn_variant_bwd");
    bool done;
    if (int rc = launch_both_stages<true>(a, B, s, "lcn_variant_bwd (two stages)", &done)) return rc;
    if (done) return LC_OK;
    if (int rc = launch_pass<kBwdTwoA>(a, B, s, "lcn_variant_bwd (dv)")) return rc;
    return launch_pass<kBwdTwoB>(a, B, s, "lcn_variant_bwd (mean)");
}

}  // namespace lc

// ---------------------------------------------------------------------------------------------
// lcn_variant_bwd_static: lcn_variant_bwd for callers that cannot allocate.  The scratch field of the two-stage
// gradient (one float per statistic) lives in a file-scope device array instead of a caller's workspace.  Every GPU
// the library runs on holds its own copy of the array at its own address until the process ends; the address is
// looked up once per device, on the first call there, and only that pointer (never the array's name, which in host
// code is a stand-in and no device address) is handed to the kernels.  Nothing in the array has to start at zero:
// the first pass writes every element the second pass reads.
namespace lc {
namespace {

constexpr size_t kStaticScratchBytes = (size_t)LCN_STATIC_SCRATCH_BYTES;
__device__ __align__(256) unsigned char lcn_static_scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

// the calling thread's current device's copy of the array; LC_OK or LC_EHIP
int static_scratch(void **out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) { set_hip_error(e, "lcn_variant_bwd_static: hipGetDevice"); return LC_EHIP; }
    if (dev < 0 || dev >= kMaxDevices) { set_error_text("lcn_variant_bwd_static: device index out of range"); return LC_EHIP; }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(lcn_static_scratch));
        if (e != hipSuccess || !p) { set_hip_error(e, "lcn_variant_bwd_static: hipGetSymbolAddress"); return LC_EHIP; }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return LC_OK;
}

}  // namespace
}  // namespace lc

extern "C" int lcn_variant_bwd_static(const float *x, const float *mu, const float *rstd, const float *dy, float *dx,
                                      int32_t B, int32_t H, int32_t W, int32_t C, int32_t ksize, float gauss_sigma,
                                      uint32_t flags, void *hip_stream) {
    using namespace lc;
    if (int rc = check_lcn_variant_bwd_args(x, mu, rstd, dy, dx, B, H, W, C, ksize, gauss_sigma, flags)) return rc;
    const size_t need = lcn_variant_scratch_bytes(B, H, W, C, flags);
    if (need > kStaticScratchBytes) {
        set_error_text("lcn_variant_bwd_static: the two-stage gradient of this map needs more scratch than the "
                       "library's static array holds (LCN_STATIC_SCRATCH_BYTES); use lcn_variant_bwd with a workspace");
        return LC_EWORKSPACE;
    }
    void *scratch = nullptr;
    if (need > 0)
        if (int rc = static_scratch(&scratch)) return rc;
    return launch_lcn_variant_bwd(x, mu, rstd, dy, dx, B, H, W, C, ksize, gauss_sigma, flags, scratch, need,
                                  (hipStream_t)hip_stream);
}

