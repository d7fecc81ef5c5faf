// L2 pooling and local contrast normalisation, forward and backward.  Bandwidth-bound stencils over
// [B][H][W][C] activations: every kernel reads its inputs once from HBM (neighbour re-reads are served
// by L1/L2) and writes its output once.
//
// Pooling is not part of the paper's network (Sec. 3.1 leaves it out); LCN is applied after each layer
// (Sec. 3.1) and is taken here as Gaussian-windowed local standardisation with statistics pooled over
// the channels: the channel sums are wavefront reductions, the window sums a small LDS stencil.
#include <algorithm>
#include <type_traits>

#include "lc_common.hpp"

namespace lc {

// threads per workgroup of the band kernels: a band of whole image rows lives in their registers (512 threads with
// bands half as long measured the same)
constexpr int kBandThreads = 1024;

// ------------------------------------------------------------------ L2 pooling
template <int VEC>
__global__ __launch_bounds__(256) void l2pool_fwd_kernel(const float *__restrict__ x, float *__restrict__ y, int B,
                                                         int H, int W, int C, int Ho, int Wo, int ks, int st,
                                                         float eps, long long total) {
    const int CV = C / VEC;
    for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long long)gridDim.x * 256) {
        const int cv = (int)(e % CV);
        long long t = e / CV;
        const int j = (int)(t % Wo);
        t /= Wo;
        const int i = (int)(t % Ho), b = (int)(t / Ho);
        const float *xp = x + (((size_t)b * H + (size_t)i * st) * W + (size_t)j * st) * C + cv * VEC;
        float s[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) s[v] = 0.f;
        for (int p = 0; p < ks; ++p)
            for (int q = 0; q < ks; ++q) {
                const float *src = xp + ((size_t)p * W + q) * C;
                if (VEC == 4) {
                    const float4 t4 = *(const float4 *)src;
                    s[0] += t4.x * t4.x; s[1 % VEC] += t4.y * t4.y; s[2 % VEC] += t4.z * t4.z; s[3 % VEC] += t4.w * t4.w;
                } else {
                    s[0] += src[0] * src[0];
                }
            }
        float *dst = y + (size_t)e * VEC;
        if (VEC == 4)
            *(float4 *)dst = make_float4(sqrtf(eps + s[0]), sqrtf(eps + s[1 % VEC]), sqrtf(eps + s[2 % VEC]),
                                         sqrtf(eps + s[3 % VEC]));
        else
            dst[0] = sqrtf(eps + s[0]);
    }
}

template <int VEC>
__global__ __launch_bounds__(256) void l2pool_bwd_kernel(const float *__restrict__ x, const float *__restrict__ y,
                                                         const float *__restrict__ dy, float *__restrict__ dx, int B,
                                                         int H, int W, int C, int Ho, int Wo, int ks, int st,
                                                         long long total) {
    const int CV = C / VEC;
    for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < total; e += (long long)gridDim.x * 256) {
        const int cv = (int)(e % CV);
        long long t = e / CV;
        const int col = (int)(t % W);
        t /= W;
        const int row = (int)(t % H), b = (int)(t / H);
        // windows (i,j) with i*st <= row < i*st+ks
        const int i_hi = min(row / st, Ho - 1), j_hi = min(col / st, Wo - 1);
        const int i_lo = max(0, (row - ks + st) / st), j_lo = max(0, (col - ks + st) / st);
        float s[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) s[v] = 0.f;
        for (int i = i_lo; i <= i_hi; ++i)
            for (int j = j_lo; j <= j_hi; ++j) {
                const size_t o = (((size_t)b * Ho + i) * Wo + j) * C + cv * VEC;
                if (VEC == 4) {
                    const float4 g4 = *(const float4 *)(dy + o), y4 = *(const float4 *)(y + o);
                    s[0] += g4.x / y4.x; s[1 % VEC] += g4.y / y4.y; s[2 % VEC] += g4.z / y4.z; s[3 % VEC] += g4.w / y4.w;
                } else {
                    s[0] += dy[o] / y[o];
                }
            }
        const size_t xo = (size_t)e * VEC;
        if (VEC == 4) {
            const float4 x4 = *(const float4 *)(x + xo);
            *(float4 *)(dx + xo) = make_float4(x4.x * s[0], x4.y * s[1 % VEC], x4.z * s[2 % VEC], x4.w * s[3 % VEC]);
        } else {
            dx[xo] = x[xo] * s[0];
        }
    }
}

// Stride-1 windows, C % 4 == 0: a thread owns OW consecutive output columns of one (image, row, channel
// quad) and keeps the per-column partial sums in registers, so every input is loaded ks times (once
// per output row it belongs to) instead of ks*ks times.
constexpr int kPoolOW = 4;
constexpr int kPoolMaxK = 5;

__global__ __launch_bounds__(256) void l2pool_fwd_rows_kernel(const float *__restrict__ x, float *__restrict__ y,
                                                              int H, int W, int C, int Ho, int Wo, int ks, float eps,
                                                              int groups) {
    // grid: x over (output row, column group, channel quad) of one image, y = image
    const int CV = C >> 2;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= Ho * groups * CV) return;
    const int t = e / CV, cv = e - t * CV;
    const int i = t / groups, jg = t - i * groups;
    const int b = blockIdx.y;
    const int j0 = jg * kPoolOW;
    const int ncol = min(kPoolOW, Wo - j0) + ks - 1;          // input columns this thread needs
    f32x4 col[kPoolOW + kPoolMaxK - 1];
#pragma unroll
    for (int c = 0; c < kPoolOW + kPoolMaxK - 1; ++c) col[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
    const float *xp = x + (((size_t)b * H + i) * W + j0) * C + cv * 4;
    for (int p = 0; p < ks; ++p) {
#pragma unroll
        for (int c = 0; c < kPoolOW + kPoolMaxK - 1; ++c) {
            if (c < ncol) {
                const f32x4 v = *(const f32x4 *)(xp + ((size_t)p * W + c) * C);
                col[c] += v * v;
            }
        }
    }
    float *yp = y + (((size_t)b * Ho + i) * Wo + j0) * C + cv * 4;
#pragma unroll
    for (int o = 0; o < kPoolOW; ++o) {
        if (j0 + o < Wo) {
            f32x4 sacc = (f32x4){eps, eps, eps, eps};
#pragma unroll
            for (int q = 0; q < kPoolMaxK; ++q)
                if (q < ks) sacc += col[o + q];
            *(f32x4 *)(yp + (size_t)o * C) =
                (f32x4){sqrtf(sacc[0]), sqrtf(sacc[1]), sqrtf(sacc[2]), sqrtf(sacc[3])};
        }
    }
}

// Backward, same shapes: a thread owns OW consecutive input columns of one (image, row, channel quad); the
// per-column sums of dy/y over the output rows that cover this input row are kept in registers.
__global__ __launch_bounds__(256) void l2pool_bwd_rows_kernel(const float *__restrict__ x, const float *__restrict__ y,
                                                              const float *__restrict__ dy, float *__restrict__ dx,
                                                              int H, int W, int C, int Ho, int Wo, int ks, int groups) {
    // grid: x over (input row, column group, channel quad) of one image, y = image
    const int CV = C >> 2;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e >= H * groups * CV) return;
    const int t = e / CV, cv = e - t * CV;
    const int row = t / groups, jg = t - row * groups;
    const int b = blockIdx.y;
    const int c0 = jg * kPoolOW;                               // first input column
    const int i_lo = max(0, row - ks + 1), i_hi = min(row, Ho - 1);
    // output columns jo in [c0-ks+1, c0+OW-1] may cover this thread's inputs
    f32x4 col[kPoolOW + kPoolMaxK - 1];
#pragma unroll
    for (int c = 0; c < kPoolOW + kPoolMaxK - 1; ++c) col[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
    for (int i = i_lo; i <= i_hi; ++i) {
        const size_t rb = (((size_t)b * Ho + i) * Wo) * C + cv * 4;
#pragma unroll
        for (int c = 0; c < kPoolOW + kPoolMaxK - 1; ++c) {
            const int jo = c0 - (ks - 1) + c;
            if (c < kPoolOW + ks - 1 && jo >= 0 && jo < Wo) {
                const f32x4 g = *(const f32x4 *)(dy + rb + (size_t)jo * C), yy = *(const f32x4 *)(y + rb + (size_t)jo * C);
                col[c] += g / yy;
            }
        }
    }
    const size_t xo = (((size_t)b * H + row) * W + c0) * C + cv * 4;
#pragma unroll
    for (int o = 0; o < kPoolOW; ++o) {
        if (c0 + o < W) {
            // input column c0+o is covered by output columns jo = c0+o-ks+1 .. c0+o, i.e. col[o .. o+ks-1]
            f32x4 sacc = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int q = 0; q < kPoolMaxK; ++q)
                if (q < ks) sacc += col[o + q];
            *(f32x4 *)(dx + xo + (size_t)o * C) = *(const f32x4 *)(x + xo + (size_t)o * C) * sacc;
        }
    }
}

// Tiled variant for stride-1 windows and C % 4 == 0: a workgroup stages the (TH+ks-1) x (TW+ks-1) patch its
// TH x TW tile needs in LDS once (forward: x^2; backward: dy/y), so every input leaves L2 about once instead
// of once per window row, and the window sums come out of LDS.
constexpr int kPoolTH = 8, kPoolTW = 16;

// MODE 0: y = sqrt(eps + window sum of x^2) on a tile of outputs.
// MODE 1: dx = x * (window sum of dy/y) on a tile of inputs; the patch holds dy/y at outputs
//         (row-ks+1 .. row, col-ks+1 .. col), zero where no such output exists.
// MODE 2: the same with dy/y handed in as one array (in `dy`; `y` is not read).
template <int MODE>
__global__ __launch_bounds__(256) void l2pool_tile_kernel(const float *__restrict__ x, const float *__restrict__ y,
                                                          const float *__restrict__ dy, float *__restrict__ out,
                                                          int H, int W, int C, int Ho, int Wo, int ks, float eps,
                                                          int tiles_w, int tiles_per_img) {
    extern __shared__ __attribute__((aligned(16))) float patch[];   // [(TH+ks-1)*(TW+ks-1)][C]
    const int tid = threadIdx.x, CV = C >> 2;
    // each XCD walks a contiguous range of tiles: the tiles of one image, whose halos overlap, share an L2
    const int blk = remap_xcd(blockIdx.x, gridDim.x);
    const int b = blk / tiles_per_img, tile = blk - b * tiles_per_img;
    const int ti = (tile / tiles_w) * kPoolTH, tj = (tile % tiles_w) * kPoolTW;
    const int PH = kPoolTH + ks - 1, PW = kPoolTW + ks - 1;
    // patch origin in the source grid: forward reads inputs (ti.., tj..); backward reads outputs (ti-ks+1.., tj-ks+1..)
    const int oi0 = MODE == 0 ? ti : ti - (ks - 1), oj0 = MODE == 0 ? tj : tj - (ks - 1);
    const int SH = MODE == 0 ? H : Ho, SW = MODE == 0 ? W : Wo;
    const size_t sbase = (size_t)b * SH * SW;
    // eight loads in flight per thread before the first goes to LDS
    const int npatch = PH * PW * CV;
    for (int e0 = tid; e0 < npatch; e0 += 256 * 8) {
        f32x4 v[8], v2[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int e = e0 + 256 * q;
            const int cv = e % CV, pp = e / CV;
            const int pi = pp / PW, pj = pp - pi * PW;
            const int r = oi0 + pi, c = oj0 + pj;
            v[q] = (f32x4){0.f, 0.f, 0.f, 0.f};
            v2[q] = (f32x4){1.f, 1.f, 1.f, 1.f};
            if (e < npatch && r >= 0 && r < SH && c >= 0 && c < SW) {
                const size_t o = (sbase + (size_t)r * SW + c) * C + cv * 4;
                if (MODE == 0) {
                    v[q] = *(const f32x4 *)(x + o);
                } else {
                    v[q] = *(const f32x4 *)(dy + o);
                    if (MODE == 1) v2[q] = *(const f32x4 *)(y + o);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int e = e0 + 256 * q;
            if (e < npatch) *(f32x4 *)(patch + (size_t)e * 4) = MODE == 0 ? v[q] * v[q] : MODE == 1 ? v[q] / v2[q] : v[q];
        }
    }
    __syncthreads();
    // a thread owns 4 consecutive columns of one tile row and channel quad
    const int OH = MODE == 0 ? Ho : H, OWid = MODE == 0 ? Wo : W;
    for (int e = tid; e < kPoolTH * (kPoolTW / 4) * CV; e += 256) {
        const int cv = e % CV, t = e / CV;
        const int cg = t % (kPoolTW / 4), tr = t / (kPoolTW / 4);
        const int row = ti + tr, col0 = tj + cg * 4;
        if (row >= OH || col0 >= OWid) continue;
        f32x4 col[4 + kPoolMaxK - 1];
#pragma unroll
        for (int c = 0; c < 4 + kPoolMaxK - 1; ++c) col[c] = (f32x4){0.f, 0.f, 0.f, 0.f};
        for (int p = 0; p < ks; ++p) {
            const float *prow = patch + ((size_t)(tr + p) * PW + cg * 4) * C + cv * 4;
#pragma unroll
            for (int c = 0; c < 4 + kPoolMaxK - 1; ++c)
                if (c < 4 + ks - 1) col[c] += *(const f32x4 *)(prow + (size_t)c * C);
        }
        const size_t o = (((size_t)b * OH + row) * OWid + col0) * C + cv * 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (col0 + q >= OWid) continue;
            f32x4 sacc = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < kPoolMaxK; ++k)
                if (k < ks) sacc += col[q + k];
            if (MODE == 0) {
                *(f32x4 *)(out + o + (size_t)q * C) =
                    (f32x4){sqrtf(eps + sacc[0]), sqrtf(eps + sacc[1]), sqrtf(eps + sacc[2]), sqrtf(eps + sacc[3])};
            } else {
                *(f32x4 *)(out + o + (size_t)q * C) = *(const f32x4 *)(x + o + (size_t)q * C) * sacc;
            }
        }
    }
}

// Forward pooling as a stream, stride 1 and a KS x KS window: a thread owns one output column and channel quad
// and walks down RS output rows.  Each input row it meets gives one horizontal sum of squares (KS loads whose
// neighbours in the wave read the same lines); the last KS-1 of them stay in registers, so an output costs one new
// row of loads.  No LDS and no barriers: every wave reads and writes all the time, and the loads of RU rows are in
// flight together.  Segments of RS rows re-read KS-1 input rows of the segment above.
template <int KS, int RU>
__global__ __launch_bounds__(256) void l2pool_fwd_stream_kernel(const float *__restrict__ x, float *__restrict__ y,
                                                                int H, int W, int CV, int Ho, int Wo, int RS,
                                                                int nseg, float eps, long long total) {
    const long long e = (long long)remap_xcd(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
    if (e >= total) return;
    const int per_row = Wo * CV;
    const int cj = (int)(e % per_row);
    const long long t = e / per_row;
    const int sg = (int)(t % nseg), b = (int)(t / nseg);
    const int ro0 = sg * RS, ro1 = min(ro0 + RS, Ho);
    const size_t xrow = (size_t)W * CV, yrow = (size_t)Wo * CV;     // row strides in float4
    const f32x4 *xp = (const f32x4 *)x + (size_t)b * H * xrow + cj;  // column j, quad cv: offset j*CV + cv = cj
    f32x4 *yp = (f32x4 *)y + (size_t)b * Ho * yrow + cj;
    f32x4 ring[KS - 1];
#pragma unroll
    for (int d = 0; d < KS - 1; ++d) {
        const f32x4 *p = xp + (size_t)min(ro0 + d, H - 1) * xrow;
        f32x4 h = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int dj = 0; dj < KS; ++dj) { const f32x4 v = p[dj * CV]; h += v * v; }
        ring[d] = h;
    }
    for (int ro = ro0; ro < ro1; ro += RU) {
        f32x4 v[RU][KS];
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            // rows past the segment are read from the last input row and never stored
            const f32x4 *p = xp + (size_t)min(ro + u + KS - 1, H - 1) * xrow;
#pragma unroll
            for (int dj = 0; dj < KS; ++dj) v[u][dj] = p[dj * CV];
        }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            f32x4 h = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int dj = 0; dj < KS; ++dj) h += v[u][dj] * v[u][dj];
            f32x4 sacc = h;
#pragma unroll
            for (int d = 0; d < KS - 1; ++d) sacc += ring[d];
            if (ro + u < ro1)
                yp[(size_t)(ro + u) * yrow] = (f32x4){sqrtf(eps + sacc[0]), sqrtf(eps + sacc[1]),
                                                      sqrtf(eps + sacc[2]), sqrtf(eps + sacc[3])};
#pragma unroll
            for (int d = 0; d + 1 < KS - 1; ++d) ring[d] = ring[d + 1];
            ring[KS - 2] = h;
        }
    }
}

// Backward pooling as a stream, stride 1 and a KS x KS window: a thread owns one input column and channel quad and walks
// down RS rows.  Each output row it meets gives one horizontal sum of dy/y over the KS output columns that cover the
// column; the last KS-1 of them stay in registers.  DIV: dy and y are two arrays; otherwise dy/y is handed in as one.  A
// quotient is formed KS times, which still takes less than the arrays' way from memory.
template <int KS, int RU, bool DIV>
__global__ __launch_bounds__(256) void l2pool_bwd_stream_kernel(const float *__restrict__ x, const float *__restrict__ y,
                                                                const float *__restrict__ dy, float *__restrict__ dx,
                                                                int H, int W, int CV, int Ho, int Wo, int RS, int nseg,
                                                                long long total) {
    const long long e = (long long)remap_xcd(blockIdx.x, gridDim.x) * 256 + threadIdx.x;
    if (e >= total) return;
    const int per_row = W * CV;
    const int cj = (int)(e % per_row), col = cj / CV;
    const long long t = e / per_row;
    const int sg = (int)(t % nseg), b = (int)(t / nseg);
    const int r0 = sg * RS, r1 = min(r0 + RS, H);
    const size_t xrow = (size_t)W * CV, yrow = (size_t)Wo * CV;     // row strides in float4
    const f32x4 *xp = (const f32x4 *)x + (size_t)b * H * xrow + cj;
    f32x4 *dp = (f32x4 *)dx + (size_t)b * H * xrow + cj;
    const size_t ybase = (size_t)b * Ho * yrow;
    int off[KS];
    bool in[KS];
#pragma unroll
    for (int d = 0; d < KS; ++d) {
        in[d] = col - d >= 0 && col - d < Wo;
        off[d] = min(max(col - d, 0), Wo - 1) * CV + (cj - col * CV);
    }
    // horizontal sum of output row i (zero outside the map); every lane loads, from an address clamped into it
    struct Raw { f32x4 g[KS], y[DIV ? KS : 1]; };
    auto fetch = [&](int i, Raw &v) {
        const size_t o = ybase + (size_t)min(max(i, 0), Ho - 1) * yrow;
#pragma unroll
        for (int d = 0; d < KS; ++d) {
            v.g[d] = ((const f32x4 *)dy)[o + off[d]];
            if constexpr (DIV) v.y[d] = ((const f32x4 *)y)[o + off[d]];
        }
    };
    auto sum = [&](int i, const Raw &v) -> f32x4 {
        f32x4 h = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int d = 0; d < KS; ++d) {
            f32x4 q = v.g[d];
            if constexpr (DIV) q = q / v.y[d];
            h += in[d] && i >= 0 && i < Ho ? q : (f32x4){0.f, 0.f, 0.f, 0.f};
        }
        return h;
    };
    f32x4 ring[KS - 1];
#pragma unroll
    for (int d = 0; d < KS - 1; ++d) {
        Raw v;
        fetch(r0 - (KS - 1) + d, v);
        ring[d] = sum(r0 - (KS - 1) + d, v);
    }
    for (int row = r0; row < r1; row += RU) {
        Raw v[RU];
        f32x4 xv[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            fetch(row + u, v[u]);
            xv[u] = xp[(size_t)min(row + u, H - 1) * xrow];
        }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const f32x4 h = sum(row + u, v[u]);
            f32x4 acc = h;
#pragma unroll
            for (int d = 0; d < KS - 1; ++d) acc += ring[d];
            if (row + u < r1) dp[(size_t)(row + u) * xrow] = xv[u] * acc;
#pragma unroll
            for (int d = 0; d + 1 < KS - 1; ++d) ring[d] = ring[d + 1];
            ring[KS - 2] = h;
        }
    }
}

// ------------------------------------------------------------------------ LCN
constexpr int kLcnTile = 16;   // output tile edge
constexpr int kLcnMaxK = 15;   // largest window
constexpr int kLcnHalo = kLcnTile + kLcnMaxK - 1;

struct GaussTaps { float g[kLcnMaxK]; };

__device__ __forceinline__ float group_sum(float v, int lpp) {
    for (int o = lpp >> 1; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// sum of the taps that stay inside [0,n) around position p (the normaliser of a window truncated at the border;
// with zero padding, zpad, the taps keep their full-window normalisation instead)
__device__ __forceinline__ float tap_norm(const GaussTaps &t, int p, int n, int r) {
    float z = 0.f;
    for (int d = -r; d <= r; ++d)
        if (p + d >= 0 && p + d < n) z += t.g[d + r];
    return z;
}

// Statistics pooled over the channels, tile by tile.  One stage: OP 0 forward (x -> mu, rstd, y), OP 1 gradient (x, mu, rstd,
// dy -> dx).  Two stages (subtract the window mean, divide by the root of the window mean of the neighbours' own squared
// differences), both in one kernel: OP 2 forward, OP 3 gradient.
//
// A workgroup takes a th x tw tile and a halo of one window radius, or of two.  Per-pixel sums over the channels come first:
// lpp lanes share a pixel, and a lane has NF vectors of each of PX pixels in flight.  The window sums of those run in LDS,
// rows first, then columns.  The two-stage forward pass forms the squared differences from the window means of tile and inner
// halo in a second round over x; the gradient needs none: the channel sum of dv is rstd sum(dy) + 2 s sum(x - mu), s the
// window sum of the variances' gradients.  The last round writes the tile, several vectors a lane in flight.
//
// VEC 4 with RAG takes channels that are no multiple of four: vectors at any element, the last one of a pixel starting at
// C - 4 and its elements that the one before it holds left out of the sums (they are written twice, alike).  VEC 1 is left
// for one to three channels.  DIVX (OP 1, VEC 4): leave dx / x.
// Bound by latency on small maps (a round of loads, a reduction and two window passes, one after the other) and by the reads
// of tile, halo and tile again on large ones.  Before, the two-stage form took two kernels each way that moved the mean, dv and its
// channel sums through memory, window sums took KS*KS steps, a group of lanes had one pixel in flight, and channels that are no
// multiple of four came one by one.  Over 300 maps (10 thousand to 20 million values, windows of 3 to 15) out of the caches and in
// them: two stages 1.55 and 1.73 times as fast forward, 1.79 and 2.01 backward; one stage 1.22 and 1.28, 1.22 and 1.33 (1.07 to
// 1.10 with windows up to 9 and channels in fours); the slowest 0.95 ([224,76,7,72], 13 x 13, gradient 42.3 -> 43.6 us in them).
constexpr int kLcnThreads = 1024;   // at most
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
template <int VEC, int OP, int NF, bool RAG, bool DIVX>
__global__ __launch_bounds__(kLcnThreads) void lcn_pooled_kernel(const float *__restrict__ x, const float *__restrict__ dy,
                                                         float *__restrict__ out, float *__restrict__ mu,
                                                         float *__restrict__ rstd, int H, int W, int C, int ks, float eps,
                                                         GaussTaps taps, int lpp, int th, int tw, int tiles_w,
                                                         int tiles_per_img, int zpad) {
    constexpr bool kGrad = OP == 1 || OP == 3, kTwo = OP >= 2;
    constexpr int PX = 8 / NF / (kGrad && NF < 4 ? 2 : 1), U = kGrad ? 4 : 8;
    const int nthr = blockDim.x;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ float zr[kLcnTile + 2 * kLcnMaxK], zc[kLcnTile + 2 * kLcnMaxK], gt[kLcnMaxK + 1];
    const int r = (ks - 1) / 2, R = kTwo ? 2 * r : r, hh = th + 2 * R, hw = tw + 2 * R;
    const int iw = tw + 2 * r, ih = th + 2 * r, hcols = hw - 2 * r;
    float *const m1 = lds, *const m2 = m1 + hh * hw;                       // sums per pixel of tile and halo
    float *const m3 = m2 + (OP == 2 ? 0 : hh * hw);
    float *const h1 = m3 + (OP == 3 ? hh * hw : 0), *const h2 = h1 + hh * hcols;   // row sums
    float *const n1 = h2 + (kTwo ? 0 : hh * hcols), *const n2 = n1 + (kTwo ? ih * iw : 0);   // inner halo: second window's
    float *const t1 = n2 + (OP == 2 ? ih * iw : 0), *const t2 = t1 + th * tw, *const tm = t2 + th * tw, *const tr = tm + th * tw;
    const int tid = threadIdx.x;
    // each XCD walks a contiguous range of tiles: the tiles of one image, whose halos overlap, share an L2
    const int blk = remap_xcd(blockIdx.x, gridDim.x);
    const int b = blk / tiles_per_img, tile = blk - b * tiles_per_img;
    const int ti = (tile / tiles_w) * th, tj = (tile % tiles_w) * tw;
    const int CV = VEC == 4 ? (C + 3) >> 2 : C;
    const size_t img = (size_t)b * H * W;
    if (tid < hh) zr[tid] = zpad ? 1.f : tap_norm(taps, ti - R + tid, H, r);
    else if (tid >= 64 && tid < 64 + hw) zc[tid - 64] = zpad ? 1.f : tap_norm(taps, tj - R + tid - 64, W, r);
    else if (tid >= 128 && tid < 128 + ks) gt[tid - 128] = taps.g[tid - 128];
    if (kGrad) __syncthreads();
    // a pixel's normaliser, by its place among the staged ones
    auto norm_at = [&](int hi, int hj) { return zr[hi] * zc[hj] * (float)C; };
    const float inv_tw = 1.0f / (float)tw, inv_hw = 1.0f / (float)hw, inv_iw = 1.0f / (float)iw, inv_hc = 1.0f / (float)hcols;
    auto divided = [&](int a, float inv) { return (int)(((float)a + 0.5f) * inv); };   // exact below 2^20

    typedef float fv __attribute__((ext_vector_type(VEC == 4 ? 4 : 2)));   // VEC = 1: the second component stays zero
    auto fetch = [&](const float *p) -> fv {
        if constexpr (VEC == 4 && RAG) return (fv)(*(const f32x4u *)p);
        else if constexpr (VEC == 4) return *(const fv *)p;
        else return (fv){*p, 0.f};
    };
    auto at = [&](int cv) { return RAG && cv == CV - 1 ? C - 4 : cv * VEC; };
    auto total = [&](const fv &v) -> float {
        if constexpr (VEC == 4) return (v[0] + v[1]) + (v[2] + v[3]);
        else return v[0];
    };
    const int grp = tid / lpp, gl = tid % lpp, ngrp = nthr / lpp, back = RAG ? 4 * CV - C : 0;

    // A round over the pixels of an area of ph x pw at (ti - ro, tj - ro), PX of them per group of lanes in flight.
    // SQ: sums of squared differences from n1, into n2; otherwise the sums of the first window, into m1 to m3.
    auto round = [&](int ph, int pw, float inv_pw, int ro, auto squares) {
        constexpr bool SQ = decltype(squares)::value;
        for (int base = grp; base < ph * pw; base += ngrp * PX) {
            size_t pix[PX];
            bool in[PX];
            float mp[PX], rsp[PX], s1[PX], s2[PX], s3[PX];
#pragma unroll
            for (int k = 0; k < PX; ++k) {
                const int hp = min(base + k * ngrp, ph * pw - 1), hi = divided(hp, inv_pw), hj = hp - hi * pw;
                const int row = ti - ro + hi, col = tj - ro + hj;
                in[k] = row >= 0 && row < H && col >= 0 && col < W;
                pix[k] = img + (in[k] ? (size_t)row * W + col : 0);        // outside: the image's first, left out below
                mp[k] = rsp[k] = s1[k] = s2[k] = s3[k] = 0.f;
                if constexpr (SQ) mp[k] = n1[hp];
                if constexpr (kGrad) { mp[k] = mu[pix[k]]; rsp[k] = rstd[pix[k]]; }
            }
            for (int c0 = gl; c0 < CV; c0 += NF * lpp) {
                fv v[PX][NF], d[kGrad ? PX : 1][NF];
#pragma unroll
                for (int k = 0; k < PX; ++k)
                    if (base + k * ngrp < ph * pw)
#pragma unroll
                    for (int u = 0; u < NF; ++u) {
                        const size_t o = pix[k] * C + at(min(c0 + u * lpp, CV - 1));   // past the end: the last again, left out below
                        v[k][u] = fetch(x + o);
                        if constexpr (kGrad) d[kGrad ? k : 0][u] = fetch(dy + o);
                    }
#pragma unroll
                for (int k = 0; k < PX; ++k)
#pragma unroll
                    for (int u = 0; u < NF; ++u) {
                        const int cv = c0 + u * lpp;
                        if (cv >= CV) continue;
                        fv e = v[k][u], dv = d[kGrad ? k : 0][u];
                        if constexpr (SQ || kGrad) {
#pragma unroll
                            for (int q = 0; q < VEC; ++q) e[q] -= mp[k];
                        }
                        if constexpr (RAG) {
                            const int skip = cv == CV - 1 ? back : 0;
#pragma unroll
                            for (int q = 0; q < 3; ++q)
                                if (q < skip) e[q] = dv[q] = 0.f;
                        }
                        if constexpr (kGrad) {
                            s1[k] += total(dv);
                            s2[k] += total(dv * e);
                            if (OP == 3) s3[k] += total(e);
                        } else if constexpr (SQ) {
                            s1[k] += total(e * e);
                        } else {
                            s1[k] += total(e);
                            if (OP == 0) s2[k] += total(e * e);
                        }
                    }
            }
            for (int o = lpp >> 1; o > 0; o >>= 1) {
#pragma unroll
                for (int k = 0; k < PX; ++k) {
                    s1[k] += __shfl_xor(s1[k], o, 64);
                    if (kGrad || OP == 0) s2[k] += __shfl_xor(s2[k], o, 64);
                    if (OP == 3) s3[k] += __shfl_xor(s3[k], o, 64);
                }
            }
            if (gl != 0) continue;
#pragma unroll
            for (int k = 0; k < PX; ++k) {
                const int hp = base + k * ngrp;
                if (hp >= ph * pw) continue;
                if constexpr (SQ) {
                    n2[hp] = in[k] ? 0.5f * s1[k] : 0.f;
                } else if constexpr (!kGrad) {
                    m1[hp] = in[k] ? 0.5f * s1[k] : 0.f;
                    if (OP == 0) m2[hp] = in[k] ? 0.5f * s2[k] : 0.f;
                } else {
                    const int hi = divided(hp, inv_pw), hj = hp - hi * pw;
                    const float z = norm_at(hi, hj), bc = rsp[k] * rsp[k] * rsp[k] * s2[k];
                    if (OP == 1) {
                        // this pixel's own normaliser and statistics, folded into the two maps of the transposed window sums
                        m1[hp] = in[k] ? 0.5f * ((bc * mp[k] - rsp[k] * s1[k]) / z) : 0.f;
                        m2[hp] = in[k] ? 0.5f * (bc / z) : 0.f;
                    } else {
                        m1[hp] = in[k] ? -0.25f * bc / z : 0.f;           // gradient of its variance, over its normaliser
                        m2[hp] = rsp[k] * s1[k];
                        m3[hp] = s3[k];
                    }
                    const int oi = hi - ro, oj = hj - ro;
                    if (oi >= 0 && oi < th && oj >= 0 && oj < tw) { tm[oi * tw + oj] = mp[k]; tr[oi * tw + oj] = rsp[k]; }
                }
            }
        }
    };
    // window sums along the rows: of mh x (ow + 2r) values, mh x ow
    auto along = [&](const float *m, const float *q, float *h, float *hq, int mh, int ow, float inv_ow, auto both) {
        constexpr bool TWO = decltype(both)::value;
        const int mw = ow + 2 * r;
        for (int e = tid; e < mh * ow; e += nthr) {
            const int i = divided(e, inv_ow), o = i * mw + (e - i * ow) + r;
            float s = gt[r] * m[o], s2 = TWO ? gt[r] * q[o] : 0.f;
#pragma unroll 2
            for (int d = 1; d <= r; ++d) {
                const float g = gt[r + d];
                s += g * (m[o - d] + m[o + d]);
                if (TWO) s2 += g * (q[o - d] + q[o + d]);
            }
            h[e] = s;
            if (TWO) hq[e] = s2;
        }
    };
    // and down a column of them, around element o.  What the windows sum lies in LDS halved: the two values of a tap meet
    // before they are weighted, and their sum leaves the range of a float where the window's mean does not.
    auto down = [&](const float *h, int o, int ow) -> float {
        float s = gt[r] * h[o];
#pragma unroll 2
        for (int d = 1; d <= r; ++d) s += gt[r + d] * (h[o - d * ow] + h[o + d * ow]);
        return 2.f * s;
    };

    // both at once around element o of mh x hw values, for 3 x 3 windows of one stage: a barrier less for six reads more
    auto nine = [&](const float *m, int o) -> float {
        auto row = [&](int p) { return __fmaf_rn(gt[2], m[p - 1] + m[p + 1], gt[1] * m[p]); };
        return 2.f * __fmaf_rn(gt[2], row(o - hw) + row(o + hw), gt[1] * row(o));
    };

    round(hh, hw, inv_hw, R, std::false_type{});
    __syncthreads();
    const bool three = !kTwo && r == 1;
    if (!three) {
        along(m1, m2, h1, h2, hh, hcols, inv_hc, std::bool_constant<!kTwo>{});
        __syncthreads();
    }
    if constexpr (!kTwo) {
        for (int e = tid; e < th * tw; e += nthr) {
            const int oi = divided(e, inv_tw), oj = e - oi * tw, row = ti + oi, col = tj + oj;
            if (row >= H || col >= W) continue;
            const int o = (oi + 1) * hw + oj + 1;
            const float s1 = three ? nine(m1, o) : down(h1, e + r * tw, tw), s2 = three ? nine(m2, o) : down(h2, e + r * tw, tw);
            if (OP == 0) {
                const float z = norm_at(oi + R, oj + R), m = s1 / z, var = fmaxf(s2 / z - m * m, 0.f);
                const float rs = 1.0f / sqrtf(var + eps);
                const size_t pix = img + (size_t)row * W + col;
                mu[pix] = m;
                rstd[pix] = rs;
                t1[e] = m;
                t2[e] = rs;
            } else {
                t1[e] = s1;
                t2[e] = s2;
            }
        }
    } else {
        for (int e = tid; e < ih * iw; e += nthr) {
            const int i = divided(e, inv_iw), j = e - i * iw, row = ti - r + i, col = tj - r + j;
            const bool in = row >= 0 && row < H && col >= 0 && col < W, own = in && i >= r && i < r + th && j >= r && j < r + tw;
            const float s = down(h1, e + r * iw, iw), z = norm_at(i + r, j + r);
            if (OP == 2) {
                const float m = in ? s / z : 0.f;
                n1[e] = m;
                if (own) {
                    mu[img + (size_t)row * W + col] = m;
                    t1[(i - r) * tw + j - r] = m;
                }
            } else {
                const int o = (i + r) * hw + j + r;
                n1[e] = in ? 0.5f * ((m2[o] + 2.f * s * m3[o]) / z) : 0.f;
                if (own) t2[(i - r) * tw + j - r] = 2.f * s;
            }
        }
        __syncthreads();
        if constexpr (OP == 2) {
            round(ih, iw, inv_iw, r, std::true_type{});
            __syncthreads();
        }
        along(OP == 2 ? n2 : n1, nullptr, h1, nullptr, ih, tw, inv_tw, std::false_type{});
        __syncthreads();
        for (int e = tid; e < th * tw; e += nthr) {
            const int oi = divided(e, inv_tw), oj = e - oi * tw, row = ti + oi, col = tj + oj;
            if (row >= H || col >= W) continue;
            const float s = down(h1, e + r * tw, tw);
            if (OP == 2) {
                const float rs = 1.0f / sqrtf(s / norm_at(oi + R, oj + R) + eps);
                rstd[img + (size_t)row * W + col] = rs;
                t2[e] = rs;
            } else {
                t1[e] = s;
            }
        }
    }
    __syncthreads();

    // the tile's outputs
    const int count = th * tw * CV;
    for (int e0 = tid; e0 < count; e0 += nthr * U) {
        fv xv[U], d[kGrad ? U : 1];
        size_t o[U];
        int op[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int e = e0 + nthr * k;
            op[k] = -1;
            if (e >= count) continue;
            const int px = e / CV, cv = e - px * CV, oi = divided(px, inv_tw), oj = px - oi * tw;
            const int row = ti + oi, col = tj + oj;
            if (row >= H || col >= W) continue;
            op[k] = px;
            o[k] = (img + (size_t)row * W + col) * C + at(cv);
            xv[k] = fetch(x + o[k]);
            if constexpr (kGrad) d[kGrad ? k : 0] = fetch(dy + o[k]);
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (op[k] < 0) continue;
            const float u = t1[op[k]], v = t2[op[k]];
            fv g;
            if constexpr (!kGrad) {
                g = (xv[k] - u) * v;
            } else {
                const fv dv = d[kGrad ? k : 0];
                if (OP == 1) g = dv * tr[op[k]] + u - xv[k] * v;
                else g = dv * tr[op[k]] + (xv[k] - tm[op[k]]) * v - u;
                if constexpr (DIVX) g = g / xv[k];            // the quotient the pooling gradient takes (x is its output)
            }
            if constexpr (VEC == 4 && RAG) *(f32x4u *)(out + o[k]) = g;
            else if constexpr (VEC == 4) *(fv *)(out + o[k]) = g;
            else out[o[k]] = g[0];
        }
    }
}

// Forward pass for C = 4*LPP channels with LPP in {2, 4, 8}: a pixel is exactly one float4 per lane of its group,
// so the tile's own pixels are loaded once, in phase 1, and stay in registers for phase 3; only the halo ring is
// read a second time by the neighbouring tiles.  (The backward pass would keep twice the registers and measured
// slower this way than re-reading the tile.)
template <int LPP>
__global__ __launch_bounds__(256) void lcn_fwd_cached_kernel(const float *__restrict__ x, float *__restrict__ out,
                                                             float *__restrict__ mu, float *__restrict__ rstd, int H,
                                                             int W, int ks, float eps, GaussTaps taps, int tiles_w,
                                                             int tiles_per_img, int zpad) {
    constexpr int C = 4 * LPP, NG = 256 / LPP, NI = LPP;   // NG pixel groups; NI passes cover the 256 tile pixels
    __shared__ float m1[kLcnHalo * kLcnHalo], m2[kLcnHalo * kLcnHalo];
    __shared__ float t1[kLcnTile * kLcnTile], t2[kLcnTile * kLcnTile];
    const int r = (ks - 1) / 2, halo = kLcnTile + 2 * r;
    const int tid = threadIdx.x, grp = tid / LPP, gl = tid % LPP;
    // each XCD walks a contiguous range of tiles: the tiles of one image, whose halos overlap, share an L2
    const int blk = remap_xcd(blockIdx.x, gridDim.x);
    const int b = blk / tiles_per_img, tile = blk - b * tiles_per_img;
    const int ti = (tile / tiles_w) * kLcnTile, tj = (tile % tiles_w) * kLcnTile;
    const size_t img = (size_t)b * H * W;
    // window normalisers of the tile's rows and columns (read after phase 1's barrier)
    __shared__ float zr[kLcnTile], zc[kLcnTile];
    if (tid < kLcnTile) zr[tid] = zpad ? 1.f : tap_norm(taps, ti + tid, H, r);
    else if (tid >= 64 && tid < 64 + kLcnTile) zc[tid - 64] = zpad ? 1.f : tap_norm(taps, tj + tid - 64, W, r);

    // one halo pixel's channel sums -> the two maps of phase 2 (lane 0 of the group writes)
    auto put = [&](int hp, const float4 &v) {
        const float a = group_sum((v.x + v.y) + (v.z + v.w), LPP);
        const float c2 = group_sum((v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w), LPP);
        if (gl == 0) {
            m1[hp] = a;
            m2[hp] = c2;
        }
    };

    // phase 1a: the tile's own pixels, kept in registers (zeros outside the image)
    float4 xv[NI];
    bool inv[NI];
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const int op = grp + it * NG, oi = op / kLcnTile, oj = op % kLcnTile;
        const int row = ti + oi, col = tj + oj;
        inv[it] = row < H && col < W;
        xv[it] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (inv[it]) xv[it] = *(const float4 *)(x + (img + (size_t)row * W + col) * C + gl * 4);
    }
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const int op = grp + it * NG, oi = op / kLcnTile, oj = op % kLcnTile;
        put((oi + r) * halo + oj + r, xv[it]);
    }
    // phase 1b: the halo ring around the tile
    for (int hp = grp; hp < halo * halo; hp += NG) {
        const int hi = hp / halo, hj = hp - hi * halo;
        if (hi >= r && hi < r + kLcnTile && hj >= r && hj < r + kLcnTile) continue;   // uniform over the group
        const int row = ti - r + hi, col = tj - r + hj;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (row >= 0 && row < H && col >= 0 && col < W) v = *(const float4 *)(x + (img + (size_t)row * W + col) * C + gl * 4);
        put(hp, v);
    }
    __syncthreads();

    // phase 2: window sums and statistics, one thread per output pixel
    {
        const int oi = tid / kLcnTile, oj = tid % kLcnTile;
        const int row = ti + oi, col = tj + oj;
        if (row < H && col < W) {
            float s1 = 0.f, s2 = 0.f;
            for (int p = 0; p < ks; ++p)
                for (int q = 0; q < ks; ++q) {
                    const float wt = taps.g[p] * taps.g[q];
                    const int hp = (oi + p) * halo + oj + q;
                    s1 += wt * m1[hp];   // out-of-image halo entries are zero
                    s2 += wt * m2[hp];
                }
            const float z = zr[oi] * zc[oj] * (float)C;
            const float m = s1 / z, q2 = s2 / z;
            const float var = fmaxf(q2 - m * m, 0.f);
            const float rs = 1.0f / sqrtf(var + eps);
            const size_t pix = img + (size_t)row * W + col;
            mu[pix] = m;
            rstd[pix] = rs;
            t1[tid] = m;
            t2[tid] = rs;
        }
    }
    __syncthreads();

    // phase 3: normalise the registers of phase 1a
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        if (!inv[it]) continue;
        const int op = grp + it * NG, oi = op / kLcnTile, oj = op % kLcnTile;
        const size_t pix = img + (size_t)(ti + oi) * W + tj + oj;
        const float u = t1[op], v = t2[op];
        const float4 xq = xv[it];
        *(float4 *)(out + pix * C + gl * 4) = make_float4((xq.x - u) * v, (xq.y - u) * v, (xq.z - u) * v, (xq.w - u) * v);
    }
}

// Band kernels for the one-stage pooled form, C = 4*LPP channels (LPP a power of two up to 16): a workgroup owns
// RB whole rows of one image.  Its own pixels are loaded once and stay in registers (NV float4 per thread, of x and,
// backward, of dy); only the (ks-1)/2 rows above and below the band are read a second time by the neighbouring
// bands, so a 5x5 window over a band of 22 rows re-reads 18 % of the input where a 16x16 tile re-reads 56 %.
// The maps of per-pixel channel sums carry a margin of (ks-1)/2 zero columns on both sides: phase 2 has no bounds
// checks.  MODE 0: forward (x -> y, mu, rstd).  MODE 1: backward (x, mu, rstd, dy -> dx).
template <int LPP, int MODE, int NTHR, int NV>
__global__ __launch_bounds__(NTHR) void lcn_band_kernel(const float *__restrict__ x, const float *__restrict__ dy,
                                                        float *__restrict__ out, float *__restrict__ mu,
                                                        float *__restrict__ rstd, int H, int W, int ks, float eps,
                                                        GaussTaps taps, int RB, int bands, int zpad, int divx) {
    constexpr int C = 4 * LPP, NH = 2;
    extern __shared__ __attribute__((aligned(16))) float band_lds[];
    const int r = (ks - 1) / 2, MW = W + 2 * r, MH = RB + 2 * r;
    float *m1 = band_lds, *m2 = m1 + MH * MW, *t1 = m2 + MH * MW, *t2 = t1 + RB * W;
    float *zr = t2 + RB * W, *zc = zr + MH;                       // window normalisers of the staged rows, of all columns
    const int tid = threadIdx.x, gl = tid % LPP;
    const int blk = remap_xcd(blockIdx.x, gridDim.x);             // the bands of one image stay in one XCD
    const int b = blk / bands, r0 = (blk - b * bands) * RB;
    const size_t img = (size_t)b * H * W;
    const int npix = RB * W;

    for (int i = tid; i < MH + W; i += NTHR) {
        if (i < MH) zr[i] = zpad ? 1.f : tap_norm(taps, r0 - r + i, H, r);
        else zc[i - MH] = zpad ? 1.f : tap_norm(taps, i - MH, W, r);
    }
    // map cells outside the image are zero; every other cell is written exactly once below
    for (int cell = tid; cell < MH * MW; cell += NTHR) {
        const int hi = cell / MW, hj = cell - hi * MW;
        const int row = r0 - r + hi, col = hj - r;
        if (row < 0 || row >= H || col < 0 || col >= W) m1[cell] = m2[cell] = 0.f;
    }
    if (MODE == 1) __syncthreads();                               // the backward maps use zr and zc

    // channel sums of one pixel (all LPP lanes of its group call this) -> the two maps of phase 2
    auto put = [&](int row, int col, bool in, const float4 &v, const float4 &d) {
        float a, c2;
        float mp = 0.f, rsp = 0.f;
        if (MODE == 0) {
            a = (v.x + v.y) + (v.z + v.w);
            c2 = (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
        } else {
            if (in) { mp = mu[img + (size_t)row * W + col]; rsp = rstd[img + (size_t)row * W + col]; }
            a = (d.x + d.y) + (d.z + d.w);
            c2 = (d.x * (v.x - mp) + d.y * (v.y - mp)) + (d.z * (v.z - mp) + d.w * (v.w - mp));
        }
        a = group_sum(a, LPP);
        c2 = group_sum(c2, LPP);
        if (gl == 0 && in) {
            const int cell = (row - r0 + r) * MW + col + r;
            if (MODE == 0) {
                m1[cell] = a;
                m2[cell] = c2;
            } else {
                // this pixel's own normaliser and statistics folded into what the transposed window sums need
                const float z = zr[row - r0 + r] * zc[col] * (float)C;
                const float bc = rsp * rsp * rsp * c2;
                m1[cell] = (bc * mp - rsp * a) / z;
                m2[cell] = bc / z;
            }
        }
    };

    // phase 1: every load of the workgroup is issued before the first reduction: the band's own pixels, kept in
    // registers, and NH rounds of the rows above and below the band (further rounds, if any, follow)
    float4 xv[NV], dv[MODE == 1 ? NV : 1], hx[NH], hd[MODE == 1 ? NH : 1];
    const float4 zero4 = make_float4(0.f, 0.f, 0.f, 0.f);
    const int nhalo = 2 * r * W * LPP;
    auto halo_row = [&](int e) { const int hr = e / (W * LPP); return hr < r ? r0 - r + hr : r0 + RB + hr - r; };
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const int pp = (q * NTHR + tid) / LPP;
        const int row = r0 + pp / W, col = pp % W;
        xv[q] = zero4;
        if (MODE == 1) dv[q] = zero4;
        if (pp < npix && row < H) {
            const size_t o = (img + (size_t)row * W + col) * C + gl * 4;
            xv[q] = *(const float4 *)(x + o);
            if (MODE == 1) dv[q] = *(const float4 *)(dy + o);
        }
    }
#pragma unroll
    for (int q = 0; q < NH; ++q) {
        const int e = q * NTHR + tid, row = halo_row(e), col = (e / LPP) % W;
        hx[q] = zero4;
        if (MODE == 1) hd[q] = zero4;
        if (e < nhalo && row >= 0 && row < H) {
            const size_t o = (img + (size_t)row * W + col) * C + gl * 4;
            hx[q] = *(const float4 *)(x + o);
            if (MODE == 1) hd[q] = *(const float4 *)(dy + o);
        }
    }
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const int pp = (q * NTHR + tid) / LPP;
        const int row = r0 + pp / W, col = pp % W;
        put(row, col, pp < npix && row < H, xv[q], MODE == 1 ? dv[q] : zero4);
    }
#pragma unroll
    for (int q = 0; q < NH; ++q) {
        const int e = q * NTHR + tid, row = halo_row(e), col = (e / LPP) % W;
        put(row, col, e < nhalo && row >= 0 && row < H, hx[q], MODE == 1 ? hd[q] : zero4);
    }
    for (int e = NH * NTHR + tid; e < nhalo; e += NTHR) {
        const int row = halo_row(e), col = (e / LPP) % W;
        const bool in = row >= 0 && row < H;
        float4 v = zero4, d = zero4;
        if (in) {
            const size_t o = (img + (size_t)row * W + col) * C + gl * 4;
            v = *(const float4 *)(x + o);
            if (MODE == 1) d = *(const float4 *)(dy + o);
        }
        put(row, col, in, v, d);
    }
    __syncthreads();

    // phase 2: window sums, one thread per pixel of the band
    for (int pp = tid; pp < npix; pp += NTHR) {
        const int oi = pp / W, oj = pp - oi * W, row = r0 + oi;
        if (row >= H) break;
        float s1 = 0.f, s2 = 0.f;
        for (int p = 0; p < ks; ++p) {
            const float *a1 = m1 + (oi + p) * MW + oj, *a2 = m2 + (oi + p) * MW + oj;
            float u1 = 0.f, u2 = 0.f;
            for (int q = 0; q < ks; ++q) {
                u1 += taps.g[q] * a1[q];
                u2 += taps.g[q] * a2[q];
            }
            s1 += taps.g[p] * u1;
            s2 += taps.g[p] * u2;
        }
        if (MODE == 0) {
            const float z = zr[oi + r] * zc[oj] * (float)C;
            const float m = s1 / z, q2 = s2 / z;
            const float rs = 1.0f / sqrtf(fmaxf(q2 - m * m, 0.f) + eps);
            mu[img + (size_t)row * W + oj] = m;
            rstd[img + (size_t)row * W + oj] = rs;
            t1[pp] = m;
            t2[pp] = rs;
        } else {
            t1[pp] = s1;
            t2[pp] = s2;
        }
    }
    __syncthreads();

    // phase 3: elementwise pass over the registers of phase 1a
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const int pp = (q * NTHR + tid) / LPP;
        const int row = r0 + pp / W, col = pp % W;
        if (pp >= npix || row >= H) continue;
        const size_t pix = img + (size_t)row * W + col;
        const float u = t1[pp], v = t2[pp];
        const float4 xq = xv[q];
        if (MODE == 0) {
            *(float4 *)(out + pix * C + gl * 4) =
                make_float4((xq.x - u) * v, (xq.y - u) * v, (xq.z - u) * v, (xq.w - u) * v);
        } else {
            const float rs = rstd[pix];
            const float4 d = dv[q];
            float4 o = make_float4(d.x * rs + u - xq.x * v, d.y * rs + u - xq.y * v, d.z * rs + u - xq.z * v,
                                   d.w * rs + u - xq.w * v);
            // divx: the gradient divided by x itself, which is what the backward pass of a pooling layer in front
            // of this one sums up (x is that layer's output, positive)
            if (divx) o = make_float4(o.x / xq.x, o.y / xq.y, o.z / xq.z, o.w / xq.w);
            *(float4 *)(out + pix * C + gl * 4) = o;
        }
    }
}

// Fused forward pass: 3x3 stride-1 L2 pooling, then the one-stage pooled LCN of the pooled map, which is written out
// as well (the backward passes need it).  x [B,H,W,C] -> p [B,H-2,W-2,C] -> y, mu, rstd; C = 4*LPP.
// A workgroup owns PB whole rows of p of one image (plus the (ks-1)/2 rows above and below them, which the
// neighbouring bands compute a second time).  Pooling: a wave covers 64/LPP consecutive columns of x and walks down
// rpt + 2 rows; a lane squares its own pixels (every x value the workgroup needs is loaded exactly once, all loads in
// flight together), adds three rows at a time in registers and takes the two columns to its right from the lanes
// LPP and 2 LPP further on, so a wave produces 64/LPP - 2 columns of p.  WPS such waves cover a row; the 16 waves
// are 16/WPS segments of rpt rows each.  The pooled values stay in registers (at most RPT float4 per lane); their
// channel sums go into the LDS maps, and the rest is the band kernel's phases 2 and 3.
template <int LPP, int RPT>
__global__ __launch_bounds__(kBandThreads) void pool_lcn_band_kernel(const float *__restrict__ x, float *__restrict__ p,
                                                                     float *__restrict__ out, float *__restrict__ mu,
                                                                     float *__restrict__ rstd, int H, int W, int ks,
                                                                     float peps, float eps, GaussTaps taps, int PB,
                                                                     int bands, int WPS, int rpt) {
    constexpr int C = 4 * LPP, CPW = 64 / LPP, OPW = CPW - 2, NTHR = kBandThreads;
    extern __shared__ __attribute__((aligned(16))) float band_lds[];
    const int Hp = H - 2, Wp = W - 2;
    const int r = (ks - 1) / 2, MW = Wp + 2 * r, MH = PB + 2 * r;
    float *m1 = band_lds, *m2 = m1 + MH * MW, *t1 = m2 + MH * MW, *t2 = t1 + PB * Wp;
    float *zr = t2 + PB * Wp, *zc = zr + MH, *tg = zc + Wp;     // tg: the taps (indexed by loop counters below)
    // the wave index as a scalar: every row index below is then scalar too, and a row's address is a scalar base
    // plus one lane offset that all rows share
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int gl = lane % LPP, cw = lane / LPP;
    const int seg = wave / WPS, ws = wave - seg * WPS;
    const int blk = remap_xcd(blockIdx.x, gridDim.x);
    const int b = blk / bands, r0 = (blk - b * bands) * PB;
    const size_t ximg = (size_t)b * H * W, pimg = (size_t)b * Hp * Wp;

    for (int i = tid; i < MH + Wp; i += NTHR) {
        if (i < MH) zr[i] = tap_norm(taps, r0 - r + i, Hp, r);
        else zc[i - MH] = tap_norm(taps, i - MH, Wp, r);
    }
    if (tid < kLcnMaxK) tg[tid] = taps.g[tid];
    // map cells outside the pooled image are zero; every other cell is written exactly once below
    for (int cell = tid; cell < MH * MW; cell += NTHR) {
        const int hi = cell / MW, hj = cell - hi * MW;
        const int row = r0 - r + hi, col = hj - r;
        if (row < 0 || row >= Hp || col < 0 || col >= Wp) m1[cell] = m2[cell] = 0.f;
    }

    // pooling: staged row hrow of the band is row r0 - r + hrow of p and needs rows r0 - r + hrow .. + 2 of x
    const int col = ws * OPW + cw;          // column of x this lane loads = column of p it produces
    const int hrow0 = seg * rpt;
    const int xoff = min(col, W - 1) * C + gl * 4, poff = min(col, Wp - 1) * C + gl * 4;
    f32x4 q[RPT + 2];
#pragma unroll
    for (int t = 0; t < RPT + 2; ++t) {
        // every lane loads, from an address clamped into the image; what lies outside counts as zero
        const int xrow = r0 - r + hrow0 + t;
        const bool in = t < rpt + 2 && hrow0 < MH && xrow >= 0 && xrow < H && col < W;
        const float *rowp = x + (ximg + (size_t)min(max(xrow, 0), H - 1) * W) * C;
        const f32x4 v = *(const f32x4 *)(rowp + xoff);
        q[t] = in ? v : (f32x4){0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int t = 0; t < RPT + 2; ++t) q[t] *= q[t];
#pragma unroll
    for (int t = 0; t < RPT; ++t) {
        const f32x4 v = (q[t] + q[t + 1]) + q[t + 2];
        f32x4 o;
#pragma unroll
        for (int c = 0; c < 4; ++c)
            o[c] = __builtin_amdgcn_sqrtf(peps + ((v[c] + __shfl_down(v[c], LPP, 64)) + __shfl_down(v[c], 2 * LPP, 64)));
        q[t] = o;                            // p[hrow0 + t][col], valid for cw < OPW
        // one row's cross-lane reads at a time (the next row's input is tied to this row's result): with all of
        // them in flight the results alone fill the registers
        asm volatile("" : "+v"(q[t + 1][0]), "+v"(q[t + 1][1]), "+v"(q[t + 1][2]), "+v"(q[t + 1][3]) : "v"(o[0]), "v"(o[1]), "v"(o[2]), "v"(o[3]));
    }
    // channel sums of the pooled pixels -> the two maps of phase 2 (all lanes take part in the reductions)
#pragma unroll
    for (int t = 0; t < RPT; ++t) {
        const int hrow = hrow0 + t, prow = r0 - r + hrow;
        const f32x4 v = q[t];
        float a = (v[0] + v[1]) + (v[2] + v[3]);
        float c2 = (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
        a = group_sum(a, LPP);
        c2 = group_sum(c2, LPP);
        if (gl == 0 && t < rpt && hrow < MH && prow >= 0 && prow < Hp && cw < OPW && col < Wp) {
            const int cell = hrow * MW + col + r;
            m1[cell] = a;
            m2[cell] = c2;
        }
    }
    __syncthreads();

    // phase 2: window sums, one thread per pixel of the band
    for (int pp = tid; pp < PB * Wp; pp += NTHR) {
        const int oi = pp / Wp, oj = pp - oi * Wp, row = r0 + oi;
        if (row >= Hp) break;
        float s1 = 0.f, s2 = 0.f;
        for (int a = 0; a < ks; ++a) {
            const float *a1 = m1 + (oi + a) * MW + oj, *a2 = m2 + (oi + a) * MW + oj;
            float u1 = 0.f, u2 = 0.f;
            for (int c = 0; c < ks; ++c) {
                u1 += tg[c] * a1[c];
                u2 += tg[c] * a2[c];
            }
            s1 += tg[a] * u1;
            s2 += tg[a] * u2;
        }
        const float z = zr[oi + r] * zc[oj] * (float)C;
        const float m = s1 / z, q2 = s2 / z;
        const float rs = 1.0f / sqrtf(fmaxf(q2 - m * m, 0.f) + eps);
        mu[pimg + (size_t)row * Wp + oj] = m;
        rstd[pimg + (size_t)row * Wp + oj] = rs;
        t1[pp] = m;
        t2[pp] = rs;
    }
    __syncthreads();

    // phase 3: the band's own rows: p and the normalised values
#pragma unroll
    for (int t = 0; t < RPT; ++t) {
        const int prow = r0 - r + hrow0 + t;
        if (t >= rpt || prow < r0 || prow >= r0 + PB || prow >= Hp || cw >= OPW || col >= Wp) continue;
        const int pp = (prow - r0) * Wp + col;
        const float u = t1[pp], v = t2[pp];
        const size_t o = (pimg + (size_t)prow * Wp) * C;
        *(f32x4 *)(p + o + poff) = q[t];
        *(f32x4 *)(out + o + poff) = (f32x4){(q[t][0] - u) * v, (q[t][1] - u) * v, (q[t][2] - u) * v, (q[t][3] - u) * v};
    }
}

namespace {

int grid_for(long long total) {
    long long blocks = (total + 255) / 256;
    const long long cap = 256LL * 32;  // 32 workgroups per compute unit, grid-stride beyond that
    return (int)(blocks < cap ? (blocks > 0 ? blocks : 1) : cap);
}

bool make_taps(int ks, float sigma, GaussTaps *t) {
    if (ks < 1 || ks > kLcnMaxK || (ks & 1) == 0 || !(sigma > 0.f)) return false;
    const int r = (ks - 1) / 2;
    double s = 0.0, g[kLcnMaxK];
    for (int p = -r; p <= r; ++p) {
        g[p + r] = exp(-(double)(p * p) / (2.0 * (double)sigma * (double)sigma));
        s += g[p + r];
    }
    for (int p = 0; p < kLcnMaxK; ++p) t->g[p] = p < ks ? (float)(g[p] / s) : 0.f;
    return true;
}

// Lanes that share a pixel in the tile kernel, and how many of its vectors each has in flight (*nf): four where a pixel has
// them, and as few lanes as take the pixel at once (fewer lanes reduce in fewer steps); half of them, and two rounds, where over
// two fifths would be idle ([158,6,52,72]: 15.4 us with eight lanes, 14.4 with four).  The gradients' two arrays on maps of
// fewer than 48 channels whose three arrays the 256 MB Infinity Cache does not hold: a lane for every vector, whose wave reads
// whole lines from HBM ([105,251,58,20] 168 us with the former, 119 with this; [102,56,209,44] 284 and 201; [151,24,199,24], a
// quarter of the cache each, 61 and 72).
int lanes_per_pixel(int cv, bool whole_lines, int *nf) {
    *nf = whole_lines || cv == 1 ? 1 : cv == 2 ? 2 : 4;
    int l = 1;
    while (l * *nf < cv && l < 64) l <<= 1;
    return *nf == 4 && l > 1 && 5 * cv <= 3 * l * *nf ? l / 2 : l;
}

// Threads of a workgroup: more where its lanes would have over 16 vectors each, one after the other, and the chip holds few
// workgroups (two-stage gradient of [1,34,5,384], 7 x 7: 65 us with 256 threads on its few tiles, 32 with 1024).
int lcn_threads(int pixels, int cv, int arrays, long long workgroups) {
    int n = 256;
    while (n < kLcnThreads && (long long)pixels * cv * arrays > 16LL * n && workgroups * n * 2 <= 256LL * 1024) n *= 2;
    return n;
}

// Tile of the tile kernel: at most 16 x 16 pixels, the image split evenly; halved, the longer side first, until there are two
// workgroups per compute unit, as long as a tile with a halo of one radius is at most four times the tile; with the two radii
// of the two-stage form that is up to nine times, which is still the better side (the bound on two radii: 120 maps 0.97 times as
// fast, 0.56 to 1.27; [1,96,16,384], 9 x 9, gradient 31 -> 53 us).  On maps of eight such tiles
// per compute unit and more 16 columns where the last tile's missing ones are few (tiles then start on whole lines at few
// channels: [64,224,104,4] 26 us against 29 in tiles of 15).
void lcn_tile(int B, int H, int W, int r, int *th, int *tw) {
    int nh = (H + kLcnTile - 1) / kLcnTile, nw = (W + kLcnTile - 1) / kLcnTile;
    const bool many = (long long)B * nh * nw >= 8 * 256;
    for (;;) {
        *th = (H + nh - 1) / nh;
        *tw = (W + nw - 1) / nw;
        if (many && 8 * nw * kLcnTile <= 9 * W) *tw = kLcnTile;
        if ((long long)B * nh * nw >= 2 * 256) return;
        const int h2 = *th >= *tw ? (*th + 1) / 2 : *th, w2 = *th >= *tw ? *tw : (*tw + 1) / 2;
        if (h2 * w2 == *th * *tw || (h2 + 2 * r) * (w2 + 2 * r) > 4 * h2 * w2) return;
        nh = (H + h2 - 1) / h2;
        nw = (W + w2 - 1) / w2;
    }
}

}  // namespace

int launch_l2pool_fwd(const float *x, float *y, int B, int H, int W, int C, int ks, int st, float eps,
                      hipStream_t s) {
    const int Ho = (H - ks) / st + 1, Wo = (W - ks) / st + 1;
    const size_t patch_bytes = (size_t)(kPoolTH + ks - 1) * (kPoolTW + ks - 1) * C * sizeof(float);
    if (C % 4 == 0 && st == 1 && ks == 3 && Ho > 0 && Wo > 0 && B > 0) {
        // segments of RS rows, a multiple of the four rows a thread has in flight: enough segments for about
        // sixteen waves per compute unit (48 x 48 x 32 maps, batch 128: 8 rows 11.7 us, 4 rows 12.1 us, 16 rows 13.5 us)
        const int CV = C / 4;
        const long long cols = (long long)B * Wo * CV;
        const long long want = std::max<long long>((256LL * 16 * 64 + cols - 1) / cols, 1);
        const int RS = (int)std::max<long long>(((Ho + want - 1) / want + 3) / 4 * 4, 4);
        const int nseg = (Ho + RS - 1) / RS;
        const long long total = cols * nseg, nblk = (total + 255) / 256;
        if (nblk > 0x7fffffffLL) return LC_EUNSUPPORTED;
        hipLaunchKernelGGL((l2pool_fwd_stream_kernel<3, 4>), dim3((unsigned)nblk), dim3(256), 0, s, x, y, H, W, CV, Ho,
                           Wo, RS, nseg, eps, total);
    } else if (C % 4 == 0 && st == 1 && ks <= kPoolMaxK && patch_bytes <= 64 * 1024) {
        const int th = (Ho + kPoolTH - 1) / kPoolTH, tw = (Wo + kPoolTW - 1) / kPoolTW;
        const long long nblk = (long long)B * th * tw;
        if (nblk > 0x7fffffffLL) return LC_EUNSUPPORTED;
        auto kern = l2pool_tile_kernel<0>;
        if (int rc_lds = allow_dynamic_lds((const void *)kern, patch_bytes, "l2pool_fwd: hipFuncSetAttribute")) return rc_lds;
        hipLaunchKernelGGL(kern, dim3((unsigned)nblk), dim3(256), patch_bytes, s, x, (const float *)nullptr,
                           (const float *)nullptr, y, H, W, C, Ho, Wo, ks, eps, tw, th * tw);
    } else if (C % 4 == 0 && st == 1 && ks <= kPoolMaxK && B <= 65535 && (long long)H * W * C < (1LL << 30)) {
        const int groups = (Wo + kPoolOW - 1) / kPoolOW;
        hipLaunchKernelGGL(l2pool_fwd_rows_kernel, dim3((Ho * groups * (C / 4) + 255) / 256, B), dim3(256), 0, s, x, y, H,
                           W, C, Ho, Wo, ks, eps, groups);
    } else if (C % 4 == 0) {
        const long long total = (long long)B * Ho * Wo * (C / 4);
        hipLaunchKernelGGL(l2pool_fwd_kernel<4>, dim3(grid_for(total)), dim3(256), 0, s, x, y, B, H, W, C, Ho, Wo, ks,
                           st, eps, total);
    } else {
        const long long total = (long long)B * Ho * Wo * C;
        hipLaunchKernelGGL(l2pool_fwd_kernel<1>, dim3(grid_for(total)), dim3(256), 0, s, x, y, B, H, W, C, Ho, Wo, ks,
                           st, eps, total);
    }
    LC_HIP_LAUNCH_CHECK("l2pool_fwd launch");
    return LC_OK;
}

namespace {

// 3 x 3 windows at stride 1, C % 4 == 0; y null: dy holds dy/y
int launch_pool_bwd_stream(const float *x, const float *y, const float *dy, float *dx, int B, int H, int W, int C,
                           hipStream_t s) {
    const int CV = C / 4, RU = 2;
    const long long cols = (long long)B * W * CV;
    const long long want = std::max<long long>((256LL * 16 * 64 + cols - 1) / cols, 1);
    const int RS = (int)std::max<long long>(((H + want - 1) / want + RU - 1) / RU * RU, 4);
    const int nseg = (H + RS - 1) / RS;
    const long long total = cols * nseg, nblk = (total + 255) / 256;
    if (nblk > 0x7fffffffLL) return LC_EUNSUPPORTED;
    if (y)
        hipLaunchKernelGGL((l2pool_bwd_stream_kernel<3, RU, true>), dim3((unsigned)nblk), dim3(256), 0, s, x, y, dy, dx, H, W,
                           CV, H - 2, W - 2, RS, nseg, total);
    else
        hipLaunchKernelGGL((l2pool_bwd_stream_kernel<3, RU, false>), dim3((unsigned)nblk), dim3(256), 0, s, x, y, dy, dx, H, W,
                           CV, H - 2, W - 2, RS, nseg, total);
    LC_HIP_LAUNCH_CHECK("l2pool_bwd launch");
    return LC_OK;
}

}  // namespace

// Whether the gradient of 3 x 3 stride-1 pooling streams.  The tile kernel forms each quotient once and is faster only at
// around 32 channels, where several of its workgroups share a compute unit's LDS, and only with tiles that are nearly full
// and at least four of them per compute unit: 128 images of 48 x 48 x 32 24 us against 26, of 200 x 200 x 32 465 against
// 553.  Fewer tiles (16 images of 48 x 48 x 36 9.6 against 7.8, one of 96 x 96 x 40 8.2 against 5.7), tiles that hang over the
// border (128 of 33 x 40 x 24 18 against 15) or other channels stream (128 of 57 x 57 x 16: 27 against 21; of 30 x 30 x 64: 27
// against 21; 38 of 65 x 35 x 128, where a tile does not fit LDS and the row kernel ran: 60 against 33).  Over 40 maps of 24
// to 40 channels and 32 to 300 pixels a side, at 1 to 128 images, the kernel picked is on average 0.5 % slower than the
// faster one, at most 13 %.  (With dy / y handed in as one array, behind the normalisation, the line lies higher, but the two
// are within 12 % of each other where it would differ.)
bool pool_bwd_streams(int B, int H, int W, int C, int ks, int st) {
    if (C % 4 != 0 || ks != 3 || st != 1) return false;
    if (C < 24 || C > 40 || H < 32 || W < 32) return true;
    const long long tiles = (long long)((H + kPoolTH - 1) / kPoolTH) * ((W + kPoolTW - 1) / kPoolTW);
    const bool full = (long long)H * W * 100 >= tiles * (kPoolTH * kPoolTW) * 85;
    return !(full && B * tiles >= 4 * 256);
}

int launch_l2pool_bwd(const float *x, const float *y, const float *dy, float *dx, int B, int H, int W, int C, int ks,
                      int st, hipStream_t s) {
    if (pool_bwd_streams(B, H, W, C, ks, st)) return launch_pool_bwd_stream(x, y, dy, dx, B, H, W, C, s);
    const int Ho = (H - ks) / st + 1, Wo = (W - ks) / st + 1;
    const size_t patch_bytes = (size_t)(kPoolTH + ks - 1) * (kPoolTW + ks - 1) * C * sizeof(float);
    if (C % 4 == 0 && st == 1 && ks <= kPoolMaxK && patch_bytes <= 64 * 1024) {
        const int th = (H + kPoolTH - 1) / kPoolTH, tw = (W + kPoolTW - 1) / kPoolTW;
        const long long nblk = (long long)B * th * tw;
        if (nblk > 0x7fffffffLL) return LC_EUNSUPPORTED;
        auto kern = y ? l2pool_tile_kernel<1> : l2pool_tile_kernel<2>;
        if (int rc_lds = allow_dynamic_lds((const void *)kern, patch_bytes, "l2pool_bwd: hipFuncSetAttribute")) return rc_lds;
        hipLaunchKernelGGL(kern, dim3((unsigned)nblk), dim3(256), patch_bytes, s, x, y, dy, dx, H, W, C, Ho, Wo, ks,
                           0.f, tw, th * tw);
    } else if (C % 4 == 0 && st == 1 && ks <= kPoolMaxK && B <= 65535 && (long long)H * W * C < (1LL << 30)) {
        const int groups = (W + kPoolOW - 1) / kPoolOW;
        hipLaunchKernelGGL(l2pool_bwd_rows_kernel, dim3((H * groups * (C / 4) + 255) / 256, B), dim3(256), 0, s, x, y, dy,
                           dx, H, W, C, Ho, Wo, ks, groups);
    } else if (C % 4 == 0) {
        const long long total = (long long)B * H * W * (C / 4);
        hipLaunchKernelGGL(l2pool_bwd_kernel<4>, dim3(grid_for(total)), dim3(256), 0, s, x, y, dy, dx, B, H, W, C, Ho,
                           Wo, ks, st, total);
    } else {
        const long long total = (long long)B * H * W * C;
        hipLaunchKernelGGL(l2pool_bwd_kernel<1>, dim3(grid_for(total)), dim3(256), 0, s, x, y, dy, dx, B, H, W, C, Ho,
                           Wo, ks, st, total);
    }
    LC_HIP_LAUNCH_CHECK("l2pool_bwd launch");
    return LC_OK;
}

namespace {

// Rows per band: as many as the registers hold (NV float4 per thread), split evenly over the image.  The band
// kernel pays where a band is at least 8 rows and two window radii high; below that the 16x16 tiles re-read less.
template <int LPP, int MODE>
int launch_lcn_band_lpp(const float *x, const float *dy, float *out, float *mu, float *rstd, int B, int H, int W,
                        int ks, float eps, const GaussTaps &taps, hipStream_t s, int zero_pad, bool *done, int divx) {
    constexpr int NTHR = kBandThreads, NV = 8;
    const int r = (ks - 1) / 2;
    const int rb_max = (NTHR * NV) / (W * LPP);
    if (rb_max < 8 || rb_max < 2 * r) return LC_OK;
    const int bands = (H + rb_max - 1) / rb_max, RB = (H + bands - 1) / bands;
    const size_t lds = ((size_t)2 * (RB + 2 * r) * (W + 2 * r) + (size_t)2 * RB * W + (RB + 2 * r) + W) * sizeof(float);
    const long long nblk = (long long)B * bands;
    if (lds > 64 * 1024 || nblk > 0x7fffffffLL) return LC_OK;
    auto kern = lcn_band_kernel<LPP, MODE, NTHR, NV>;
    if (int rc_lds = allow_dynamic_lds((const void *)kern, lds, "lcn: hipFuncSetAttribute")) return rc_lds;
    *done = true;
    hipLaunchKernelGGL(kern, dim3((unsigned)nblk), dim3(NTHR), lds, s, x, dy, out, mu, rstd, H, W, ks, eps, taps, RB,
                       bands, zero_pad, divx);
    LC_HIP_LAUNCH_CHECK("lcn launch");
    return LC_OK;
}

int launch_lcn_band(int mode, const float *x, const float *dy, float *out, float *mu, float *rstd, int B, int H, int W,
                    int C, int ks, float eps, const GaussTaps &taps, hipStream_t s, int zero_pad, bool *done,
                    int divx = 0) {
#define LC_BAND(LPP_)                                                                                                  \
    return mode == 0 ? launch_lcn_band_lpp<LPP_, 0>(x, dy, out, mu, rstd, B, H, W, ks, eps, taps, s, zero_pad, done, 0) \
                     : launch_lcn_band_lpp<LPP_, 1>(x, dy, out, mu, rstd, B, H, W, ks, eps, taps, s, zero_pad, done, divx)
    switch (C) {
        case 4: LC_BAND(1);
        case 8: LC_BAND(2);
        case 16: LC_BAND(4);
        case 32: LC_BAND(8);
        case 64: LC_BAND(16);
        default: return LC_OK;
    }
#undef LC_BAND
}

}  // namespace

namespace {

template <int LPP, int RPT>
int launch_pool_lcn_band(const LaunchPlan &plan, const float *x, float *p, float *out, float *mu, float *rstd, int H,
                         int W, int ks, float peps, float eps, const GaussTaps &taps, int PB, int bands, int WPS,
                         int rpt, hipStream_t s) {
    auto kern = pool_lcn_band_kernel<LPP, RPT>;
    LC_LAUNCH(plan, "l2pool_lcn_fwd launch", kern, s, x, p, out, mu, rstd, H, W, ks, peps, eps, taps, PB, bands, WPS,
              rpt);
    return LC_OK;
}

}  // namespace

// Gradient of l2pool_lcn_fwd with respect to its input: lcn_bwd, then l2pool_bwd, with `scratch` ([B,Ho,Wo,C]) between
// them.  Where the streaming or the tile kernel does the second, the first leaves its gradient already divided by p there,
// so the second reads one array less.
int launch_lcn_pool_bwd(const float *x, const float *p, const float *mu, const float *rstd, const float *dn,
                        float *scratch, float *dx, int B, int H, int W, int C, int pks, int pst, int ks, float sigma,
                        hipStream_t s) {
    const int Ho = (H - pks) / pst + 1, Wo = (W - pks) / pst + 1;
    const size_t patch_bytes = (size_t)(kPoolTH + pks - 1) * (kPoolTW + pks - 1) * C * sizeof(float);
    const int th = (H + kPoolTH - 1) / kPoolTH, tw = (W + kPoolTW - 1) / kPoolTW;
    const bool quotient = pool_bwd_streams(B, H, W, C, pks, pst) || (C % 4 == 0 && pst == 1 && pks <= kPoolMaxK &&
                                                                   patch_bytes <= 64 * 1024 && (long long)B * th * tw <= 0x7fffffffLL);
    if (int rc = launch_lcn(1, p, dn, scratch, const_cast<float *>(mu), const_cast<float *>(rstd), B, Ho, Wo, C, ks, sigma,
                            0.f, s, 0, quotient))
        return rc;
    return launch_l2pool_bwd(x, quotient ? nullptr : p, scratch, dx, B, H, W, C, pks, pst, s);
}

// Host check of a pool_lcn_band_kernel launch.  tparam = {LPP, RPT}; arg = {PB, bands, WPS, rpt, H, W, ks, B}.
int check_pool_lcn_band(const LaunchPlan &p) {
    const int LPP = p.tparam[0], RPT = p.tparam[1];
    const int PB = p.arg[0], bands = p.arg[1], WPS = p.arg[2], rpt = p.arg[3], H = p.arg[4], W = p.arg[5], ks = p.arg[6];
    const int B = p.arg[7];
    const int Hp = H - 2, Wp = W - 2, r = (ks - 1) / 2, MH = PB + 2 * r, MW = Wp + 2 * r;
    LC_PLAN_REQUIRE(p, (int)p.block == kBandThreads && (LPP == 2 || LPP == 4 || LPP == 8 || LPP == 16));
    LC_PLAN_REQUIRE(p, Hp >= 1 && Wp >= 1 && PB >= 1 && bands >= 1 && (long long)PB * bands >= Hp);
    // the waves of a segment cover a row of p, the segments cover the band and its halo rows, a lane's rows fit
    const int OPW = 64 / LPP - 2;
    LC_PLAN_REQUIRE(p, WPS >= 1 && WPS <= 16 && WPS * OPW >= Wp);
    LC_PLAN_REQUIRE(p, rpt >= 1 && rpt <= RPT && (16 / WPS) * rpt >= MH);
    LC_PLAN_REQUIRE(p, p.lds_bytes >= ((size_t)2 * MH * MW + (size_t)2 * PB * Wp + MH + Wp + kLcnMaxK) * sizeof(float));
    LC_PLAN_REQUIRE(p, (long long)p.grid[0] == (long long)B * bands && p.grid[1] == 1 && p.grid[2] == 1);
    return LC_OK;
}

// Fused pooling + LCN forward for 3x3 stride-1 pooling and 8, 16, 32 or 64 channels, where a row of the pooled map
// fits the 16 waves of a workgroup; *done tells whether it was launched.
int launch_pool_lcn_fused(const float *x, float *p, float *out, float *mu, float *rstd, int B, int H, int W, int C,
                          float peps, int ks, float sigma, float eps, hipStream_t s, bool *done) {
    *done = false;
    GaussTaps taps;
    if (!make_taps(ks, sigma, &taps)) return LC_EINVAL;
    const int LPP = C / 4, Hp = H - 2, Wp = W - 2, r = (ks - 1) / 2;
    if (C % 4 != 0 || (LPP != 2 && LPP != 4 && LPP != 8 && LPP != 16) || Hp < 1 || Wp < 1) return LC_OK;
    const int OPW = 64 / LPP - 2, WPS = (Wp + OPW - 1) / OPW;
    if (WPS > 16) return LC_OK;
    const int nseg = 16 / WPS;
    // bands per image: enough for one workgroup per compute unit (twice as many measured the same or slower: 25.0
    // against 26.3 us on 128 x 46 x 46 x 32 maps, 13.1 against 10.8 us on 128 x 25 x 25 x 32), and as many more as it
    // takes for a lane's rows to fit its registers and the band's maps 64 KB of LDS
    int bands = std::min(Hp, std::max(1, (256 + B - 1) / B)), PB = 0, rpt = 0;
    size_t lds = 0;
    for (;; ++bands) {
        PB = (Hp + bands - 1) / bands;
        rpt = (PB + 2 * r + nseg - 1) / nseg;
        lds = ((size_t)2 * (PB + 2 * r) * (Wp + 2 * r) + (size_t)2 * PB * Wp + (PB + 2 * r) + Wp + kLcnMaxK) * sizeof(float);
        if ((rpt <= 13 && lds <= 64 * 1024) || bands >= Hp) break;
    }
    if (rpt > 13 || lds > 64 * 1024) return LC_OK;
    bands = (Hp + PB - 1) / PB;
    if ((long long)B * bands > 0x7fffffffLL) return LC_OK;
    const int RPT = rpt <= 4 ? 4 : rpt <= 8 ? 8 : 13;
    const LaunchPlan plan = make_plan("pool_lcn_band", {LPP, RPT}, {PB, bands, WPS, rpt, H, W, ks, B},
                                      dim3((unsigned)(B * bands)), kBandThreads, lds);
    if (int rc = check_pool_lcn_band(plan)) return rc;
    *done = true;
#define LC_PLB(LPP_, RPT_) \
    return launch_pool_lcn_band<LPP_, RPT_>(plan, x, p, out, mu, rstd, H, W, ks, peps, eps, taps, PB, bands, WPS, rpt, s)
#define LC_PLB_R(LPP_) do { if (RPT == 4) LC_PLB(LPP_, 4); if (RPT == 8) LC_PLB(LPP_, 8); LC_PLB(LPP_, 13); } while (0)
    switch (LPP) {
        case 2: LC_PLB_R(2);
        case 4: LC_PLB_R(4);
        case 8: LC_PLB_R(8);
        default: LC_PLB_R(16);
    }
#undef LC_PLB_R
#undef LC_PLB
}

// op: 0 and 1 one stage, forward and gradient; 2 and 3 two stages
int launch_lcn(int op, const float *x, const float *dy, float *out, float *mu, float *rstd, int B, int H, int W,
               int C, int ks, float sigma, float eps, hipStream_t s, int zero_pad, int divx) {
    GaussTaps taps;
    if (!make_taps(ks, sigma, &taps)) return LC_EINVAL;
    if (op < 0 || op > 3) return LC_EINVAL;
    const int tiles_h = (H + kLcnTile - 1) / kLcnTile, tiles_w = (W + kLcnTile - 1) / kLcnTile;
    const long long nblk = (long long)B * tiles_h * tiles_w;
    if (nblk > 0x7fffffffLL) return LC_EUNSUPPORTED;
    if (op < 2) {
        bool done = false;
        const int rc = launch_lcn_band(op, x, dy, out, mu, rstd, B, H, W, C, ks, eps, taps, s, zero_pad, &done, divx);
        if (done) return rc;
    }
    const int vec = C >= 4 ? 4 : 1, CV = vec == 4 ? (C + 3) / 4 : C;
    int th, tw;
    lcn_tile(B, H, W, (ks - 1) / 2, &th, &tw);
    const int tw_n = (W + tw - 1) / tw, t_img = (H + th - 1) / th * tw_n;
    if ((long long)B * t_img > 0x7fffffffLL) return LC_EUNSUPPORTED;
    const bool large = C < 48 && (long long)B * H * W * C >= 24LL << 20;
    int nf;
    const int lpp = lanes_per_pixel(CV, C % 4 == 0 && (op & 1) && large, &nf);
    dim3 grid((unsigned)nblk), tgrid((unsigned)((long long)B * t_img));
    const int R = op >= 2 ? ks - 1 : (ks - 1) / 2, hh = th + 2 * R, hw = tw + 2 * R, inner = (th + ks - 1) * (tw + ks - 1);
    const int hrows = hh * (hw - (ks - 1));
    const int nthr = lcn_threads(hh * hw, CV, (op & 1) + 1, (long long)B * t_img);
    const size_t lds = sizeof(float) * (4 * th * tw + (op < 2 ? 2 * hh * hw + 2 * hrows
                                                        : op == 2 ? hh * hw + hrows + 2 * inner : 3 * hh * hw + hrows + inner));
#define LC_LCN(...)                                                                                                   \
    hipLaunchKernelGGL((lcn_pooled_kernel<__VA_ARGS__>), tgrid, dim3(nthr), lds, s, x, dy, out, mu, rstd, H, W, C, ks, eps, \
                       taps, lpp, th, tw, tw_n, t_img, zero_pad)
#define LC_LCN_OP(OP_)                                                  \
    do {                                                                \
        if (vec == 1) LC_LCN(1, OP_, 4, false, false);                  \
        else if (C % 4 == 0 && nf == 1) LC_LCN(4, OP_, 1, false, false); \
        else if (C % 4 == 0 && nf == 2) LC_LCN(4, OP_, 2, false, false); \
        else if (C % 4 == 0) LC_LCN(4, OP_, 4, false, false);           \
        else if (nf == 2) LC_LCN(4, OP_, 2, true, false);               \
        else LC_LCN(4, OP_, 4, true, false);                            \
    } while (0)
#define LC_LCN_CACHED(LPP_)                                                                                    \
    hipLaunchKernelGGL((lcn_fwd_cached_kernel<LPP_>), grid, dim3(256), 0, s, x, out, mu, rstd, H, W, ks, eps, taps, \
                       tiles_w, tiles_h * tiles_w, zero_pad)
    if (op == 0 && C == 32) LC_LCN_CACHED(8);
    else if (op == 0 && C == 16) LC_LCN_CACHED(4);
    else if (op == 0 && C == 8) LC_LCN_CACHED(2);
    else if (op == 0) LC_LCN_OP(0);
    else if (op == 1 && divx && C % 4 != 0) return LC_EINTERNAL;   // the quotient is asked for with whole vectors only
    else if (op == 1 && divx && nf == 1) LC_LCN(4, 1, 1, false, true);
    else if (op == 1 && divx && nf == 2) LC_LCN(4, 1, 2, false, true);
    else if (op == 1 && divx) LC_LCN(4, 1, 4, false, true);
    else if (op == 1) LC_LCN_OP(1);
    else if (op == 2) LC_LCN_OP(2);
    else LC_LCN_OP(3);
#undef LC_LCN_CACHED
#undef LC_LCN_OP
#undef LC_LCN
    LC_HIP_LAUNCH_CHECK("lcn launch");
    return LC_OK;
}

}  // namespace lc
