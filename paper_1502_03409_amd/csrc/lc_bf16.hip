// bf16-operand, fp32-accumulate contractions (x, w, dy stored as bf16; y, dx, dw fp32): the choice between the bf16
// kernels, and two of one wave per task, forward and backward data.  Same mathematics and layouts as the fp32 kernels
// (Eq. 1 / Sec. 3.1 geometry).
//
// Both use v_mfma_f32_16x16x16_bf16: lane (i, kk) of an operand holds four consecutive contraction indices 4kk..4kk+3 of
// row/column i.  Where the contraction index is contiguous in memory (backward data: f) a lane's four values are one 8-byte
// load.  Where it is the strided index (forward: k of w[k][f]) a lane loads four rows of four consecutive free indices and
// transposes the 4x4 block in registers (v_perm_b32): it then owns column i of four different tiles, free index 4i+u in
// tile u, and 16 lanes still cover whole 128-byte lines.
// Waves are independent (no LDS); loads run one or two steps ahead in a register ring.  What these two keep is short
// patches (forward) and layers beyond the general kernels' limits.
#include "lc_common.hpp"

namespace lc {

typedef const __attribute__((address_space(1))) u32x2 *g2_ptr;
typedef const __attribute__((address_space(1))) unsigned short *gh_ptr;

// r[t] = four bf16 (e0..e3) of row t.  o[u] = (r[0].e_u, r[1].e_u, r[2].e_u, r[3].e_u).
__device__ __forceinline__ void transpose4x4_bf16(const u32x2 (&r)[4], u32x2 (&o)[4]) {
    constexpr unsigned LO = 0x05040100u, HI = 0x07060302u;   // low / high halves of {src0:src1}
    o[0] = (u32x2){__builtin_amdgcn_perm(r[1][0], r[0][0], LO), __builtin_amdgcn_perm(r[3][0], r[2][0], LO)};
    o[1] = (u32x2){__builtin_amdgcn_perm(r[1][0], r[0][0], HI), __builtin_amdgcn_perm(r[3][0], r[2][0], HI)};
    o[2] = (u32x2){__builtin_amdgcn_perm(r[1][1], r[0][1], LO), __builtin_amdgcn_perm(r[3][1], r[2][1], LO)};
    o[3] = (u32x2){__builtin_amdgcn_perm(r[1][1], r[0][1], HI), __builtin_amdgcn_perm(r[3][1], r[2][1], HI)};
}

// ------------------------------------------------------------------------------------ forward
// wave task = (location, 64 filters, 16*MT images).  Contraction step = 16 patch elements.
template <int MT>
__global__ __launch_bounds__(256) void lc_forward_bf16_kernel(Geom g, const unsigned short *__restrict__ x,
                                                              const unsigned short *__restrict__ w,
                                                              const float *__restrict__ bias, float alpha,
                                                              float *__restrict__ y, int fblocks, int btiles,
                                                              int ntasks) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, kk = lane >> 4;
    const int task = remap_xcd(blockIdx.x, gridDim.x) * 4 + wave;
    if (task >= ntasks) return;
    const int per_loc = fblocks * btiles;
    const int loc = task / per_loc, rest = task - loc * per_loc;
    const int f0 = (rest / btiles) * 64, b0 = (rest % btiles) * 16 * MT;
    const int i = loc / g.LW, j = loc - i * g.LW;
    const size_t img = (size_t)g.H * g.W * g.C;

    f32x4 acc[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[mt][u] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // images of this lane (rows of A); rows beyond the batch read image B-1 and are never stored
    gh_ptr xa[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int b = min(b0 + mt * 16 + n, g.B - 1);
        xa[mt] = (gh_ptr)x + (size_t)b * img + ((size_t)(i * g.S) * g.W + j * g.S) * g.C;
    }
    gh_ptr wl = (gh_ptr)w + (size_t)loc * g.K * g.F + f0 + 4 * n;
    const int WC = g.W * g.C;
    for (int kh = 0; kh < g.R; ++kh) {
        for (int q0 = 0; q0 < g.RC; q0 += 16) {          // RC % 16 == 0 on this path
            const int q = q0 + 4 * kk, k = kh * g.RC + q;
            u32x2 r[4], bo[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) r[t] = *(g2_ptr)(wl + (size_t)(k + t) * g.F);
            u32x2 a[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) a[mt] = *(g2_ptr)(xa[mt] + kh * WC + q);
            transpose4x4_bf16(r, bo);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int u = 0; u < 4; ++u) acc[mt][u] = mfma16_bf16(a[mt], bo[u], acc[mt][u]);
        }
    }
    f32x4 bv = (f32x4){0.f, 0.f, 0.f, 0.f};
    if (bias) bv = *(const f32x4 *)(bias + (size_t)loc * g.F + f0 + 4 * n);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int b = b0 + mt * 16 + 4 * kk + rr;
            if (b >= g.B) continue;
            f32x4 o;
#pragma unroll
            for (int u = 0; u < 4; ++u) o[u] = alpha * acc[mt][u][rr] + bv[u];
            *(f32x4 *)(y + ((size_t)b * g.L + loc) * g.F + f0 + 4 * n) = o;
        }
}

// ------------------------------------------------------------------------------ backward data
// wave task = (cell, 64 cell values, 16*MT images); contraction over (a, a', f), 16 f per step.
template <int MT>
__global__ __launch_bounds__(256) void lc_bwd_data_bf16_kernel(Geom g, const unsigned short *__restrict__ dy,
                                                               const unsigned short *__restrict__ w,
                                                               float *__restrict__ dx, int CW, int nblocks,
                                                               int btiles, int ntasks) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, kk = lane >> 4;
    const int task = remap_xcd(blockIdx.x, gridDim.x) * 4 + wave;
    if (task >= ntasks) return;
    const int per_cell = nblocks * btiles;
    const int cell = task / per_cell, rest = task - cell * per_cell;
    const int n0 = (rest / btiles) * 64, b0 = (rest % btiles) * 16 * MT;
    const int ri = cell / CW, wi = cell - ri * CW;
    const int SC = g.S * g.C, NCV = g.S * SC, AP = g.R / g.S;

    int kn[4];          // offset of this lane's cell value inside a field's K x F matrix, per N-tile
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const int nn = n0 + nt * 16 + m;
        const int nc = nn < NCV ? nn : 0;
        const int dr = nc / SC;
        kn[nt] = (dr * g.RC + (nc - dr * SC)) * g.F + 4 * kk;
    }
    f32x4 acc[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};

    const size_t dyimg = (size_t)g.L * g.F;
    gh_ptr da[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) da[mt] = (gh_ptr)dy + (size_t)min(b0 + mt * 16 + m, g.B - 1) * dyimg + 4 * kk;

    for (int a = 0; a < AP; ++a) {
        const int i = ri - a;
        if (i < 0 || i >= g.LH) continue;
        for (int ap = 0; ap < AP; ++ap) {
            const int j = wi - ap;
            if (j < 0 || j >= g.LW) continue;
            const size_t loc = (size_t)i * g.LW + j;
            gh_ptr wl = (gh_ptr)w + (loc * g.K + (size_t)g.S * a * g.RC + g.S * ap * g.C) * g.F;
            for (int f = 0; f < g.F; f += 16) {          // F % 16 == 0 on this path
                u32x2 bo[4], av[MT];
#pragma unroll
                for (int nt = 0; nt < 4; ++nt) bo[nt] = *(g2_ptr)(wl + kn[nt] + f);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) av[mt] = *(g2_ptr)(da[mt] + loc * g.F + f);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < 4; ++nt) acc[mt][nt] = mfma16_bf16(av[mt], bo[nt], acc[mt][nt]);
            }
        }
    }
#pragma unroll
    for (int nt = 0; nt < 4; ++nt) {
        const int nn = n0 + nt * 16 + m;
        if (nn >= NCV) continue;
        const int dr = nn / SC, rem = nn - dr * SC;
        const int row = ri * g.S + dr, col = wi * g.S + rem / g.C;
        if (row >= g.H || col >= g.W) continue;
        const size_t pix = ((size_t)row * g.W + wi * g.S) * g.C + rem;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int b = b0 + mt * 16 + 4 * kk + r;
                if (b < g.B) dx[(size_t)b * g.H * g.W * g.C + pix] = acc[mt][nt][r];
            }
    }
}

// Shapes this file handles: patch rows, strides and filter counts that keep every 8-byte access aligned.
bool bf16_shape_supported(const Geom &g) {
    return g.RC % 16 == 0 && (g.S * g.C) % 4 == 0 && (g.W * g.C) % 4 == 0 && g.F % 64 == 0 && g.B % 16 == 0 &&
           g.R % g.S == 0;
}

// Host checks of the one-wave-per-task kernels of this file.  tparam = {MT}; arg as listed per function.
namespace {

// arg = {filter blocks of 64, batch tiles, wave tasks}
int check_forward_bf16_simple(const Geom &g, const LaunchPlan &p) {
    const int MT = p.tparam[0], fblocks = p.arg[0], btiles = p.arg[1], ntasks = p.arg[2];
    LC_PLAN_REQUIRE(p, p.block == 256 && bf16_shape_supported(g));
    LC_PLAN_REQUIRE(p, fblocks == g.F / 64 && btiles == ceil_div(g.B, 16 * MT));
    LC_PLAN_REQUIRE(p, (long long)ntasks == (long long)g.L * fblocks * btiles);
    LC_PLAN_REQUIRE(p, (long long)p.grid[0] * 4 >= ntasks && (long long)(p.grid[0] - 1) * 4 < ntasks);
    return LC_OK;
}

// arg = {cells per row, blocks of 64 cell values, batch tiles, wave tasks}
int check_backward_data_bf16_simple(const Geom &g, const LaunchPlan &p) {
    const int MT = p.tparam[0], CW = p.arg[0], nblocks = p.arg[1], btiles = p.arg[2], ntasks = p.arg[3];
    LC_PLAN_REQUIRE(p, p.block == 256 && bf16_shape_supported(g));
    LC_PLAN_REQUIRE(p, CW == ceil_div(g.W, g.S) && nblocks == ceil_div(g.S * g.S * g.C, 64) && btiles == ceil_div(g.B, 16 * MT));
    LC_PLAN_REQUIRE(p, (long long)ntasks == (long long)ceil_div(g.H, g.S) * CW * nblocks * btiles);
    LC_PLAN_REQUIRE(p, (long long)p.grid[0] * 4 >= ntasks && (long long)(p.grid[0] - 1) * 4 < ntasks);
    LC_PLAN_REQUIRE(p, (long long)g.K * g.F < (1LL << 31));
    return LC_OK;
}

template <int MT>
int launch_forward_simple(const Geom &g, const void *x, const void *w, const float *bias, float alpha, float *y,
                          hipStream_t s) {
    const int fblocks = g.F / 64, btiles = (g.B + 16 * MT - 1) / (16 * MT);
    const long long ntasks = (long long)g.L * fblocks * btiles;
    if (ntasks > (1LL << 30)) return LC_EUNSUPPORTED;
    const LaunchPlan plan = make_plan("lc_forward_bf16_simple", {MT}, {fblocks, btiles, (int)ntasks},
                                      dim3((unsigned)((ntasks + 3) / 4)), 256, 0);
    if (int rc = check_forward_bf16_simple(g, plan)) return rc;
    LC_LAUNCH(plan, "lc_forward (bf16) launch", lc_forward_bf16_kernel<MT>, s, g, (const unsigned short *)x,
              (const unsigned short *)w, bias, alpha, y, fblocks, btiles, (int)ntasks);
    return LC_OK;
}

template <int MT>
int launch_backward_data_simple(const Geom &g, const void *dy, const void *w, float *dx, hipStream_t s) {
    const int CH = (g.H + g.S - 1) / g.S, CW = (g.W + g.S - 1) / g.S;
    const int nblocks = (g.S * g.S * g.C + 63) / 64, btiles = (g.B + 16 * MT - 1) / (16 * MT);
    const long long ntasks = (long long)CH * CW * nblocks * btiles;
    if (ntasks > (1LL << 30)) return LC_EUNSUPPORTED;
    const LaunchPlan plan = make_plan("lc_bwd_data_bf16_simple", {MT}, {CW, nblocks, btiles, (int)ntasks},
                                      dim3((unsigned)((ntasks + 3) / 4)), 256, 0);
    if (int rc = check_backward_data_bf16_simple(g, plan)) return rc;
    LC_LAUNCH(plan, "lc_backward_data (bf16) launch", lc_bwd_data_bf16_kernel<MT>, s, g, (const unsigned short *)dy,
              (const unsigned short *)w, dx, CW, nblocks, btiles, (int)ntasks);
    return LC_OK;
}

}  // namespace

// Order of preference, every pass: the workgroup-tiled kernels (wide layers), the strip-sharing / pipelined / transposing
// kernels of the narrow layers (faster than the one-wave-per-task kernels of this file wherever both apply: a 32 x 32 x 4
// layer forward 30 against 37 us, backward data 13 against 21), the kernels of this file, the fp32 pipelined kernels on
// bf16 storage, for nearly every other shape the general kernels, and for the rest the masked fp32 kernels on bf16 storage.
//
// Where the general kernels come first (both sides measured on some 130 layers):
//  - forward: instead of the strip kernel where that would have fewer workgroups than the chip compute units, counted with its
//    widest blocks of filters (24 to 255 of them: faster or the same on 88 of 100 layers, 1.43 times on average and up to 8.5: 64
//    images of 82 x 85 x 8, 13 x 13 at stride 7, 16 filters 181 -> 21 us; the other twelve, most at stride 1, are up to 1.6 times
//    slower: 69 images of 21 x 70 x 8, 14 x 14, 64 filters 53 against 85; a line by stride and patch would keep those), and
//    instead of the one-wave-per-task kernel but for patches of at most 128 elements (128
//    images of 36 x 54 x 32, 16 x 16 at stride 2, 64 filters 470 -> 151 us; 16 of 84 x 76 x 8, 4 x 4 at stride 2: 7.2
//    against 8.8 us);
//  - backward data: instead of the one-wave-per-task kernel (10 layers of 11 faster, by 1.2 to 3.4 times: 32 images of
//    128 x 128 x 8, 8 x 8 at stride 4, 128 filters 75 -> 35 us);
//  - weight gradient: instead of the strip kernel for patches of at most 512 elements (18 of 18, 100 of 102 x 102 x 4, 8 x 8
//    at stride 2, 16 filters 42 -> 21 us; longer ones are up to 1.5 times slower);
//  - instead of the workgroup-tiled kernels of the wide layers where these have at most kFewTiles tiles, a quarter of the
//    compute units, or for the weight gradient kFewGradTiles, whose workgroups also split the patch (128 images of 32 x 32 x 16,
//    one field, 1024 filters: forward 246 -> 65 us, weight gradient 59 -> 26; 14 x 14 x 32, 8 x 8 at stride 2, 256 filters:
//    forward 34 -> 18, backward data 79 -> 34; at 64 tiles 36 -> 27, at 102 the same, from 128 on the tiled kernels are up to
//    2.5 times faster; backward data at 49 workgroups 40 -> 24, at 121 to 128 between 0.88 and 1.16 times; weight gradient at
//    16 tiles 11.3 -> 10.6, at 32 14 against 17).
constexpr int kFewTiles = 64, kFewGradTiles = 16;

static long long tiles128(long long places, const Geom &g, int per_place) { return places * per_place * ceil_div(g.B, 128); }

int launch_forward_bf16(const Geom &g, const void *x, const void *w, const float *bias, float alpha, float *y,
                        hipStream_t s) {
    const bool general = forward_general_supported(g, 2);
    if (bf16_shape_supported(g) && bf16_tiled_forward_supported(g)) {
        if (general && tiles128(g.L, g, g.F / 128) <= kFewTiles) return launch_forward_general_bf16(g, x, w, bias, alpha, y, s);
        return launch_forward_bf16_tiled(g, x, w, bias, alpha, y, s);
    }
    if (bf16_strip_forward_supported(g)) {
        if (general && bf16_strip_forward_workgroups(g) < 256) return launch_forward_general_bf16(g, x, w, bias, alpha, y, s);
        return launch_forward_bf16_strip(g, x, w, bias, alpha, y, s);
    }
    if (!bf16_shape_supported(g)) return launch_forward_bf16_storage(g, x, w, bias, alpha, y, s);
    if (general && g.K > 128) return launch_forward_general_bf16(g, x, w, bias, alpha, y, s);
    if (g.B >= 64) return launch_forward_simple<4>(g, x, w, bias, alpha, y, s);
    return launch_forward_simple<1>(g, x, w, bias, alpha, y, s);
}

int launch_backward_data_bf16(const Geom &g, const void *dy, const void *w, float *dx, hipStream_t s) {
    if (bf16_shape_supported(g) && bf16_tiled_backward_data_supported(g)) {
        const long long cells = (long long)ceil_div(g.H, g.S) * ceil_div(g.W, g.S);
        if (tiles128(cells, g, g.S * g.S * g.C / 128) <= kFewTiles && backward_data_general_supported(g, 2))
            return launch_backward_data_general_bf16(g, dy, w, dx, s);
        return launch_backward_data_bf16_tiled(g, dy, w, dx, s);
    }
    if (!bf16_shape_supported(g) || backward_data_bf16_pipelined_supported(g))
        return launch_backward_data_bf16_storage(g, dy, w, dx, s);   // pipelined (bf16 MFMAs), general or masked kernel
    if (backward_data_general_supported(g, 2)) return launch_backward_data_general_bf16(g, dy, w, dx, s);
    if (g.B >= 128) return launch_backward_data_simple<8>(g, dy, w, dx, s);
    if (g.B >= 64) return launch_backward_data_simple<4>(g, dy, w, dx, s);
    return launch_backward_data_simple<1>(g, dy, w, dx, s);
}

int launch_backward_weights_bf16(const Geom &g, const void *x, const void *dy, float beta, float *dw,
                                 hipStream_t s) {
    if (bf16_shape_supported(g) && bf16_tiled_backward_weights_supported(g)) {
        if ((long long)g.L * (g.F / 128) <= kFewGradTiles && backward_weights_general_supported(g, 2))
            return launch_backward_weights_general_bf16(g, x, dy, beta, dw, s);
        return launch_backward_weights_bf16_tiled(g, x, dy, beta, dw, s);
    }
    if (g.K <= 512 && bf16_strip_backward_weights_supported(g) && backward_weights_general_supported(g, 2))
        return launch_backward_weights_general_bf16(g, x, dy, beta, dw, s);
    if (bf16_rows_backward_weights_supported(g)) return launch_backward_weights_bf16_rows(g, x, dy, beta, dw, s);
    return launch_backward_weights_bf16_storage(g, x, dy, beta, dw, s);
}

}  // namespace lc
