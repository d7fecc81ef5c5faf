// lc_backward_data for layers whose S x S x C cells hold a multiple of 128 values (Eq. 1's decoder term):
// the workgroup tiling of the wide forward kernel with the operands' roles changed.
//
// A workgroup owns one cell of the input (128 of its values) and a batch tile of 32*MT images; each of its four waves has 32
// of the values and all of the images.  The contraction runs over the fields that cover the cell and over their filters, in
// chunks of 32 filters of one field.  Fields outside the grid are not in the chunk list; a cell no field covers gets zeros.
//
// fp32 products are split into bf16 parts (mfma_split): 96 MFMA cycles per 16 x 16 tile and chunk against 264 of fp32 MFMAs,
// which moreover keep the vector unit idle.  dy is taken apart once per workgroup, on its way into LDS (two buffers, one barrier
// per chunk).  The filters of a cell value are 128 contiguous bytes of a chunk: eight lanes load them, so that neighbouring lanes
// meet in a cache line (16 lanes with 16 rows take the cache four times as long), and the wave turns them in its own LDS.
#include "lc_general.hpp"

namespace lc {

namespace {

constexpr int kChunk = 32;          // filters per LDS chunk

// DENSE: a layer of one field that covers its whole input (R = H = W, the dense last layer of Sec. 3.1).  Every
// input value then has the same single covering field, so a "cell" is any block of 128 consecutive values k and
// dx[b][k] = sum_f w[k][f] dy[b][f].
template <int MT, int PD, bool DENSE>
__global__ __launch_bounds__(256, 2) void lc_bwd_data_wide_kernel(Geom g, const float *__restrict__ dy,
                                                                  const float *__restrict__ w,
                                                                  float *__restrict__ dx, int CW, int nblk,
                                                                  int btiles) {
    static_assert(PD == 2, "two chunks of lookahead");
    // floats of a buffer: NT tiles of 16 images in three parts of 1 KB.  Filters 8 kk .. 8 kk + 7 of row m lie at slot
    // 4 m + (kk ^ m/4) of 16 bytes: sixteen neighbouring lanes of a store (four or eight a row) or a read (lane (m, kk)) touch every
    // bank once (13 % of the cycles see a conflict all the same).
    constexpr int BT = 32 * MT, NT = 2 * MT, BUF = NT * 3 * 256;
    extern __shared__ __attribute__((aligned(16))) float xs[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kk = lane >> 4;
    int t_id = remap_xcd(blockIdx.x, gridDim.x);
    const int bt = t_id % btiles;
    t_id /= btiles;
    const int nb = DENSE ? 0 : t_id % nblk, cell = DENSE ? t_id : t_id / nblk;
    const int ri = DENSE ? 0 : cell / CW, wi = DENSE ? 0 : cell - ri * CW;
    const int b0 = bt * BT;
    const int SC = g.S * g.C, AP = g.R / g.S;
    // fields (ri - a, wi - ap) inside the grid
    const int a_lo = max(0, ri - (g.LH - 1)), a_hi = min(AP - 1, ri);
    const int p_lo = max(0, wi - (g.LW - 1)), p_hi = min(AP - 1, wi);
    const int cpf = g.F / kChunk;
    const int nchunks = (a_hi >= a_lo && p_hi >= p_lo) ? (a_hi - a_lo + 1) * (p_hi - p_lo + 1) * cpf : 0;

    f32x4 acc[NT][2];
    auto clear = [&] {
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t][0] = acc[t][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
    };

    // a cursor walks the chunk list in order and stays on the last chunk once it gets there
    struct Cursor { int a, ap, hf; };
    auto advance = [&](Cursor &q) {
        if (q.a == a_hi && q.ap == p_hi && q.hf == cpf - 1) return;
        if (++q.hf == cpf) {
            q.hf = 0;
            if (++q.ap > p_hi) { q.ap = p_lo; ++q.a; }
        }
    };

    const int seg = tid & 7, brow = tid >> 3;
    const int LF = g.L * g.F;
    // 32 images' first one is the wave's, the rest of a place 32 bits of bytes: a whole address a lane would cost eight registers
    // more than there are
    gbytes dyp[MT];
    unsigned doff[MT];
#pragma unroll
    for (int s = 0; s < MT; ++s) {
        const int first = min(b0 + 32 * s, g.B - 1);
        dyp[s] = (gbytes)(dy + (size_t)first * LF);
        doff[s] = ((unsigned)min(brow, g.B - 1 - first) * (unsigned)LF + seg * 4) * 4u;
    }
    // this thread's slot in a tile of 16 images (tile brow / 16 + 2 s), in floats, and the half of it
    const int sslot = (brow >> 4) * (3 * 256) + 4 * (4 * (brow & 15) + ((seg >> 1) ^ ((brow >> 2) & 3))), shalf = seg & 1;
    const int aslot = 4 * (4 * n + (kk ^ (n >> 2)));
    // the wave's own 4 KB behind the buffers: two tiles of 16 weight rows, two halves of a slot each
    float *wx = xs + 2 * BUF + wave * 1024;
    // lane 4 r + q loads filters 8 k .. 8 k + 7, k = q ^ r/4, of row r of either tile, relative to the cell's corner in a field:
    // that is the slot 4 r + q, its own number
    const int value0 = (DENSE ? cell * 128 : nb * 128) + wave * 32;
    unsigned kn[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int r = lane >> 2, nn = value0 + u * 16 + r, dr = nn / SC;
        const int row = DENSE ? min(nn, g.K - 1) : dr * g.RC + (nn - dr * SC);      // (dense: rows beyond K are not stored)
        kn[u] = ((unsigned)row * (unsigned)g.F + 8 * ((lane & 3) ^ (r >> 2))) * 4u;
    }

    bool nans = false;                  // (the same in all threads)
    unsigned low = 0;
    auto pass = [&](auto split_tag) {
        constexpr bool SPLIT = decltype(split_tag)::value;
        Cursor sq = {a_lo, p_lo, 0};
        auto stage_load = [&](f32x4 (&st)[MT]) {
            const int o = ((ri - sq.a) * g.LW + (wi - sq.ap)) * g.F + sq.hf * kChunk;
#pragma unroll
            for (int s = 0; s < MT; ++s) st[s] = load_quad<float>(opaque(dyp[s] + (size_t)o * 4), doff[s]);
            advance(sq);
        };
        auto stage_store = [&](int p, const f32x4 (&st)[MT]) {
            float *buf = xs + p * BUF + sslot;
#pragma unroll
            for (int s = 0; s < MT; ++s) {
                if constexpr (SPLIT) {
                    float e[4] = {st[s][0], st[s][1], st[s][2], st[s][3]};
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        const u32x2 v = {cvt_pk_bf16(e[0], e[1]), cvt_pk_bf16(e[2], e[3])};
                        if (q == 2) {
                            gather_low(low, e[0], e[1]);
                            gather_low(low, e[2], e[3]);
                        }
                        *(u32x2 *)(buf + (s * 2 * 3 + q) * 256 + 2 * shalf) = v;
#pragma unroll
                        for (int r = 0; r < 4; ++r) e[r] -= r & 1 ? bf16_hi(v[r >> 1]) : bf16_lo(v[r >> 1]);
                    }
                } else {
                    *(f32x4 *)(buf + (s * 2 * 3 + shalf) * 256) = st[s];
                }
            }
        };
        Cursor wq = {a_lo, p_lo, 0};
        auto wload = [&](f32x4 (&r)[2][2]) {
            const size_t loc = (size_t)((ri - wq.a) * g.LW + (wi - wq.ap));
            const gbytes p = opaque((gbytes)(w + (loc * g.K + (size_t)g.S * wq.a * g.RC + g.S * wq.ap * g.C) * g.F + wq.hf * kChunk));
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int h = 0; h < 2; ++h) r[u][h] = load_quad<float>(p, kn[u] + 16 * h);
            advance(wq);
        };
        f32x4 st[PD][MT], wr[PD][2][2];
#pragma unroll
        for (int p = 0; p < PD; ++p) wload(wr[p]);
        stage_load(st[0]);
        stage_store(0, st[0]);
#pragma unroll
        for (int p = 0; p < PD; ++p) stage_load(st[p]);          // set p: chunk p+1
        __syncthreads();
        for (int c0 = 0; c0 < nchunks; c0 += 2) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int c = c0 + p;               // chunk c lies in buffer p, and the set p holds the next one's images
                if (c < nchunks) {
                    const float *ab = xs + p * BUF + aslot;
                    // (a wave's LDS operations keep their order; nobody else has this part)
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int h = 0; h < 2; ++h) *(f32x4 *)(wx + (2 * u + h) * 256 + 4 * lane) = wr[p][u][h];
                    wload(wr[p]);
                    __builtin_amdgcn_wave_barrier();
                    float e[2][8];
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            const f32x4 v = *(const f32x4 *)(wx + (2 * u + h) * 256 + aslot);
#pragma unroll
                            for (int q = 0; q < 4; ++q) e[u][4 * h + q] = v[q];
                        }
                    __builtin_amdgcn_wave_barrier();
                    if constexpr (SPLIT) {
                        const Parts pb[2] = {split8(e[0], low), split8(e[1], low)};
#pragma unroll
                        for (int t = 0; t < NT; t += 2) {
                            Parts pa[2];
#pragma unroll
                            for (int m = 0; m < 2; ++m)
#pragma unroll
                                for (int q = 0; q < 3; ++q) pa[m].p[q] = *(const u32x4 *)(ab + ((t + m) * 3 + q) * 256);
                            mfma_split_rows(pa, pb, acc + t);
                            // (or the compiler reads all tiles ahead, and spills what the next chunk's loads need: 690 -> 747 us)
                            if (t + 2 == NT / 2) __builtin_amdgcn_sched_barrier(0);
                        }
                    } else {
#pragma unroll
                        for (int t = 0; t < NT; ++t)
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                const f32x4 a = *(const f32x4 *)(ab + (t * 3 + h) * 256);
#pragma unroll
                                for (int q = 0; q < 4; ++q)
#pragma unroll
                                    for (int u = 0; u < 2; ++u) acc[t][u] = mfma16(a[q], e[u][4 * h + q], acc[t][u]);
                            }
                    }
                    if (c + 1 < nchunks) stage_store(p ^ 1, st[p]);
                    if (c + 1 + PD < nchunks) stage_load(st[p]);
                }
                // Operands of a diverged layer show in the first two chunks: the fp32 pass starts there and then, unless
                // every value has a NaN among its first weights, so that no sum is anything else.
                if (SPLIT && p == 1 && c0 == 0) {
                    if (__syncthreads_or(!all_finite<2 * NT>(&acc[0][0]) || inexact(low))) {
                        f32x4 first[2][2];
                        wq = {a_lo, p_lo, 0};
                        wload(first);
                        bool every = true;
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            bool a = false;
#pragma unroll
                            for (int h = 0; h < 2; ++h)
#pragma unroll
                                for (int q = 0; q < 4; ++q) a |= first[u][h][q] != first[u][h][q];
                            unsigned long long m = __ballot(a);         // lanes 4 r .. 4 r + 3: row r
                            m |= m >> 1;
                            m |= m >> 2;
                            every = every && (m & 0x1111111111111111ull) == 0x1111111111111111ull;
                        }
                        nans = !__syncthreads_or(!every);
                        if (!nans) return;
                        // where the loads ahead were: chunk min(2 + PD, last)
                        wq = {a_lo, p_lo, 0};
                        for (int k = 0; k < 2 + PD; ++k) advance(wq);
                    }
                } else {
                    __syncthreads();
                }
            }
        }
    };
    clear();
    if (nchunks > 0) {
        pass(std::true_type{});
        // an operand that is not finite or too small, or a part that overflowed: once more in fp32
        if (!nans && __syncthreads_or(!all_finite<2 * NT>(&acc[0][0]) || inexact(low))) {
            clear();
            pass(std::false_type{});
        }
    }

#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int nn = value0 + u * 16 + n;
        size_t pix = (size_t)nn;                     // dense, R = H = W: the patch index is the pixel index
        if (DENSE) {
            if (nn >= g.K) continue;
        } else {
            const int dr = nn / SC, rem = nn - dr * SC;
            const int row = ri * g.S + dr, col = wi * g.S + rem / g.C;
            pix = ((size_t)row * g.W + wi * g.S) * g.C + rem;
            if (row >= g.H || col >= g.W) continue;
        }
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int b = b0 + 16 * t + 4 * kk + r;
                if (b < g.B) dx[(size_t)b * g.H * g.W * g.C + pix] = acc[t][u][r];
            }
    }
}

// Host check of a lc_bwd_data_wide_kernel launch.  tparam = {MT, PD, DENSE}; arg = {cells per row, 128-value blocks
// per cell, batch tiles}.
int check_backward_data_wide(const Geom &g, const LaunchPlan &p) {
    const int MT = p.tparam[0], DENSE = p.tparam[2];
    const int CW = p.arg[0], nblk = p.arg[1], btiles = p.arg[2];
    const int BT = 32 * MT;
    LC_PLAN_REQUIRE(p, p.block == 256);
    LC_PLAN_REQUIRE(p, g.F % kChunk == 0 && btiles == ceil_div(g.B, BT));
    // 32-bit byte offsets into 32 images' dy and inside a field's K x F matrix
    LC_PLAN_REQUIRE(p, (long long)32 * g.L * g.F * 4 < (1LL << 32) && (long long)g.K * g.F * 4 <= (1LL << 32));
    long long cells;
    if (DENSE) {
        LC_PLAN_REQUIRE(p, g.L == 1 && g.R == g.H && g.R == g.W && nblk == 1);
        cells = ceil_div(g.K, 128);
    } else {
        LC_PLAN_REQUIRE(p, g.R % g.S == 0 && (g.S * g.S * g.C) % 128 == 0 && nblk == g.S * g.S * g.C / 128);
        LC_PLAN_REQUIRE(p, CW == ceil_div(g.W, g.S));
        cells = (long long)ceil_div(g.H, g.S) * CW;
    }
    LC_PLAN_REQUIRE(p, (long long)p.grid[0] == cells * nblk * btiles && p.grid[1] == 1 && p.grid[2] == 1);
    LC_PLAN_REQUIRE(p, p.lds_bytes >= (size_t)2 * BT * 32 * 6 + 4 * 4096);
    return LC_OK;
}

template <int MT, int PD, bool DENSE>
int launch_wide(const Geom &g, const float *dy, const float *w, float *dx, hipStream_t s) {
    constexpr int BT = 32 * MT;
    const size_t lds = (size_t)2 * BT * 32 * 6 + 4 * 4096;
    auto kern = lc_bwd_data_wide_kernel<MT, PD, DENSE>;
    const int CH = (g.H + g.S - 1) / g.S, CW = (g.W + g.S - 1) / g.S;
    const int nblk = DENSE ? 1 : g.S * g.S * g.C / 128, btiles = (g.B + BT - 1) / BT;
    const long long cells = DENSE ? (g.K + 127) / 128 : (long long)CH * CW;
    const LaunchPlan plan = make_plan("lc_bwd_data_wide", {MT, PD, DENSE ? 1 : 0}, {CW, nblk, btiles},
                                      dim3((unsigned)(cells * nblk * btiles)), 256, lds);
    if (int rc = check_backward_data_wide(g, plan)) return rc;
    LC_LAUNCH(plan, "lc_backward_data (wide) launch", kern, s, g, dy, w, dx, CW, nblk, btiles);
    return LC_OK;
}

}  // namespace

bool backward_data_wide_supported(const Geom &g) {
    const long long cells = (long long)((g.H + g.S - 1) / g.S) * ((g.W + g.S - 1) / g.S);
    return g.R % g.S == 0 && g.F % kChunk == 0 && (g.S * g.S * g.C) % 128 == 0 && g.B > 64 &&
           (long long)g.B * g.L * g.F < (1ll << 31) && (long long)g.K * g.F < (1ll << 31) &&
           cells * (g.S * g.S * g.C / 128) * ((g.B + 127) / 128) < (1ll << 31);
}

// one field covering the whole input: any K, filters in chunks of 32
bool backward_data_dense_supported(const Geom &g) {
    return g.L == 1 && g.R == g.H && g.R == g.W && g.F % kChunk == 0 && g.B > 64 &&
           (long long)g.B * g.F < (1ll << 31) && (long long)g.K * g.F < (1ll << 31);
}

int launch_backward_data_wide_f32(const Geom &g, const float *dy, const float *w, float *dx, hipStream_t s) {
    // batch tile of 128, 96 or 64 images: the one that pads the batch least, the larger one on a tie (B = 192: two
    // tiles of 128 waste a quarter of the MFMAs)
    int mt = batch_tile_mt(g.B, true);
    const bool dense = backward_data_dense_supported(g);
    if (!dense && !backward_data_wide_supported(g)) return LC_EUNSUPPORTED;
    // a layer that gives fewer workgroups than the chip has compute units takes 64-image tiles where they pad the
    // batch no more: twice the workgroups, each half as long (a 23 x 23 x 32 input under 6 x 6 fields at stride 2,
    // 144 cells, batch 128: 27.6 -> 26.4 us; 32-image tiles: 29.0 us, the chunk pipeline's latency is what is left)
    {
        const long long cells = dense ? (g.K + 127) / 128
                                      : (long long)((g.H + g.S - 1) / g.S) * ((g.W + g.S - 1) / g.S) * (g.S * g.S * g.C / 128);
        const int bt = 32 * mt;
        if (mt > 2 && cells * ((g.B + bt - 1) / bt) < 256 && (g.B + 63) / 64 * 64 <= (g.B + bt - 1) / bt * bt) mt = 2;
    }
    if (mt == 2) return dense ? launch_wide<2, 2, true>(g, dy, w, dx, s) : launch_wide<2, 2, false>(g, dy, w, dx, s);
    if (mt == 3) return dense ? launch_wide<3, 2, true>(g, dy, w, dx, s) : launch_wide<3, 2, false>(g, dy, w, dx, s);
    return dense ? launch_wide<4, 2, true>(g, dy, w, dx, s) : launch_wide<4, 2, false>(g, dy, w, dx, s);
}

}  // namespace lc
