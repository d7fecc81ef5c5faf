// lc_forward for layers of few fields and long patches (F a multiple of 128, patch rows that split into chunks of 32 or
// 16 values): Eq. 1's encoder term with a workgroup tile of one field x 128 filters x 32*MT images.
//
// Each of the four waves has 32 of the filters and all of the images.  fp32 products are split into bf16 parts (mfma_split), in
// steps of 32 contraction indices: 96 MFMA cycles per 16 x 16 tile against 264 of fp32 MFMAs, which moreover keep the vector
// unit idle.  What is left to bound the kernel is taking values apart, 22 vector instructions for four, and a barrier a step: the
// matrix unit and the vector ALU are busy 51 % of the time each (256 images of 64 x 64 x 32, 8 x 8 at stride 2, 128 filters).  An
// image's values are taken apart once per workgroup, on their way into LDS, and a filter's once, by the only wave that has it.
#include <algorithm>

#include "lc_general.hpp"

namespace lc {

namespace {

typedef FVec<2>::T f32x2;
typedef const __attribute__((address_space(1))) f32x2 *g2_ptr;

// KCH = contraction indices per chunk (32, or 16 for patch rows that are only a multiple of 16): KCH*4 contiguous bytes
// per image.  A step is one chunk of 32 or two of 16; the second of the last step may be missing (zeros then).
//
// LDS: 1 KB per part of 16 images and 32 indices, two buffers, one barrier per step.  Indices 8 kk .. 8 kk + 7 of image m lie
// at slot 4 m + (kk ^ m/4) of 16 bytes, so that sixteen neighbouring lanes of a store (eight a row) or a read (lane (m, kk)) touch
// every bank once.  13 % of the cycles see a conflict all the same (SQ_LDS_BANK_CONFLICT).
//
// A layer with few fields (the dense last layer of Sec. 3.1 is a single one) gives too few workgroups; its
// contraction is then cut into `nslices` ranges of steps, each range a workgroup of its own that writes a partial
// result into the caller's workspace, and a second kernel adds the slices in a fixed order and applies alpha and
// the bias.
template <int MT, int PD, int KCH>
__global__ __launch_bounds__(256, 2) void lc_forward_wide_kernel(Geom g, const float *__restrict__ x,
                                                                 const float *__restrict__ w,
                                                                 const float *__restrict__ bias, float alpha,
                                                                 const float *__restrict__ alpha_dev,
                                                                 float *__restrict__ y, float *__restrict__ partial,
                                                                 int fblocks, int btiles, int nslices) {
    static_assert(PD == 2, "two steps of lookahead");
    constexpr int BT = 32 * MT, NT = 2 * MT, BUF = NT * 3 * 256;       // BUF: floats of a buffer, NT tiles of 16 images
    extern __shared__ __attribute__((aligned(16))) float xs[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kk = lane >> 4;
    // batch tiles of one (field, filter block) are neighbours in dispatch order: they share the filters in L2
    int t_id = remap_xcd(blockIdx.x, gridDim.x);
    const int bt = t_id % btiles;
    t_id /= btiles;
    const int fb = t_id % fblocks;
    t_id /= fblocks;
    const int loc = t_id % g.L, slice = t_id / g.L;
    const int i = loc / g.LW, j = loc - i * g.LW;
    const int b0 = bt * BT, f0 = fb * 128 + wave * 32;
    const int WC = g.W * g.C;
    const int cpr = g.RC / KCH, nchunks = g.R * cpr, nsteps_all = (nchunks * KCH + 31) / 32;
    // this workgroup's range of steps
    const int s_lo = (int)((long long)nsteps_all * slice / nslices);
    const int nsteps = (int)((long long)nsteps_all * (slice + 1) / nslices) - s_lo;

    f32x4 acc[NT][2];
    auto clear = [&] {
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t][0] = acc[t][1] = (f32x4){0.f, 0.f, 0.f, 0.f};
    };

    // staging: slot s moves 16 bytes (values 4 seg ..) of image tid / 8 + 32 s; images beyond the batch repeat image B-1 and
    // their results are never stored
    const int seg = tid & 7, brow = tid >> 3;
    // (32 images' first one is the wave's, the rest of a place 32 bits of bytes: a whole address a lane would cost eight registers
    // more than there are)
    gbytes xp[MT];
    unsigned xoff[MT];
#pragma unroll
    for (int s = 0; s < MT; ++s) {
        const int first = min(b0 + 32 * s, g.B - 1);
        xp[s] = (gbytes)(x + ((size_t)first * g.H + i * g.S) * WC + j * g.S * g.C);
        xoff[s] = ((unsigned)min(brow, g.B - 1 - first) * (unsigned)(g.H * WC) + (KCH == 32 ? seg : seg & 3) * 4) * 4u;
    }
    // its slot in a tile of 16 images (tile brow / 16 + 2 s), in floats, and the half of it
    const int sslot = (brow >> 4) * (3 * 256) + 4 * (4 * (brow & 15) + ((seg >> 1) ^ ((brow >> 2) & 3))), shalf = seg & 1;
    const int aslot = 4 * (4 * n + (kk ^ (n >> 2)));
    // the field's filters: lane (n, kk) has rows 8 kk .. 8 kk + 7 of a step at filters 2 n, 2 n + 1 of the wave's
    const gbytes wl = (gbytes)(w + (size_t)loc * g.K * g.F + f0);
    unsigned woff = (8u * kk * (unsigned)g.F + 2 * n) * 4u;
    // a last step of one chunk of 16: rows beyond the patch are read 16 rows earlier and count as zero
    unsigned woff_half = (8u * (kk & 1) * (unsigned)g.F + 2 * n) * 4u;

    bool nans = false;                  // (the same in all threads)
    unsigned low = 0;
    auto pass = [&](auto split_tag) {
        constexpr bool SPLIT = decltype(split_tag)::value;
        // the chunk to be staged next (it stays on the last one)
        int c = KCH == 32 ? s_lo : 2 * s_lo, kh = c / cpr, cc = c - kh * cpr;
        auto next_chunk = [&] {
            const int o = kh * WC + cc * KCH;
            if (c < nchunks - 1) {
                ++c;
                if (++cc == cpr) { cc = 0; ++kh; }
            }
            return o;
        };
        auto stage_load = [&](f32x4 (&st)[MT]) {
            const int o = next_chunk();
            if constexpr (KCH == 16) {
                const int o1 = next_chunk();
                const unsigned oh = (unsigned)(seg < 4 ? o : o1) * 4u;
#pragma unroll
                for (int s = 0; s < MT; ++s) st[s] = load_quad<float>(xp[s], xoff[s] + oh);
            } else {
#pragma unroll
                for (int s = 0; s < MT; ++s) st[s] = load_quad<float>(opaque(xp[s] + (size_t)__builtin_amdgcn_readfirstlane(o) * 4), xoff[s]);
            }
        };
        auto stage_store = [&](int step, f32x4 (&st)[MT]) {
            float *buf = xs + (step & 1) * BUF + sslot;
            if constexpr (KCH == 16) {
                if (2 * (s_lo + step) + 1 == nchunks && seg >= 4) {
#pragma unroll
                    for (int s = 0; s < MT; ++s) st[s] = (f32x4){0.f, 0.f, 0.f, 0.f};
                }
            }
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
        auto wload = [&](int step, f32x2 (&r)[8]) {
            const int sa = s_lo + min(step, nsteps - 1);
            gbytes p = wl + (size_t)(32 * sa) * (size_t)(4 * g.F);
            const bool half = KCH == 16 && 2 * sa + 1 == nchunks;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                r[q] = *(g2_ptr)(opaque(p) + (half ? woff_half : woff));
                p += 4 * g.F;
            }
        };
        f32x4 st[PD][MT];
        f32x2 wr[PD][8];
#pragma unroll
        for (int p = 0; p < PD; ++p) wload(p, wr[p]);
        stage_load(st[0]);
        stage_store(0, st[0]);
#pragma unroll
        for (int p = 0; p < PD; ++p) stage_load(st[p]);             // set p: step p + 1
        __syncthreads();
        for (int c0 = 0; c0 < nsteps; c0 += 2) {
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const int step = c0 + p;            // it lies in buffer p, and the set p holds the next one's images
                if (step < nsteps) {
                    const float *ab = xs + p * BUF + aslot;
                    float e[2][8];
#pragma unroll
                    for (int u = 0; u < 2; ++u)
#pragma unroll
                        for (int q = 0; q < 8; ++q) e[u][q] = wr[p][q][u];
                    if constexpr (KCH == 16) {
                        // (an infinite weight times the zero of an image is a NaN)
                        if (2 * (s_lo + step) + 1 == nchunks && kk >= 2) {
#pragma unroll
                            for (int u = 0; u < 2; ++u)
#pragma unroll
                                for (int q = 0; q < 8; ++q) e[u][q] = 0.f;
                        }
                    }
                    if constexpr (SPLIT) {
                        const Parts pb[2] = {split8(e[0], low), split8(e[1], low)};
                        wload(step + PD, wr[p]);
#pragma unroll
                        for (int t = 0; t < NT; t += 2) {
                            Parts pa[2];
#pragma unroll
                            for (int m = 0; m < 2; ++m)
#pragma unroll
                                for (int q = 0; q < 3; ++q) pa[m].p[q] = *(const u32x4 *)(ab + ((t + m) * 3 + q) * 256);
                            mfma_split_rows(pa, pb, acc + t);
                            // (four tiles read ahead, not eight: the registers of the largest batch tile; 651 -> 638 us)
                            if (MT == 4 && t + 2 == NT / 2) __builtin_amdgcn_sched_barrier(0);
                        }
                    } else {
                        wload(step + PD, wr[p]);
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
                    // the other buffer was last read in the step before, which every wave left at the barrier
                    if (step + 1 < nsteps) stage_store(step + 1, st[p]);
                    if (step + 1 + PD < nsteps) stage_load(st[p]);
                }
                // Operands of a diverged layer show in the first two steps: the fp32 pass starts there and then, unless
                // every filter has a NaN among its first weights, so that no sum is anything else.
                if (SPLIT && p == 1 && c0 == 0) {
                    if (__syncthreads_or(!all_finite<2 * NT>(&acc[0][0]) || inexact(low))) {
                        f32x2 first[8];
                        wload(0, first);
                        bool a = false, b = false;
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            a |= first[q][0] != first[q][0];
                            b |= first[q][1] != first[q][1];
                        }
                        const unsigned long long ma = __ballot(a), mb = __ballot(b);
                        nans = !__syncthreads_or(!every_column(ma) || !every_column(mb));
                        if (!nans) return;
                    }
                } else {
                    __syncthreads();
                }
            }
        }
    };
    clear();
    if (nsteps > 0) {
        pass(std::true_type{});
        // an operand that is not finite or too small, or a part that overflowed: once more in fp32
        if (!nans && __syncthreads_or(!all_finite<2 * NT>(&acc[0][0]) || inexact(low))) {
            clear();
            pass(std::false_type{});
        }
    }

    const bool whole = nslices == 1;
    if (whole && alpha_dev) alpha = *alpha_dev;
    f32x2 bv = (f32x2){0.f, 0.f};
    if (whole && bias) bv = *(const f32x2 *)(bias + (size_t)loc * g.F + f0 + 2 * n);
    float *yo = whole ? y : partial + (size_t)slice * g.B * g.L * g.F;
    const float sc = whole ? alpha : 1.f;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) {
            const int b = b0 + 16 * t + 4 * kk + rr;
            if (b >= g.B) continue;
            const f32x2 o = {sc * acc[t][0][rr] + bv[0], sc * acc[t][1][rr] + bv[1]};
            *(f32x2 *)(yo + ((size_t)b * g.L + loc) * g.F + f0 + 2 * n) = o;
        }
}

// y = alpha * (sum of the slices, in order) + bias
__global__ __launch_bounds__(256) void lc_forward_slices_kernel(const float *__restrict__ partial, int nslices,
                                                                size_t n4, int LF4, const float *__restrict__ bias,
                                                                float alpha, const float *__restrict__ alpha_dev,
                                                                float *__restrict__ y) {
    if (alpha_dev) alpha = *alpha_dev;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < n4; e += (size_t)gridDim.x * 256) {
        f32x4 s = ((const f32x4 *)partial)[e];
        for (int k = 1; k < nslices; ++k) s += ((const f32x4 *)partial)[(size_t)k * n4 + e];
        f32x4 bv = (f32x4){0.f, 0.f, 0.f, 0.f};
        if (bias) bv = ((const f32x4 *)bias)[e % (size_t)LF4];
        ((f32x4 *)y)[e] = alpha * s + bv;
    }
}

int chunk_floats(const Geom &g) { return g.RC % 32 == 0 ? 32 : 16; }

// slices that would give a layer with few fields about two rounds of workgroups; 1 = no split
int wide_slices(const Geom &g) {
    const long long wgs = (long long)g.L * (g.F / 128) * ((g.B + 127) / 128);
    if (wgs >= 256) return 1;
    const int nchunks = g.R * (g.RC / chunk_floats(g));
    int ns = (int)((1024 + wgs - 1) / wgs);
    if (ns > 16) ns = 16;
    if (ns > nchunks / 8) ns = nchunks / 8;      // keep slices long enough to amortise their pipeline fill
    return ns < 2 ? 1 : ns;
}

// Host check of a lc_forward_wide_kernel launch.  tparam = {MT, PD, KCH}; arg = {filter blocks, batch tiles, slices}.
int check_forward_wide(const Geom &g, const LaunchPlan &p) {
    const int MT = p.tparam[0], KCH = p.tparam[2];
    const int fblocks = p.arg[0], btiles = p.arg[1], nslices = p.arg[2];
    const int BT = 32 * MT;
    LC_PLAN_REQUIRE(p, p.block == 256 && (KCH == 32 || KCH == 16));
    // 128 filters per workgroup; patch rows in whole chunks whose starts are 16-byte aligned in every image row
    LC_PLAN_REQUIRE(p, g.F % 128 == 0 && fblocks == g.F / 128);
    LC_PLAN_REQUIRE(p, g.RC % KCH == 0 && (g.S * g.C) % 4 == 0 && (g.W * g.C) % 4 == 0);
    LC_PLAN_REQUIRE(p, btiles == ceil_div(g.B, BT));
    // 32-bit byte offsets into 32 images
    LC_PLAN_REQUIRE(p, (long long)32 * g.H * g.W * g.C * 4 < (1LL << 32));
    const int nchunks = g.R * (g.RC / KCH);
    LC_PLAN_REQUIRE(p, nslices >= 1 && nslices <= nchunks);
    LC_PLAN_REQUIRE(p, (long long)p.grid[0] == (long long)g.L * fblocks * btiles * nslices && p.grid[1] == 1 &&
                           p.grid[2] == 1);
    // two buffers of three parts of bf16, or of fp32 values where a result is not finite; a lane's 32-bit byte offset into a
    // step's filters: row 24 at most, eight rows on from the wave's (33 million filters, a field's most, are 3.2e9)
    LC_PLAN_REQUIRE(p, p.lds_bytes >= (size_t)2 * BT * 32 * 6 && (24LL * g.F + 32) * 4 <= (1LL << 32));
    return LC_OK;
}

template <int KCH, int MT = 4>
int launch_wide(const Geom &g, const float *x, const float *w, const float *bias, float alpha, const float *alpha_dev,
                float *y, float *partial, int nslices, hipStream_t s) {
    constexpr int PD = 2, BT = 32 * MT;
    const size_t lds = (size_t)2 * BT * 32 * 6;
    auto kern = lc_forward_wide_kernel<MT, PD, KCH>;
    const int fblocks = g.F / 128, btiles = (g.B + BT - 1) / BT;
    const LaunchPlan plan = make_plan("lc_forward_wide", {MT, PD, KCH}, {fblocks, btiles, nslices},
                                      dim3((unsigned)(g.L * fblocks * btiles * nslices)), 256, lds);
    if (int rc = check_forward_wide(g, plan)) return rc;
    LC_LAUNCH(plan, "lc_forward (wide) launch", kern, s, g, x, w, bias, alpha, alpha_dev, y, partial, fblocks, btiles,
              nslices);
    if (nslices > 1) {
        const size_t n4 = (size_t)g.B * g.L * g.F / 4;
        const unsigned blocks = (unsigned)std::min<size_t>((n4 + 255) / 256, 256 * 16);
        const LaunchPlan sum = make_plan("lc_forward_slices", {}, {nslices}, dim3(blocks), 256, 0);
        LC_LAUNCH(sum, "lc_forward (slices) launch", lc_forward_slices_kernel, s, partial, nslices, n4, g.L * g.F / 4,
                  bias, alpha, alpha_dev, y);
    }
    return LC_OK;
}

}  // namespace

// 128-filter blocks, patch rows that split into chunks with 16-byte aligned starts, offsets in 32 bits.  Chunks of
// 32 values always; chunks of 16 only for layers with few fields: with many overlapping fields of few channels
// (the paper's first layer) the strip-sharing kernel reads the patches far less often and is the faster one.
bool forward_wide_supported(const Geom &g) {
    const bool few_fields = (long long)g.L * (g.F / 128) * ((g.B + 127) / 128) < 256;
    return g.F % 128 == 0 && (g.RC % 32 == 0 || (g.RC % 16 == 0 && few_fields)) && (g.S * g.C) % 4 == 0 &&
           (g.W * g.C) % 4 == 0 && g.B > 64 &&
           (long long)g.B * g.H * g.W * g.C < (1ll << 31) &&
           (long long)g.L * (g.F / 128) * ((g.B + 127) / 128) * 16 < (1ll << 31);
}

// workspace that lets lc_forward cut the contraction of a layer with few fields into slices (0: not needed, or the layer
// runs another kernel)
size_t forward_wide_workspace_bytes(const Geom &g) {
    if (!forward_takes_wide(g)) return 0;
    const int ns = wide_slices(g);
    return ns > 1 ? (size_t)ns * g.B * g.L * g.F * sizeof(float) : 0;
}

int launch_forward_wide_f32(const Geom &g, const float *x, const float *w, const float *bias, float alpha,
                            const float *alpha_dev, float *y, void *ws, size_t ws_bytes, hipStream_t s) {
    if (!forward_wide_supported(g)) return LC_EUNSUPPORTED;
    int ns = wide_slices(g);
    if (ns > 1 && (!ws || ws_bytes < forward_wide_workspace_bytes(g))) ns = 1;   // no workspace: one slice
    // batch tile of 128, 96 or 64 images: the one that pads the batch least, the larger one on a tie (B = 192: two
    // tiles of 128 waste a quarter of the MFMAs)
    const int mt = batch_tile_mt(g.B, true);
    if (chunk_floats(g) == 32) {
        if (mt == 2) return launch_wide<32, 2>(g, x, w, bias, alpha, alpha_dev, y, (float *)ws, ns, s);
        if (mt == 3) return launch_wide<32, 3>(g, x, w, bias, alpha, alpha_dev, y, (float *)ws, ns, s);
        return launch_wide<32>(g, x, w, bias, alpha, alpha_dev, y, (float *)ws, ns, s);
    }
    if (mt == 2) return launch_wide<16, 2>(g, x, w, bias, alpha, alpha_dev, y, (float *)ws, ns, s);
    if (mt == 3) return launch_wide<16, 3>(g, x, w, bias, alpha, alpha_dev, y, (float *)ws, ns, s);
    return launch_wide<16>(g, x, w, bias, alpha, alpha_dev, y, (float *)ws, ns, s);
}

}  // namespace lc
