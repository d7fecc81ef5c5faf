// lc_backward_data for any geometry: dx[b,p] = sum over fields l containing pixel p, sum_f w[l,k(p,l),f] * dy[b,l,f]
// (Eq. 1's reconstruction "W^T h").  Gather form, no atomics.
//
// A wave's task is a block of PR x PC pixels (whole multiples of the stride), 16*MT images and 16*NT of the block's
// PR*PC*C values.  It contracts over every filter of every field that touches the block: the fields form a rectangle of
// the field grid, and (field row, field column, four consecutive filters) are walked as one list of vectors, lane (m,kk)
// taking every fourth from kk on.  Four filters are contiguous in dy (A operand, image m) and in w (B operand, the weight
// row of the lane's value in that field), so both come as one vector load each from global memory straight into the MFMAs.
// Where the block is one S x S cell and the fields tile the cells, every field of the rectangle covers every value;
// otherwise a value outside a field takes zero weights.  Blocks larger than a cell fill the 16 columns of an MFMA tile
// where a cell has few values (S*S*C < 16) at the price of those zeros.  (A zero weight keeps a finite dy out, not an
// infinite one: tiles that come out with a NaN are formed again from the fields that contain each value alone.)  The last
// vector of a field's filters ends at F-1, and its elements that the one before it holds already count as zero in both
// operands.
#include <type_traits>

#include "lc_general.hpp"

namespace lc {

constexpr int kBackDataWaves = 8;   // per workgroup at most
constexpr int kMostBlocks = 65535;  // blocks of a pixel block's values: the grid's second dimension

// floor(a / d) for 0 <= a < 2^20 from inv = 1 / d
__device__ __forceinline__ int small_div(int a, float inv) { return (int)(((float)a + 0.5f) * inv); }

// VW consecutive filters of one row: two quads in fp32, one 16-byte vector in bf16 (VW = 8), or half of that (VW = 4)
template <typename T, int VW>
struct Vec {
    typename Quad<T>::V q[VW / 4];
    __device__ __forceinline__ void load(gbytes base, unsigned off) {
#pragma unroll
        for (int h = 0; h < VW / 4; ++h) q[h] = load_quad<T>(base, off + h * 16);
    }
};
template <>
struct Vec<bf16_t, 8> {
    u32x4 v;
    __device__ __forceinline__ void load(gbytes base, unsigned off) {
        typedef __attribute__((address_space(1), aligned(2))) u32x4 GV;
        v = *(const GV *)(base + off);
    }
};

// acc += the products of 4*VW filters of 16 images and 16 values; the first `skip` elements of the lane's vectors are left out
template <typename T, int VW>
__device__ __forceinline__ f32x4 product(const Vec<T, VW> &a, const Vec<T, VW> &b, int skip, f32x4 acc) {
    if constexpr (sizeof(T) == 4) {
#pragma unroll
        for (int t = 0; t < VW; ++t)
            acc = mfma16(t < skip ? 0.f : a.q[t / 4][t % 4], t < skip ? 0.f : b.q[t / 4][t % 4], acc);
        return acc;
    } else if constexpr (VW == 8) {
        return mfma32_bf16(clear_below(a.v, skip), clear_below(b.v, skip), acc);
    } else {
        return mfma16_bf16(clear_below(a.q[0], skip), clear_below(b.q[0], skip), acc);
    }
}

template <int MT, int NT, typename T, int VW, bool MASK>
__global__ __launch_bounds__(64 * kBackDataWaves) void lc_bwd_data_general_kernel(
    Geom g, const T *__restrict__ dy, const T *__restrict__ w, float *__restrict__ dx, int PR, int PC, int cbc, int NVF,
    int nbt, int ks, int ntask) {
    constexpr int ES = sizeof(T), PF = VW == 4 && MT * NT <= 4 ? 4 : 2;   // groups of 4*VW filters in flight
    // Whether a value's column is only looked at where its row is in the field: fp32 tiles of four and eight blocks over several
    // image tiles are faster with the branch (82 images of 143 x 74 x 64, 15 x 15 at stride 7, 14 filters 253 -> 226 us, 256 of 152 x
    // 50 x 1, 19 x 19, 14 filters 410 -> 378; 25 layers 1.02 on average), all others without it (240 layers 1.01, one image tile 1.02).
    constexpr bool BRANCH = ES == 4 && MT > 1 && (MT * NT == 4 || MT * NT == 8);
    extern __shared__ __attribute__((aligned(16))) f32x4 slices[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, kk = lane >> 4;
    // waves of a workgroup: slices of the contraction innermost, then tasks (pixel block, batch tile), whose neighbours
    // share most of their fields' dy
    const int slice = wave % ks, grp = wave / ks;
    const int tasks = (blockDim.x >> 6) / ks;
    const int task = remap_xcd(blockIdx.x, gridDim.x) * tasks + grp;
    const int n0 = blockIdx.y * (NT * 16), N = PR * PC * g.C;
    const bool active = task < ntask;
    const int tk = min(task, ntask - 1);
    const int blk = tk / nbt, b0 = (tk - blk * nbt) * (16 * MT);
    const int rb = blk / cbc, r0 = rb * PR, c0 = (blk - rb * cbc) * PC;
    // the fields that touch the block
    const int i_lo = max(0, (r0 - g.R + g.S) / g.S), i_hi = min(g.LH - 1, (r0 + PR - 1) / g.S);
    const int j_lo = max(0, (c0 - g.R + g.S) / g.S), j_hi = min(g.LW - 1, (c0 + PC - 1) / g.S);
    const int na = i_hi - i_lo + 1, nap = j_hi - j_lo + 1;
    const int nvt = na > 0 && nap > 0 ? na * nap * NVF : 0;

    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // the values this lane supplies weights for and stores: their places relative to field (i_lo, j_lo), and the byte
    // offset of their weight row from that field's first one
    int rr[NT], cc[NT];
    unsigned kn[NT];
    bool nok[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int v = n0 + nt * 16 + m;
        nok[nt] = v < N;
        const int vc = nok[nt] ? v : 0;
        const int dr = vc / (PC * g.C), rem = vc - dr * (PC * g.C), dc = rem / g.C;
        rr[nt] = r0 + dr - i_lo * g.S;
        cc[nt] = c0 + dc - j_lo * g.S;
        kn[nt] = (unsigned)((rr[nt] * g.RC + cc[nt] * g.C + (rem - dc * g.C)) * g.F) * ES;
    }

    if (nvt > 0) {
        const size_t dyimg = (size_t)g.L * g.F;
        const size_t first = (size_t)i_lo * g.LW + j_lo;
        const gbytes yp = (gbytes)(dy + (size_t)b0 * dyimg + first * g.F);
        const gbytes wp = (gbytes)(w + first * g.K * g.F);
        unsigned ro[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) ro[mt] = (unsigned)((size_t)min(mt * 16 + m, g.B - 1 - b0) * dyimg) * ES;
        const int per = (((nvt + 3) >> 2) + ks - 1) / ks * 4;
        const int vbeg = slice * per, vend = min(vbeg + per, nvt);
        const float inv_f = 1.0f / (float)NVF, inv_a = 1.0f / (float)nap;
        const int last = MASK ? VW * NVF - g.F : 0;            // elements the last vector shares with the one before it
        const int arow = g.LW * g.K - g.S * g.RC, acol = g.K - g.S * g.C;
        int vi = vbeg + kk;
        Vec<T, VW> a[PF][MT], b[PF][NT];
        int skip[PF];                                          // leading elements that count as zero
        unsigned bad[PF];                                      // bit nt: value nt lies outside the field
        auto load = [&](int s) {
            const bool in = vi < vend;
            const int vc = in ? vi : 0;
            const int fi = small_div(vc, inv_f), fv = vc - fi * NVF;
            const int fa = small_div(fi, inv_a), fp = fi - fa * nap;
            const int sh = MASK && fv == NVF - 1 ? last : 0, fo = VW * fv - sh;
            const unsigned aoff = (unsigned)((fa * g.LW + fp) * g.F + fo) * ES;
            const unsigned boff = (unsigned)((fa * arow + fp * acol) * g.F + fo) * ES;
            skip[s] = in ? sh : VW;
            bad[s] = 0;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) a[s][mt].load(yp, ro[mt] + aoff);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                unsigned off = boff + kn[nt];
                if (MASK) {
                    const bool row = (unsigned)(rr[nt] - fa * g.S) < (unsigned)g.R;
                    const bool ok = BRANCH ? row && (unsigned)(cc[nt] - fp * g.S) < (unsigned)g.R
                                           : row & ((unsigned)(cc[nt] - fp * g.S) < (unsigned)g.R);
                    if (!ok) { off = 0; bad[s] |= 1u << nt; }
                }
                b[s][nt].load(wp, off);
            }
            vi += 4;
        };
        auto multiply = [&](int s, auto masked) {
            constexpr bool M = decltype(masked)::value;
            if constexpr (ES == 4) {
#pragma unroll
                for (int t = 0; t < VW; ++t) {
                    const bool z = M && t < skip[s];
                    float bv[NT];
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        bv[nt] = z || (M && MASK && ((bad[s] >> nt) & 1u)) ? 0.f : b[s][nt].q[t / 4][t % 4];
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const float av = z ? 0.f : a[s][mt].q[t / 4][t % 4];
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = mfma16(av, bv[nt], acc[mt][nt]);
                    }
                }
            } else {
                typedef std::conditional_t<VW == 8, u32x4, u32x2> BV;
                auto bits = [](const Vec<T, VW> &x) -> BV {
                    if constexpr (VW == 8) return x.v;
                    else return x.q[0];
                };
                BV bv[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    bv[nt] = bits(b[s][nt]);
                    if (M) bv[nt] = clear_below(bv[nt], MASK && ((bad[s] >> nt) & 1u) ? VW : skip[s]);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    BV av = bits(a[s][mt]);
                    if (M) av = clear_below(av, skip[s]);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        if constexpr (VW == 8) acc[mt][nt] = mfma32_bf16(av, bv[nt], acc[mt][nt]);
                        else acc[mt][nt] = mfma16_bf16(av, bv[nt], acc[mt][nt]);
                    }
                }
            }
        };
        const int nvec = max(vend - vbeg, 0), ng = (nvec + 3) >> 2, nfull = nvec >> 2;
        if (ng > 0 && active) {
#pragma unroll
            for (int s = 0; s < PF; ++s) {
                load(s);
                __builtin_amdgcn_sched_barrier(0);
            }
            int done = 0;
            for (; done + PF <= nfull; done += PF) {
#pragma unroll
                for (int s = 0; s < PF; ++s) {
                    multiply(s, std::bool_constant<MASK>{});
                    load(s);
                    // the refill of a slot stays right behind the MFMAs that used it
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
#pragma unroll
            for (int s = 0; s < PF; ++s)
                if (done + s < ng) multiply(s, std::true_type{});
        }
    }
    add_slices<MT * NT>(&acc[0][0], slices, grp, slice, ks);
    if (!active || slice != 0) return;

    unsigned again = 0;                                        // bit mt*NT + nt: the tile holds a NaN
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int v = n0 + nt * 16 + m;
        const int row = rr[nt] + i_lo * g.S, col = cc[nt] + j_lo * g.S;
        const bool stored = nok[nt] && row < g.H && col < g.W;
        float *o = dx + (size_t)row * g.W * g.C + (size_t)c0 * g.C + v % (PC * g.C);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            bool nan = false;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int b = b0 + mt * 16 + 4 * kk + r;
                if (!stored || b >= g.B) continue;
                o[(size_t)b * g.H * g.W * g.C] = acc[mt][nt][r];
                nan |= acc[mt][nt][r] != acc[mt][nt][r];
            }
            if (MASK && __any(nan)) again |= 1u << (mt * NT + nt);
        }
    }
    // The zero weights of a value outside a field make a NaN of an infinite or NaN dy of that field (an infinite sum has met
    // none, and stays).  A tile with a NaN is formed again field by field, each field's part added only to the values it
    // contains; once all are NaN, it ends.  Where the fields tile the cells there are no such weights.  (32 images of
    // 60 x 60 x 3, 11 x 11 at stride 4, 96 filters, every dy infinite: 120 us, the finite pass 23; product by product and
    // value by value it took 2683.)
    if constexpr (MASK) {
        if (again == 0 || (PR == g.S && PC == g.S && g.R % g.S == 0)) return;
        constexpr int STEPS = VW == 8 ? 2 : 4;                 // groups of 4*VW filters in flight
        const size_t dyimg = (size_t)g.L * g.F, first = (size_t)i_lo * g.LW + j_lo;
        const int last = VW * NVF - g.F;
        while (again) {
            const int tile = __ffs(again) - 1, mt = tile / NT, nt = tile - mt * NT;
            again &= again - 1;
            const int v = n0 + nt * 16 + m, vc = v < N ? v : 0;
            const int dr = vc / (PC * g.C), rem = vc - dr * (PC * g.C), dc = rem / g.C;
            const int r1 = r0 + dr - i_lo * g.S, c1 = c0 + dc - j_lo * g.S;      // as rr, cc and kn
            const unsigned k1 = (unsigned)((r1 * g.RC + c1 * g.C + (rem - dc * g.C)) * g.F) * ES;
            const gbytes yp = (gbytes)(dy + (size_t)min(b0 + mt * 16 + m, g.B - 1) * dyimg + first * g.F);
            const gbytes wp = (gbytes)(w + first * g.K * g.F);
            f32x4 sum = (f32x4){0.f, 0.f, 0.f, 0.f};
            for (int fi = 0; fi < na * nap; ++fi) {
                const int fa = fi / nap, fp = fi - fa * nap;
                const bool ok = v < N && (unsigned)(r1 - fa * g.S) < (unsigned)g.R && (unsigned)(c1 - fp * g.S) < (unsigned)g.R;
                if (!__any(ok)) continue;
                const unsigned aoff = (unsigned)((fa * g.LW + fp) * g.F) * ES;
                const unsigned boff = (unsigned)((fa * (g.LW * g.K - g.S * g.RC) + fp * (g.K - g.S * g.C)) * g.F) * ES + k1;
                f32x4 part = (f32x4){0.f, 0.f, 0.f, 0.f};
                for (int f0 = 0; f0 < NVF; f0 += 4 * STEPS) {
                    Vec<T, VW> a[STEPS], b[STEPS];
                    int skip[STEPS];
#pragma unroll
                    for (int s = 0; s < STEPS; ++s) {
                        const int fv = f0 + 4 * s + kk;
                        const bool in = fv < NVF;
                        const int sh = fv == NVF - 1 ? last : 0;
                        const unsigned fo = (unsigned)(in ? VW * fv - sh : 0) * ES;
                        skip[s] = in ? sh : VW;
                        a[s].load(yp, aoff + fo);
                        b[s].load(wp, ok ? boff + fo : 0u);
                    }
#pragma unroll
                    for (int s = 0; s < STEPS; ++s) part = product<T, VW>(a[s], b[s], skip[s], part);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) sum[r] += ok ? part[r] : 0.f;
                bool open = false;
#pragma unroll
                for (int r = 0; r < 4; ++r) open |= sum[r] == sum[r];
                if (!__any(v < N && open)) break;
            }
            const int row = r0 + dr, col = c0 + dc;
            const bool stored = v < N && row < g.H && col < g.W;
            float *o = dx + ((size_t)row * g.W + col) * g.C + (rem - dc * g.C);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int b = b0 + mt * 16 + 4 * kk + r;
                if (stored && b < g.B) {
                    float *p = o + (size_t)b * g.H * g.W * g.C;
                    if (*p != *p) *p = sum[r];
                }
            }
        }
    }
}

namespace {

// Filters per vector.  Eight fetch a row's cache line at once where four come back for it (bf16: and halve the loads per
// MFMA: 128 images of 50 x 73 x 64, 12 x 12 fields at stride 8, 128 filters 163 -> 97 us; fp32 within 5 % either way);
// four where eight pad the filters by more than a quarter (9 filters, bf16: 22 -> 18 us).
int vector_width(const Geom &g) { return g.F >= 8 && ceil_div(g.F, 8) * 8 <= 5 * ceil_div(g.F, 4) ? 8 : 4; }

// Host check of a lc_bwd_data_general_kernel launch.  tparam = {MT, NT, bytes per operand element, MASK, slices of the
// contraction, tasks per workgroup, VW}; arg = {PR, PC, pixel blocks per row, vectors per field's filters, batch tiles,
// tasks}.
int check_backward_data_general(const Geom &g, const LaunchPlan &p) {
    const int MT = p.tparam[0], NT = p.tparam[1], ES = p.tparam[2], MASK = p.tparam[3], ks = p.tparam[4], tasks = p.tparam[5], VW = p.tparam[6];
    const int PR = p.arg[0], PC = p.arg[1], cbc = p.arg[2], NVF = p.arg[3], nbt = p.arg[4], ntask = p.arg[5];
    LC_PLAN_REQUIRE(p, MT >= 1 && MT <= 4 && NT >= 1 && NT <= 4 && (ES == 4 || ES == 2));
    LC_PLAN_REQUIRE(p, ks >= 1 && (ks & (ks - 1)) == 0 && tasks >= 1);
    LC_PLAN_REQUIRE(p, (int)p.block == 64 * ks * tasks && (int)p.block <= 64 * kBackDataWaves);
    LC_PLAN_REQUIRE(p, PR >= g.S && PR % g.S == 0 && PC >= g.S && PC % g.S == 0 && cbc == ceil_div(g.W, PC));
    // no masks: every field of a block's rectangle covers all of the block, filters in whole vectors
    LC_PLAN_REQUIRE(p, MASK || (PR == g.S && PC == g.S && g.R % g.S == 0 && g.F % VW == 0));
    LC_PLAN_REQUIRE(p, (VW == 4 || VW == 8) && g.F >= VW && NVF == ceil_div(g.F, VW) && nbt == ceil_div(g.B, 16 * MT));
    const long long blocks = (long long)ceil_div(g.H, PR) * cbc, N = (long long)PR * PC * g.C;
    LC_PLAN_REQUIRE(p, (long long)ntask == blocks * nbt);
    LC_PLAN_REQUIRE(p, (long long)p.grid[0] * tasks >= ntask && (long long)(p.grid[0] - 1) * tasks < ntask);
    LC_PLAN_REQUIRE(p, (long long)p.grid[1] * NT * 16 >= N && (long long)(p.grid[1] - 1) * NT * 16 < N && p.grid[2] == 1);
    LC_PLAN_REQUIRE(p, ks == 1 || p.lds_bytes >= (size_t)tasks * (ks / 2) * MT * NT * 1024);
    // the divisions by small_div; 32-bit byte offsets: into a batch tile's dy, from a block's first field into w
    const long long nfr = PR / g.S + (g.R - 1) / g.S + 1, nfc = PC / g.S + (g.R - 1) / g.S + 1;
    LC_PLAN_REQUIRE(p, nfr * nfc * NVF < (1LL << 20));
    LC_PLAN_REQUIRE(p, (long long)16 * MT * g.L * g.F * ES < (1LL << 32) && (nfr * g.LW + nfc) * g.K * g.F * ES < (1LL << 32));
    return LC_OK;
}

template <int MT, int NT, int VW, typename T>
int launch_tile(const Geom &g, const T *dy, const T *w, float *dx, const DataTile &t, hipStream_t s) {
    const int PR = g.S * t.qr, PC = g.S * t.qc, cbc = ceil_div(g.W, PC), NVF = ceil_div(g.F, VW), nbt = ceil_div(g.B, 16 * MT);
    const long long ntask = (long long)ceil_div(g.H, PR) * cbc * nbt;
    const bool mask = !(t.qr == 1 && t.qc == 1 && g.R % g.S == 0 && g.F % VW == 0);
    const size_t lds = (size_t)t.tasks * (t.ks / 2) * MT * NT * 1024;
    dim3 grid((unsigned)((ntask + t.tasks - 1) / t.tasks), ceil_div(PR * PC * g.C, NT * 16));
    const LaunchPlan plan = make_plan("lc_bwd_data_general", {MT, NT, (int)sizeof(T), mask, t.ks, t.tasks, VW},
                                      {PR, PC, cbc, NVF, nbt, (int)ntask}, grid, 64 * t.ks * t.tasks, lds);
    if (int rc = check_backward_data_general(g, plan)) return rc;
    if (mask)
        LC_LAUNCH(plan, "lc_backward_data launch", (lc_bwd_data_general_kernel<MT, NT, T, VW, true>), s, g, dy, w, dx, PR, PC, cbc,
                  NVF, nbt, t.ks, (int)ntask);
    else
        LC_LAUNCH(plan, "lc_backward_data launch", (lc_bwd_data_general_kernel<MT, NT, T, VW, false>), s, g, dy, w, dx, PR, PC, cbc,
                  NVF, nbt, t.ks, (int)ntask);
    return LC_OK;
}

// The pixel block, the tile and the number of slices by estimated time, as in the forward pass: a group costs a wave its
// MFMAs and mainly the loads of its images' dy; the constants are a fit to 33 layers timed with several blocks, every tile
// and every number of slices (batches of 2 to 256, 9 to 373 filters, both types): what is picked is on average 8 % slower
// than the fastest of its layer.  (Two blocks of values of one pixel block in a workgroup, sharing its dy, took up to 1.5
// times as long as neighbouring pixel blocks, and more than eight waves per workgroup gained nothing.)
DataTile pick_tile(const Geom &g, int es) {
    DataTile best = {1, 1, 4, 1, 1, 1};
    double best_t = 1e300;
    const int NVF = ceil_div(g.F, vector_width(g));
    const double per_mfma = es == 4 ? 32.0 * vector_width(g) : 32.0;
    for (int qr : {1, 2, 3, 4, 6, 8, 12, 16})
        for (int qc : {1, 2, 3, 4, 6, 8, 12, 16}) {
            const long long N = (long long)qr * qc * g.S * g.S * g.C;
            if ((qr > 1 || qc > 1) && (N > 64 || qr > ceil_div(g.H, g.S) || qc > ceil_div(g.W, g.S))) continue;
            double fr, fc;
            int mr, mc;
            fields_across(g, qr, g.H, g.LH, &fr, &mr);
            fields_across(g, qc, g.W, g.LW, &fc, &mc);
            const double groups_all = fr * fc * NVF / 4, blocks = (double)ceil_div(g.H, g.S * qr) * ceil_div(g.W, g.S * qc);
            const int groups = ceil_div(mr * mc * NVF, 4);
            for (int mt = 1; mt <= 4; ++mt) {
                if (mt > 1 && 16 * (mt - 1) >= g.B) break;
                if (blocks * ceil_div(g.B, 16 * mt) > kMostTasks) continue;
                for (int nt = 1; nt <= 4; ++nt) {
                    if (nt > 1 && 16 * (nt - 1) >= N) break;
                    if ((N + 16 * nt - 1) / (16 * nt) > kMostBlocks) continue;
                    const double tiles = (double)ceil_div(g.B, 16 * mt) * (double)((N + 16 * nt - 1) / (16 * nt));
                    const double mm = per_mfma * mt * nt, group = mm + 11 + 96.0 * mt + 16.0 * nt;
                    for (int ks = 1, lg = 0; ks <= kBackDataWaves && (ks == 1 || 2 * ks <= groups); ks *= 2, ++lg) {
                        const double add = 1060 + (ks > 1 ? 93.0 * mt * nt + 2060.0 * lg : 0);
                        const double busy = tiles * (groups_all * group + blocks * ks * add) / 1024;
                        const double alone = 2.86 * ((double)groups / ks * (mm + 800) + 844.0 * lg);
                        if (busy + alone < best_t) {
                            best_t = busy + alone;
                            best = {mt, nt, ks >= 4 ? 1 : 4 / ks, ks, qr, qc};
                        }
                    }
                }
            }
        }
    return best;
}

template <int VW, typename T>
int launch_width(const Geom &g, const T *dy, const T *w, float *dx, hipStream_t s) {
    static thread_local TileMemo<DataTile> memo;
    const DataTile t = memo.get(g, sizeof(T), pick_tile);
    if (backward_data_turned_takes(g, sizeof(T)))
        return launch_backward_data_turned(g, dy, w, dx, t, VW, s);
#define LC_TILE(M, N) if (t.mt == M && t.nt == N) return launch_tile<M, N, VW>(g, dy, w, dx, t, s)
    LC_TILE(1, 1); LC_TILE(2, 1); LC_TILE(3, 1); LC_TILE(4, 1);
    LC_TILE(1, 2); LC_TILE(2, 2); LC_TILE(3, 2); LC_TILE(4, 2);
    LC_TILE(1, 3); LC_TILE(2, 3); LC_TILE(3, 3); LC_TILE(4, 3);
    LC_TILE(1, 4); LC_TILE(2, 4); LC_TILE(3, 4); LC_TILE(4, 4);
#undef LC_TILE
    return LC_EINTERNAL;
}

template <typename T>
int launch_general(const Geom &g, const T *dy, const T *w, float *dx, hipStream_t s) {
    return vector_width(g) == 8 ? launch_width<8>(g, dy, w, dx, s) : launch_width<4>(g, dy, w, dx, s);
}

}  // namespace

bool backward_data_general_supported(const Geom &g, int es) {
    const long long NVF = ceil_div(g.F, 4), nf = 17 + (g.R - 1) / g.S;   // at most 16 strides per block
    // the widest tile's blocks of a cell's values fit the grid, and its tasks their numbers: strides of hundreds of pixels
    // and billions of cells leave to the masked kernel
    return g.F >= 4 && (long long)ceil_div(g.H, g.S) * ceil_div(g.W, g.S) * ceil_div(g.B, 64) <= kMostTasks &&
           (long long)g.S * g.S * g.C <= 64LL * kMostBlocks && nf * nf * NVF < (1LL << 20) &&
           (long long)64 * g.L * g.F * es < (1LL << 32) && (nf * g.LW + nf) * g.K * g.F * es < (1LL << 32);
}

int launch_backward_data_general_f32(const Geom &g, const float *dy, const float *w, float *dx, hipStream_t s) {
    return launch_general(g, dy, w, dx, s);
}

int launch_backward_data_general_bf16(const Geom &g, const void *dy, const void *w, float *dx, hipStream_t s) {
    return launch_general(g, (const bf16_t *)dy, (const bf16_t *)w, dx, s);
}

}  // namespace lc
