// lc_forward for any geometry: y[b,l,f] = alpha * sum_k w[l,k,f] * patch(x)[b,l,k] + bias[l,f] (Eq. 1's "alpha W x",
// untied receptive fields of Sec. 3.1).
//
// A wave's task is one field, 16*MT images and 16*NT filters.  Both operands go from global memory straight into the
// MFMAs: lane (m,kk) loads four consecutive patch values of image m as its A operand, and NT consecutive filters of the
// same four patch elements' weight rows as its B operand, so a group of 16 patch elements is MT + 4 vector loads for
// 4*MT*NT MFMAs (fp32; on bf16 storage MT*NT MFMAs after a 4 x 4 transpose in registers).  Patch rows of any length are
// walked in vectors of four: the last vector of a row starts at RC-4 and its elements that the one before it holds
// already are set to zero in both operands.  Filters of any number are covered by runs that end at F-1: a run that
// would cross the end starts earlier, and the filters it shares with its neighbour are computed twice and stored alike.
// Images past the batch repeat the last one and are not stored.
#include <type_traits>

#include "lc_general.hpp"

namespace lc {

// waves of a workgroup at most: what lets a tile's accumulators and operands in flight stay in registers
constexpr int kForwardWaves(int mt, int nt) { return mt * nt <= 4 ? 16 : 8; }
constexpr int kMostBlocks = 65535;   // blocks of filters: the grid's second dimension

template <int MT, int NT, typename T, bool RAG>
__global__ __launch_bounds__(64 * kForwardWaves(MT, NT)) void lc_forward_general_kernel(
    Geom g, const T *__restrict__ x, const T *__restrict__ w, const float *__restrict__ bias, float alpha,
    const float *__restrict__ alpha_dev, float *__restrict__ y, int NV, int nvt, int per_slice, int nbt, int nfw, int ks,
    int ntask) {
    constexpr int ES = sizeof(T), PF = MT * NT <= 4 ? 4 : 2;   // groups of 16 patch elements in flight
    typedef typename Quad<T>::V XV;
    extern __shared__ __attribute__((aligned(16))) f32x4 slices[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, kk = lane >> 4;
    // waves of a workgroup: slices of the contraction innermost, then blocks of filters, then tasks (field, batch tile)
    const int slice = wave % ks, grp = wave / ks;
    const int tasks = (blockDim.x >> 6) / (ks * nfw);
    const int task = remap_xcd(blockIdx.x, gridDim.x) * tasks + grp / nfw;
    const int f0 = (blockIdx.y * nfw + grp % nfw) * (NT * 16);
    const bool active = task < ntask && f0 < g.F;
    const int tk = min(task, ntask - 1);
    const int loc = tk / nbt, b0 = (tk - loc * nbt) * (16 * MT);
    const int i = loc / g.LW, j = loc - i * g.LW;
    const int WC = g.W * g.C;
    const size_t img = (size_t)g.H * WC;

    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int u = 0; u < NT; ++u) acc[mt][u] = (f32x4){0.f, 0.f, 0.f, 0.f};

    const int fl = min(f0 + NT * n, g.F - NT);                // the lane's first filter
    const gbytes xp = (gbytes)(x + (size_t)b0 * img + (size_t)(i * g.S) * WC + j * g.S * g.C);
    const gbytes wp = (gbytes)(w + (size_t)loc * g.K * g.F);
    const unsigned wstep = (unsigned)g.F * ES;
    unsigned ro[MT];                                          // byte offset of image m + 16 mt
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) ro[mt] = (unsigned)((size_t)min(mt * 16 + n, g.B - 1 - b0) * img) * ES;

    // The lane's vectors are numbers kk, kk+4, .. of its slice; v counts them along a patch row of NV vectors, xo and kr
    // are the row's place in the image and its first patch element.
    const int vbeg = slice * per_slice, vend = min(vbeg + per_slice, nvt);
    const int dv = 4 % NV, dr = 4 / NV, back = RAG ? 4 * NV - g.RC : 0;
    int vi = vbeg + kk, v, xo, kr;
    {
        const int row = vi / NV;
        v = vi - row * NV;
        xo = row * WC;
        kr = row * g.RC;
    }
    XV a[PF][MT];
    Run<T, NT> bw[PF][4];
    int skip[PF];                                             // leading elements of the vector that count as zero
    auto load = [&](int s) {
        const bool in = vi < vend;
        const int sh = RAG && v == NV - 1 ? back : 0;
        const unsigned xoff = in ? (unsigned)(xo + 4 * v - sh) * ES : 0u;
        const unsigned woff = (unsigned)((in ? kr + 4 * v - sh : 0) * g.F + fl) * ES;
        skip[s] = in ? sh : 4;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) a[s][mt] = load_quad<T>(xp, ro[mt] + xoff);
#pragma unroll
        for (int t = 0; t < 4; ++t) bw[s][t].load(wp, woff + t * wstep);
        vi += 4;
        v += dv;
        xo += dr * WC;
        kr += dr * g.RC;
        if (v >= NV) { v -= NV; xo += WC; kr += g.RC; }
    };
    auto multiply = [&](int s, auto masked) {
        constexpr bool MASK = decltype(masked)::value;
        if constexpr (ES == 4) {
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bool z = MASK && t < skip[s];
                float b[NT];
#pragma unroll
                for (int u = 0; u < NT; ++u) b[u] = z ? 0.f : bw[s][t].get(u);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const float av = z ? 0.f : a[s][mt][t];
#pragma unroll
                    for (int u = 0; u < NT; ++u) acc[mt][u] = mfma16(av, b[u], acc[mt][u]);
                }
            }
        } else {
            u32x2 b[NT];
#pragma unroll
            for (int u = 0; u < NT; ++u) {
                b[u] = column4<NT>(bw[s], u);
                if (MASK) b[u] = clear_below(b[u], skip[s]);
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                const u32x2 av = MASK ? clear_below(a[s][mt], skip[s]) : a[s][mt];
#pragma unroll
                for (int u = 0; u < NT; ++u) acc[mt][u] = mfma16_bf16(av, b[u], acc[mt][u]);
            }
        }
    };
    const int nvec = max(vend - vbeg, 0), ng = (nvec + 3) >> 2, nfull = nvec >> 2;
    if (ng > 0 && active) {
#pragma unroll
        for (int s = 0; s < PF; ++s) {
            load(s);
            __builtin_amdgcn_sched_barrier(0);                // (the loop's waits count on this order)
        }
        int done = 0;
        for (; done + PF <= nfull; done += PF) {
#pragma unroll
            for (int s = 0; s < PF; ++s) {
                multiply(s, std::bool_constant<RAG>{});
                load(s);
                // the refill of a slot stays right behind the MFMAs that used it
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int s = 0; s < PF; ++s)
            if (done + s < ng) multiply(s, std::true_type{});
    }
    add_slices<MT * NT>(&acc[0][0], slices, grp, slice, ks);
    if (!active || slice != 0) return;

    if (alpha_dev) alpha = *alpha_dev;
    float bv[NT];
#pragma unroll
    for (int u = 0; u < NT; ++u) bv[u] = bias ? bias[(size_t)loc * g.F + fl + u] : 0.f;
    struct __attribute__((packed, aligned(4))) Out { float v[NT]; };
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int b = b0 + mt * 16 + 4 * kk + r;
            if (b >= g.B) continue;
            Out o;
#pragma unroll
            for (int u = 0; u < NT; ++u) o.v[u] = alpha * acc[mt][u][r] + bv[u];
            *(Out *)(y + ((size_t)b * g.L + loc) * g.F + fl) = o;
        }
}

namespace {

// Host check of a lc_forward_general_kernel launch.  tparam = {MT, NT, filter blocks per workgroup, bytes per operand
// element, RAG, slices of the contraction, tasks per workgroup}; arg = {vectors per patch row, vectors per patch, vectors
// per slice, batch tiles, tasks}.
int check_forward_general(const Geom &g, const LaunchPlan &p) {
    const int MT = p.tparam[0], NT = p.tparam[1], nfw = p.tparam[2], ES = p.tparam[3], RAG = p.tparam[4];
    const int ks = p.tparam[5], tasks = p.tparam[6];
    const int NV = p.arg[0], nvt = p.arg[1], per = p.arg[2], nbt = p.arg[3], ntask = p.arg[4];
    LC_PLAN_REQUIRE(p, MT >= 1 && MT <= 4 && NT >= 1 && NT <= 4 && (ES == 4 || (ES == 2 && NT != 3)));
    LC_PLAN_REQUIRE(p, nfw == 1 || nfw == 2);
    LC_PLAN_REQUIRE(p, (int)p.block <= 64 * kForwardWaves(MT, NT));
    LC_PLAN_REQUIRE(p, ks >= 1 && ks <= 16 && (ks & (ks - 1)) == 0 && tasks >= 1 && (int)p.block == 64 * ks * nfw * tasks);
    // whole vectors inside a patch row and whole runs inside the filters; every vector in one slice, slices in groups
    LC_PLAN_REQUIRE(p, g.RC >= 4 && g.F >= NT && NV == ceil_div(g.RC, 4) && nvt == g.R * NV && RAG == (g.RC % 4 != 0));
    LC_PLAN_REQUIRE(p, per % 4 == 0 && (long long)per * ks >= nvt);
    LC_PLAN_REQUIRE(p, nbt == ceil_div(g.B, 16 * MT) && (long long)ntask == (long long)g.L * nbt);
    LC_PLAN_REQUIRE(p, (long long)p.grid[0] * tasks >= ntask && (long long)(p.grid[0] - 1) * tasks < ntask);
    LC_PLAN_REQUIRE(p, (long long)p.grid[1] * nfw * NT * 16 >= g.F && (long long)(p.grid[1] - 1) * nfw * NT * 16 < g.F &&
                           p.grid[2] == 1);
    LC_PLAN_REQUIRE(p, ks == 1 || p.lds_bytes >= (size_t)nfw * tasks * (ks / 2) * MT * NT * 1024);
    // 32-bit byte offsets: into a batch tile's images, into a field's K x F matrix
    LC_PLAN_REQUIRE(p, (long long)16 * MT * g.H * g.W * g.C * ES < (1LL << 32) && (long long)g.K * g.F * ES < (1LL << 32));
    return LC_OK;
}

template <int MT, int NT, typename T>
int launch_tile(const Geom &g, const T *x, const T *w, const float *bias, float alpha, const float *alpha_dev, float *y,
                const ForwardTile &t, hipStream_t s) {
    const int NV = ceil_div(g.RC, 4), nvt = g.R * NV, per = ceil_div(ceil_div(nvt, 4), t.ks) * 4;
    const int nbt = ceil_div(g.B, 16 * MT), rag = g.RC % 4 != 0;
    const long long ntask = (long long)g.L * nbt;
    const size_t lds = (size_t)t.nfw * t.tasks * (t.ks / 2) * MT * NT * 1024;
    dim3 grid((unsigned)((ntask + t.tasks - 1) / t.tasks), ceil_div(g.F, t.nfw * NT * 16));
    const LaunchPlan plan = make_plan("lc_forward_general", {MT, NT, t.nfw, (int)sizeof(T), rag, t.ks, t.tasks},
                                      {NV, nvt, per, nbt, (int)ntask}, grid, 64 * t.ks * t.nfw * t.tasks, lds);
    if (int rc = check_forward_general(g, plan)) return rc;
    if (rag)
        LC_LAUNCH(plan, "lc_forward launch", (lc_forward_general_kernel<MT, NT, T, true>), s, g, x, w, bias, alpha, alpha_dev,
                  y, NV, nvt, per, nbt, t.nfw, t.ks, (int)ntask);
    else
        LC_LAUNCH(plan, "lc_forward launch", (lc_forward_general_kernel<MT, NT, T, false>), s, g, x, w, bias, alpha, alpha_dev,
                  y, NV, nvt, per, nbt, t.nfw, t.ks, (int)ntask);
    return LC_OK;
}

// The tile and the number of slices by estimated time, in clocks of a SIMD.  A group of 16 patch elements costs a wave its
// MFMAs (128 clocks per tile of 16 x 16 in fp32, 32 in bf16) and its vector loads, which all waves of a compute unit
// queue for (53 clocks each; how many bytes they bring matters less).  What all tasks cost together is spread over the
// chip's 1024 SIMDs; on top of it comes the time one wave needs by itself, which is what slices shorten, and the price
// of adding the slices.  The constants are a fit to 39 layers of the kinds below timed with every tile and every number
// of slices (batches of 2 to 256, 14 to 384 filters, patches of 27 to 16384 elements, both types): the tile picked is on
// average 8 % slower than the fastest one of its layer.
ForwardTile pick_tile(const Geom &g, int es) {
    const int groups = ceil_div(g.R * ceil_div(g.RC, 4), 4);
    ForwardTile best = {1, 1, 1, 1, 1};
    double best_t = 1e300;
    for (int mt = 1; mt <= 4; ++mt) {
        if (mt > 1 && 16 * (mt - 1) >= g.B) break;
        if ((long long)g.L * ceil_div(g.B, 16 * mt) > kMostTasks) continue;
        for (int nt = 1; nt <= 4; ++nt) {
            if (nt > g.F || (nt > 1 && 16 * (nt - 1) >= g.F) || (es == 2 && nt == 3)) continue;
            // bf16: a single tile of filters is 32 bytes of each weight row, a quarter of a cache line (128 images of
            // 52 x 160 x 16, 8 x 8 at stride 4, 48 filters: 102 -> 68 us with two, 96 of 48 x 60 x 16: 42 -> 20; no
            // slower on any of 13 layers.  fp32: between 0.74 and 1.36 times the time)
            if (es == 2 && nt == 1 && g.F > 16) continue;
            if (ceil_div(g.F, 16 * nt) > kMostBlocks) continue;
            const double tasks = (double)g.L * ceil_div(g.B, 16 * mt) * ceil_div(g.F, 16 * nt);
            const double mm = (es == 4 ? 128.0 : 32.0) * mt * nt, flight = mt * nt <= 4 ? 4 : 2;
            for (int ks = 1, lg = 0; ks <= kForwardWaves(mt, nt) && (ks == 1 || 2 * ks <= groups); ks *= 2, ++lg) {
                const double per = ceil_div(groups, ks), add = ks > 1 ? 520.0 * mt * nt + 1640.0 * lg : 0;
                const double busy = tasks * ks * (per * (mm + 53.0 * (mt + 4)) + add) / 1024;
                const double alone = 1.44 * (per * (mm + 375.0 / flight) + 3350.0 * lg);
                if (busy + alone < best_t) {
                    best_t = busy + alone;
                    best = {mt, nt, 1, 1, ks};
                }
            }
        }
    }
    // two blocks of filters of one field share its patch, and the cache lines of the weight rows that their border cuts
    const int room = kForwardWaves(best.mt, best.nt) / best.ks;
    if (g.F > 16 * best.nt && room >= 2) best.nfw = 2;
    while (best.tasks * best.nfw * best.ks < 4) best.tasks *= 2;
    return best;
}

ForwardTile direct_tile(const Geom &g, int es) {
    static thread_local TileMemo<ForwardTile> memo;
    return memo.get(g, es, pick_tile);
}

template <typename T>
int launch_general(const Geom &g, const T *x, const T *w, const float *bias, float alpha, const float *alpha_dev, float *y,
                   hipStream_t s) {
    const ForwardTile t = direct_tile(g, sizeof(T));
    if (forward_turned_takes(g, sizeof(T), t)) return launch_forward_turned(g, x, w, bias, alpha, alpha_dev, y, t, s);
#define LC_TILE(M, N) if (t.mt == M && t.nt == N) return launch_tile<M, N>(g, x, w, bias, alpha, alpha_dev, y, t, s)
    LC_TILE(1, 1); LC_TILE(2, 1); LC_TILE(3, 1); LC_TILE(4, 1);
    LC_TILE(1, 2); LC_TILE(2, 2); LC_TILE(3, 2); LC_TILE(4, 2);
    LC_TILE(1, 4); LC_TILE(2, 4); LC_TILE(3, 4); LC_TILE(4, 4);
    if constexpr (sizeof(T) == 4) { LC_TILE(1, 3); LC_TILE(2, 3); LC_TILE(3, 3); LC_TILE(4, 3); }
#undef LC_TILE
    return LC_EINTERNAL;
}

}  // namespace

bool forward_general_supported(const Geom &g, int es) {
    // the widest tile's blocks of filters fit the grid, and its tasks their numbers: millions of filters and billions of
    // fields leave to the masked kernel
    return g.RC >= 4 && g.F <= 64 * kMostBlocks && (long long)g.L * ceil_div(g.B, 64) <= kMostTasks && (long long)64 * g.H * g.W * g.C * es < (1LL << 32) && (long long)g.K * g.F * es < (1LL << 32);
}

double forward_general_clocks(const Geom &g) { return forward_turned_clocks(g, direct_tile(g, 4)); }

int launch_forward_general_f32(const Geom &g, const float *x, const float *w, const float *bias, float alpha,
                               const float *alpha_dev, float *y, hipStream_t s) {
    return launch_general(g, x, w, bias, alpha, alpha_dev, y, s);
}

int launch_forward_general_bf16(const Geom &g, const void *x, const void *w, const float *bias, float alpha, float *y,
                                hipStream_t s) {
    return launch_general(g, (const bf16_t *)x, (const bf16_t *)w, bias, alpha, nullptr, y, s);
}

}  // namespace lc
