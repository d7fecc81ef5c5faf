// lc_backward_weights for any geometry: out[l,k,f] = beta*out[l,k,f] + gamma * sum_p sum_b patch(x_p)[b,l,k] * dy_p[b,l,f]
// (the weight gradient of Eq. 1; two operand pairs because the tied weights are used twice).
//
// The contraction runs over the batch.  A wave's task is one field, G groups of 16 vectors of four patch elements and
// 16*NT filters; both operands come straight from global memory, four images a step in fp32 (lane kk one of them), sixteen
// on bf16 storage (lane kk four of them, transposed in registers into the operands of the bf16 MFMA).  Lane (m,kk) loads
// vector m of each group and a run of NT filters, so a step is G + 1 vector loads for 4*G*NT MFMAs in fp32.  Patch rows of any
// length are walked in vectors as in the general forward kernel (the last one of a row starts at RC-4), filters in runs that
// end at F-1; what two vectors or two runs share is computed twice and stored by the first.
#include <type_traits>

#include "lc_general.hpp"

namespace lc {

// G = 1: more patch elements per wave, a slice of the batch per wave, and two or eight waves per workgroup all measured the
// same or slower on 33 layers.  With SSQ (partial sums of squares of what is stored) G = 2: their workspace has room for
// one partial per 64 patch elements, and 16 vectors of a short patch row hold fewer.
template <int NT, typename T, bool SSQ>
__global__ __launch_bounds__(256, 2) void lc_bwd_weights_general_kernel(
    Geom g, const T *__restrict__ x1, const T *__restrict__ dy1, const T *__restrict__ x2, const T *__restrict__ dy2,
    float beta, float gamma, float *__restrict__ out, float *__restrict__ ssq, int NV, int nvt, int kblocks, int nfb,
    int ntask) {
    constexpr int G = SSQ ? 2 : 1;
    constexpr int ES = sizeof(T), IM = ES == 4 ? 1 : 4, STEP = 4 * IM;       // images per lane and per step
    constexpr int PF = ES == 4 ? (G * NT <= 4 ? 4 : 2) : (G * NT <= 4 ? 2 : 1);   // steps in flight
    typedef typename Quad<T>::V XV;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, kk = lane >> 4;
    const int task = remap_xcd(blockIdx.x, gridDim.x) * 4 + wave;
    if (task >= ntask) return;
    // Tasks in order of field row, block of patch elements, field of the row, block of filters: waves next to each other
    // read the same image rows (adjacent fields overlap), and the lines of a weight row that the border of two filter blocks
    // cuts are written close together.
    int rest = task;
    const int fb = rest % nfb;
    rest /= nfb;
    const int per_row = g.LW * kblocks, i = rest / per_row;
    rest -= i * per_row;
    const int kb = rest / g.LW, j = rest - kb * g.LW, loc = i * g.LW + j;
    const int f0 = fb * (NT * 16), fl = min(f0 + NT * m, g.F - NT);
    const size_t img = (size_t)g.H * g.W * g.C, dyimg = (size_t)g.L * g.F;
    const int WC = g.W * g.C, back = 4 * NV - g.RC;
    const float inv = 1.0f / (float)NV;

    f32x4 acc[G][4][NT];
#pragma unroll
    for (int gg = 0; gg < G; ++gg)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int u = 0; u < NT; ++u) acc[gg][t][u] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // byte offsets of the lane's vectors and run inside its first image of a step
    unsigned xo[G];
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
        const int vi = min((kb * G + gg) * 16 + m, nvt - 1);
        const int row = (int)(((float)vi + 0.5f) * inv), v = vi - row * NV;
        xo[gg] = (unsigned)((size_t)(IM * kk) * img + row * WC + 4 * v - (v == NV - 1 ? back : 0)) * ES;
    }
    const unsigned fo = (unsigned)((size_t)(IM * kk) * dyimg + fl) * ES;

    const int nstep = (g.B + STEP - 1) / STEP, full = g.B / STEP;   // steps, and those whose images are all there
    for (int p = 0; p < 2; ++p) {
        const T *x = p ? x2 : x1;
        const T *dy = p ? dy2 : dy1;
        if (!x) break;
        const T *xbase = x + (size_t)(i * g.S) * WC + j * g.S * g.C, *ybase = dy + (size_t)loc * g.F;
        XV a[PF][G][IM];
        Run<T, NT> b[PF][IM];
        // A step whose images are not all there loads its own first image instead of the missing ones; they are left out
        // of the products.
        auto load = [&](int s, int st) {
            const int sc = min(st, nstep - 1), left = g.B - (sc * STEP + IM * kk);   // the lane's images from here on
            const gbytes xp = (gbytes)(xbase + (size_t)(sc * STEP) * img), yp = (gbytes)(ybase + (size_t)(sc * STEP) * dyimg);
#pragma unroll
            for (int q = 0; q < IM; ++q) {
                const bool in = q < left;
                const unsigned xq = in ? (unsigned)((size_t)q * img) * ES : 0u - (unsigned)((size_t)(IM * kk) * img) * ES;
                const unsigned yq = in ? (unsigned)((size_t)q * dyimg) * ES : 0u - (unsigned)((size_t)(IM * kk) * dyimg) * ES;
#pragma unroll
                for (int gg = 0; gg < G; ++gg) a[s][gg][q] = load_quad<T>(xp, xo[gg] + xq);
                b[s][q].load(yp, fo + yq);
            }
        };
        auto multiply = [&](int s, int st, auto masked) {
            constexpr bool M = decltype(masked)::value;
            const int left = M ? g.B - (st * STEP + IM * kk) : IM;
            if constexpr (ES == 4) {
                const bool z = M && left <= 0;
#pragma unroll
                for (int gg = 0; gg < G; ++gg)
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const float av = z ? 0.f : a[s][gg][0][t];
#pragma unroll
                        for (int u = 0; u < NT; ++u)
                            acc[gg][t][u] = mfma16(av, z ? 0.f : b[s][0].get(u), acc[gg][t][u]);
                    }
            } else {
                // four images of one vector are the rows of a 4 x 4 block whose columns are the operands
                const unsigned keep_lo = !M || left >= 2 ? 0xffffffffu : left == 1 ? 0xffffu : 0u;
                const unsigned keep_hi = !M || left >= 4 ? 0xffffffffu : left == 3 ? 0xffffu : 0u;
                u32x2 bv[NT];
#pragma unroll
                for (int u = 0; u < NT; ++u) {
                    bv[u] = column4<NT>(b[s], u);
                    if (M) bv[u] = (u32x2){bv[u][0] & keep_lo, bv[u][1] & keep_hi};
                }
#pragma unroll
                for (int gg = 0; gg < G; ++gg) {
                    Run<T, 4> rows[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) rows[q].v = a[s][gg][q % IM];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        u32x2 av = column4<4>(rows, t);
                        if (M) av = (u32x2){av[0] & keep_lo, av[1] & keep_hi};
#pragma unroll
                        for (int u = 0; u < NT; ++u) acc[gg][t][u] = mfma16_bf16(av, bv[u], acc[gg][t][u]);
                    }
                }
            }
        };
#pragma unroll
        for (int s = 0; s < PF; ++s) {
            load(s, s);
            __builtin_amdgcn_sched_barrier(0);
        }
        int st = 0;
        for (; st + PF <= full; st += PF) {
#pragma unroll
            for (int s = 0; s < PF; ++s) {
                multiply(s, st + s, std::false_type{});
                load(s, st + PF + s);
                // the refill of a slot stays right behind the MFMAs that used it
                __builtin_amdgcn_sched_barrier(0);
            }
        }
#pragma unroll
        for (int s = 0; s < PF; ++s)
            if (st + s < nstep) multiply(s, st + s, std::true_type{});
    }

    // what this lane's run shares with the one before it is that one's to store
    const int shared = f0 + NT * m - fl;                       // 0 for all but the last runs; NT or more: nothing to store
    float *ol = out + (size_t)loc * g.K * g.F + fl;
    struct __attribute__((packed, aligned(4))) Row { float v[NT]; };
    float sq[NT];
#pragma unroll
    for (int u = 0; u < NT; ++u) sq[u] = 0.f;
#pragma unroll
    for (int gg = 0; gg < G; ++gg)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int vi = (kb * G + gg) * 16 + 4 * kk + r;
            if (vi >= nvt || shared >= NT) continue;
            const int row = (int)(((float)vi + 0.5f) * inv), v = vi - row * NV;
            const int skip = v == NV - 1 ? back : 0;
            float *o = ol + (size_t)(row * g.RC + 4 * v - skip) * g.F;
            Row old[4];
            if (beta != 0.f) {
#pragma unroll
                for (int t = 0; t < 4; ++t) old[t] = *(const Row *)(o + (size_t)t * g.F);
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (t < skip) continue;
                Row n;
#pragma unroll
                for (int u = 0; u < NT; ++u) {
                    n.v[u] = gamma * acc[gg][t][u][r];
                    if (beta != 0.f) n.v[u] += beta * old[t].v[u];
                }
                if (shared == 0) {
                    *(Row *)(o + (size_t)t * g.F) = n;
                } else {
#pragma unroll
                    for (int u = 0; u < NT; ++u)
                        if (u >= shared) o[(size_t)t * g.F + u] = n.v[u];
                }
                if (SSQ) {
#pragma unroll
                    for (int u = 0; u < NT; ++u)
                        if (u >= shared) sq[u] += n.v[u] * n.v[u];
                }
            }
        }
    // per-filter sums of squares of the rows this wave stored: partial [location][k block][filter]
    if (SSQ) {
#pragma unroll
        for (int u = 0; u < NT; ++u) {
            float t = sq[u];
            t += __shfl_xor(t, 16, 64);
            t += __shfl_xor(t, 32, 64);
            if (kk == 0 && u >= shared) ssq[((size_t)loc * kblocks + kb) * g.F + fl + u] = t;
        }
    }
}

namespace {

// Host check of a lc_bwd_weights_general_kernel launch.  tparam = {G, NT, bytes per operand element}; arg = {vectors per patch row, vectors per patch, blocks of 16*G vectors, filter blocks, tasks}.
int check_backward_weights_general(const Geom &g, const LaunchPlan &p) {
    const int G = p.tparam[0], NT = p.tparam[1], ES = p.tparam[2];
    const int NV = p.arg[0], nvt = p.arg[1], kblocks = p.arg[2], nfb = p.arg[3], ntask = p.arg[4];
    LC_PLAN_REQUIRE(p, (G == 1 || G == 2) && NT >= 1 && NT <= 4 && (ES == 4 || (ES == 2 && NT != 3)));
    // whole vectors inside a patch row, whole runs inside the filters; the division by NV in fp32
    LC_PLAN_REQUIRE(p, g.RC >= 4 && g.F >= NT && NV == ceil_div(g.RC, 4) && nvt == g.R * NV && nvt < (1 << 20));
    LC_PLAN_REQUIRE(p, kblocks == ceil_div(nvt, 16 * G) && nfb == ceil_div(g.F, 16 * NT));
    LC_PLAN_REQUIRE(p, (long long)ntask == (long long)g.L * kblocks * nfb && p.block == 256 && p.grid[1] == 1 &&
                           p.grid[2] == 1);
    LC_PLAN_REQUIRE(p, (long long)p.grid[0] * 4 >= ntask && (long long)(p.grid[0] - 1) * 4 < ntask);
    // 32-bit byte offsets inside the images of a step
    LC_PLAN_REQUIRE(p, (long long)(ES == 4 ? 4 : 16) * g.H * g.W * g.C * ES < (1LL << 32) &&
                           (long long)(ES == 4 ? 4 : 16) * g.L * g.F * ES < (1LL << 32));
    return LC_OK;
}

template <int NT, typename T, bool SSQ>
int launch_tile(const Geom &g, const T *x1, const T *dy1, const T *x2, const T *dy2, float beta, float gamma, float *out,
                float *ssq, int *kblocks_out, hipStream_t s) {
    constexpr int G = SSQ ? 2 : 1;
    const int NV = ceil_div(g.RC, 4), nvt = g.R * NV, kblocks = ceil_div(nvt, 16 * G), nfb = ceil_div(g.F, 16 * NT);
    const long long ntask = (long long)g.L * kblocks * nfb;
    const LaunchPlan plan = make_plan("lc_bwd_weights_general", {G, NT, (int)sizeof(T)}, {NV, nvt, kblocks, nfb, (int)ntask},
                                      dim3((unsigned)((ntask + 3) / 4)), 256, 0);
    if (int rc = check_backward_weights_general(g, plan)) return rc;
    if (kblocks_out) *kblocks_out = kblocks;
    LC_LAUNCH(plan, "lc_backward_weights launch", (lc_bwd_weights_general_kernel<NT, T, SSQ>), s, g, x1, dy1, x2, dy2, beta,
              gamma, out, ssq, NV, nvt, kblocks, nfb, (int)ntask);
    return LC_OK;
}

// Filters per wave by estimated time: per step the MFMAs of four patch elements (128 clocks per tile of 16 filters) and the
// loads, and once the stores, which cost wide tiles more (fewer waves fit a compute unit).  A fit to 33 layers timed with
// every tile (batches of 2 to 256, 16 to 230 filters, both types); what is picked is on average 1 % slower than the fastest.
int pick_filter_tiles(const Geom &g, int es) {
    const double steps = ceil_div(g.B, es == 4 ? 4 : 16), loads = es == 4 ? 96 : 711;
    int best = 1;
    double best_t = 1e300;
    for (int nt = 1; nt <= 4; ++nt) {
        if (nt > g.F || (nt > 1 && 16 * (nt - 1) >= g.F) || (es == 2 && nt == 3)) continue;
        const double t = ceil_div(g.F, 16 * nt) * (steps * (128.0 * nt + loads) + 174 + 653.0 * nt + 510.0 * nt * nt);
        if (t < best_t) { best_t = t; best = nt; }
    }
    return best;
}

template <typename T>
int launch_general(const Geom &g, const T *x1, const T *dy1, const T *x2, const T *dy2, float beta, float gamma, float *out,
                   float *ssq, int *kblocks_out, hipStream_t s) {
    const int nt = pick_filter_tiles(g, sizeof(T));
#define LC_TILE(N)                                                                                                        \
    if (nt == N) {                                                                                                        \
        if constexpr (sizeof(T) == 4) {                                                                                   \
            if (ssq) return launch_tile<N, T, true>(g, x1, dy1, x2, dy2, beta, gamma, out, ssq, kblocks_out, s);          \
        }                                                                                                                 \
        return launch_tile<N, T, false>(g, x1, dy1, x2, dy2, beta, gamma, out, ssq, kblocks_out, s);                      \
    }
    LC_TILE(1) LC_TILE(2) LC_TILE(4)
    if constexpr (sizeof(T) == 4) { LC_TILE(3) }
#undef LC_TILE
    return LC_EINTERNAL;
}

}  // namespace

bool backward_weights_general_supported(const Geom &g, int es) {
    const long long images = es == 4 ? 4 : 16, nvt = (long long)g.R * ceil_div(g.RC, 4);
    // (in blocks of 16 filters, the most tasks there can be: gradients of terabytes leave to the masked kernel)
    return g.RC >= 4 && nvt < (1 << 20) && (long long)g.L * ((nvt + 15) / 16) <= kMostTasks / ceil_div(g.F, 16) && images * g.H * g.W * g.C * es < (1LL << 32) &&
           images * g.L * g.F * es < (1LL << 32);
}

int launch_backward_weights_general_f32(const Geom &g, const float *x1, const float *dy1, const float *x2, const float *dy2,
                                        float beta, float gamma, float *out, float *ssq, int *kblocks_out, hipStream_t s) {
    return launch_general(g, x1, dy1, x2, dy2, beta, gamma, out, ssq, kblocks_out, s);
}

int launch_backward_weights_general_bf16(const Geom &g, const void *x, const void *dy, float beta, float *dw, hipStream_t s) {
    const bf16_t *none = nullptr;
    return launch_general(g, (const bf16_t *)x, (const bf16_t *)dy, none, none, beta, 1.f, dw, nullptr, nullptr, s);
}

}  // namespace lc
