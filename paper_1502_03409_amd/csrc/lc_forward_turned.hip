// lc_forward for any geometry, with operands turned in LDS: the contraction of lc_forward_general.hip, its tasks and its
// vectors, for layers whose patch rows are whole 16-element blocks and for large layers of other rows.
//
// What bounds the direct form on those is the vector cache and the issue slots.  The cache takes a cycle per four
// neighbouring lanes of one line, and a cycle per lane where neighbours read different images, as the MFMA's layout has them
// (64 a load against 16); and an fp32 MFMA holds the vector ALU's multipliers, so that every address or mask instruction
// costs as much beside one as alone.  So here a load gives four neighbouring lanes one image's four vectors and the wave turns
// them in LDS, places cost no vector instruction (kWhole) or one LDS read a group (kTable), and tiles of six blocks and more
// form fp32 products on the bf16 matrix units (mfma_split).
#include <math.h>

#include <type_traits>

#include "lc_general.hpp"

namespace lc {

// waves of a workgroup at most: what lets a tile's accumulators and operands in flight stay in registers
constexpr int kTurnedWaves(int mt, int nt) { return mt * nt <= 2 ? 16 : 8; }
template <typename T>
constexpr bool kTurnedSplit(int mt, int nt) { return sizeof(T) == 4 && mt * nt >= 6; }

// Waves per SIMD that the registers leave room for: a workgroup's, and one more for split tiles of 12 blocks and fewer, which are
// within a few registers of it (100 images of 60 x 61 x 8, 8 x 8 at stride 2, 96 filters, 4 x 3 blocks: 70 us, and 74 with 173
// registers).
template <typename T>
constexpr int kTurnedResident(int mt, int nt) { return kTurnedSplit<T>(mt, nt) && mt * nt <= 12 ? 3 : kTurnedWaves(mt, nt) / 4; }

// Where a wave's vectors are.  kWhole: four lanes' vectors are always 16 neighbouring elements of one patch row (rows of whole
// 16-element blocks), so the place is the wave's.  kTable: the workgroup writes every vector's place into LDS first.
enum { kWhole = 1, kTable = 2 };
constexpr int kMostPlaces = 4096;        // vectors a table holds: 33 KB

constexpr int kPlacesBeyond = 32;        // places read behind the last vector's and never used: five groups and the next one

// Bytes of LDS a wave turns its operands in: MT image tiles of 16 x 16 elements, and 16 rows of up to 32 filters.
template <typename T>
constexpr int turn_bytes(int mt, int nt, bool bl) { return (mt * 256 + (bl ? nt * 320 : 0)) * (int)sizeof(T); }

template <int MT, int NT, typename T, int WALK, bool BL>
__global__ __launch_bounds__(64 * kTurnedWaves(MT, NT), kTurnedResident<T>(MT, NT)) void lc_forward_turned_kernel(
    Geom g, const T *__restrict__ x, const T *__restrict__ w, const float *__restrict__ bias, float alpha,
    const float *__restrict__ alpha_dev, float *__restrict__ y, Divisor dNV, int nvt, int per_slice, Divisor dnbt, Divisor dLW,
    int lnfw, int lks, int ntask) {
    constexpr bool SPLIT = kTurnedSplit<T>(MT, NT);
    constexpr int ES = sizeof(T), GP = SPLIT ? 2 : 1;         // groups of 16 patch elements in a step
    constexpr int PF = SPLIT ? 1 : 4;                         // steps in flight
    constexpr int NB = BL ? NT : 4;                           // loads of a group's weights
    typedef typename Quad<T>::V XV;
    typedef std::conditional_t<BL, XV, Run<T, NT>> BV;
    extern __shared__ __attribute__((aligned(16))) f32x4 slices[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, kk = lane >> 4;
    // waves of a workgroup: slices of the contraction innermost, then blocks of filters, then tasks (field, batch tile)
    const int NV = (int)dNV.d, nbt = (int)dnbt.d, ks = 1 << lks;
    const int slice = wave & (ks - 1), grp = wave >> lks;
    const int ltasks = 31 - __builtin_clz(blockDim.x >> 6) - lks - lnfw;
    const int task = (remap_xcd(blockIdx.x, gridDim.x) << ltasks) + (grp >> lnfw);
    const int f0 = ((blockIdx.y << lnfw) + (grp & ((1 << lnfw) - 1))) * (NT * 16);
    const bool active = task < ntask && f0 < g.F;
    const int tk = min(task, ntask - 1);
    const int loc = dnbt.over(tk), b0 = (tk - loc * nbt) * (16 * MT);
    const int i = dLW.over(loc), j = loc - i * g.LW;
    const int WC = g.W * g.C;
    const size_t img = (size_t)g.H * WC;

    f32x4 acc[MT][NT];
    auto clear = [&] {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int u = 0; u < NT; ++u) acc[mt][u] = (f32x4){0.f, 0.f, 0.f, 0.f};
    };
    clear();

    const int fl = min(f0 + NT * n, g.F - NT);                // the lane's first filter
    // The lane's vectors are numbers kk, kk+4, .. of its slice, NV to a patch row.
    const int vbeg = slice * per_slice, vend = min(vbeg + per_slice, nvt);
    const int nvec = max(vend - vbeg, 0), ng = (nvec + 3) >> 2, nfull = nvec >> 2;
    const int back = WALK == kWhole ? 0 : 4 * NV - g.RC;       // elements a row's last vector shares with the one before it
    uint2 *const places = (uint2 *)((char *)(slices + (size_t)(ks > 1 ? (blockDim.x >> 6) / 2 * MT * NT * 64 : 0)) +
                                    (blockDim.x >> 6) * turn_bytes<T>(MT, NT, BL));
    if constexpr (WALK == kTable) {
        for (int e = threadIdx.x; e < nvt + kPlacesBeyond; e += blockDim.x) {
            const int vi = min(e, nvt - 1), row = dNV.over(vi), v = vi - row * NV, sh = v == NV - 1 ? back : 0;
            places[e] = make_uint2((unsigned)(row * WC + 4 * v - sh) * ES, (unsigned)((row * g.RC + 4 * v - sh) * g.F) * ES);
        }
        __syncthreads();
    }

    if (ng > 0 && active) {
        const gbytes xp = (gbytes)(x + (size_t)b0 * img + (size_t)(i * g.S) * WC + j * g.S * g.C);
        const gbytes wp = (gbytes)(w + (size_t)loc * g.K * g.F);
        const unsigned wstep = (unsigned)g.F * ES;
        // Lane 4m + q loads vector kl = q ^ (m / 4) of image m and writes it to LDS, lane (m,kk) reads it back; neither side
        // meets a bank twice.
        char *turn = (char *)(slices + (size_t)(ks > 1 ? (blockDim.x >> 6) / 2 * MT * NT * 64 : 0)) + wave * turn_bytes<T>(MT, NT, BL);
        const int kl = (lane & 3) ^ (lane >> 4);
        XV *const a_put = (XV *)turn + lane;
        const XV *const a_get = (const XV *)turn + 4 * n + (kk ^ (n >> 2));
        unsigned ro[MT];                                      // byte offset of image lane/4 + 16 mt
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            ro[mt] = (unsigned)((size_t)min(mt * 16 + (lane >> 2), g.B - 1 - b0) * img) * ES;
            if (WALK == kWhole) ro[mt] += 4 * kl * ES;
        }
        // The weights of up to 32 filters go the same way: 16 or 32 filters of a row in 4 or 8 lanes instead of 4 or 8 bytes a
        // lane (one or two loads of 16 rows instead of four).  A vector that would cross the last filter ends there.
        // Rows lie by t, then kk (row 4 kk + t of the group), those of one t a quarter of the banks on.
        const int wq = lane & (BL ? 4 * NT - 1 : 15), wt = BL ? (lane / (4 * NT)) & (4 / NT - 1) : 0;
        char *const wturn = turn + MT * 256 * ES;
        XV *b_put[NB];
        const char *b_get[4];
        unsigned wlane = (unsigned)(WALK == kWhole ? 4 * kk * g.F : 0) * ES;
        if constexpr (BL) {
            wlane += (unsigned)(min(f0 + 4 * wq, g.F - 4) + wt * g.F) * ES;
            const int qr = (fl - f0 + NT - 1) / 4, at = fl - min(f0 + 4 * qr, g.F - 4);   // the vector and element of the lane's run
#pragma unroll
            for (int h = 0; h < NB; ++h) b_put[h] = (XV *)(wturn + ((h * (4 / NT) + wt) * 80 * NT + kk * 16 * NT + 4 * wq) * ES);
#pragma unroll
            for (int t = 0; t < 4; ++t) b_get[t] = wturn + (t * 80 * NT + kk * 16 * NT + 4 * qr + at) * ES;
        } else {
            wlane += (unsigned)fl * ES;
        }
        struct Step {
            XV a[GP][MT];
            BV b[GP][NB];
        };
        // Places of the next group: byte offsets into a batch tile's first image (of vector kl of the group; kWhole: the wave's,
        // number v of its row) and the field's weights (vector kk).  Places beyond the last vector are clamped to it, or belong
        // to the next slice: loaded and never used.
        gbytes wrow[NB];
#pragma unroll
        for (int t = 0; t < NB; ++t) wrow[t] = opaque(wp + t * (BL ? 4 / NT : 1) * wstep);
        int v;
        unsigned xo, wo;
        const uint2 *xe = places + vbeg + kl, *we = places + vbeg + kk;
        const int dv = 4 - dNV.over(4) * NV;
        const int lastv = vbeg + 4 * (ng - 1), lastrow = dNV.over(lastv);   // kWhole: the last group's first vector
        const unsigned xmax = (unsigned)(lastrow * WC + 4 * (lastv - lastrow * NV)) * ES;
        const unsigned wmax = (unsigned)((lastrow * g.RC + 4 * (lastv - lastrow * NV)) * g.F) * ES;
        auto start = [&] {
            if constexpr (WALK == kTable) {
                xe = places + vbeg + kl;
                we = places + vbeg + kk;
                xo = xe->x;
                wo = we->y;
                return;
            }
            const int row = dNV.over(vbeg);
            v = vbeg - row * NV;
            xo = (unsigned)(row * WC + 4 * v) * ES;
            wo = (unsigned)((row * g.RC + 4 * v) * g.F) * ES;
        };
        auto load = [&](Step &s, int h) {
            if constexpr (WALK == kWhole) {
                // (opaque: otherwise the scalar and the lane's part meet in 64-bit vector additions, one a load)
                const gbytes xs = opaque(xp + min(xo, xmax));
                gbytes ws = opaque(wp + min(wo, wmax));
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) s.a[h][mt] = load_quad<T>(xs, opaque(ro[mt]));
#pragma unroll
                for (int t = 0; t < NB; ++t) {
                    if constexpr (BL) s.b[h][t] = load_quad<T>(ws, opaque(wlane));
                    else s.b[h][t].load(ws, opaque(wlane));
                    ws = opaque(ws + (BL ? 4 / NT : 1) * wstep);
                }
            } else {
                const unsigned wl = wlane + wo;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) s.a[h][mt] = load_quad<T>(xp, ro[mt] + xo);
#pragma unroll
                for (int t = 0; t < NB; ++t) {
                    if constexpr (BL) s.b[h][t] = load_quad<T>(wrow[t], wl);
                    else s.b[h][t].load(wrow[t], wl);
                }
            }
            if constexpr (WALK == kTable) {
                xe += 4;
                we += 4;
                xo = xe->x;
                wo = we->y;
            } else {
                v += 4;
                xo += 16 * ES;
                wo += 16 * wstep;
                if (v >= NV) {
                    v = 0;
                    xo += (unsigned)(WC - g.RC) * ES;
                }
            }
        };
        auto load_step = [&](Step &s) {
#pragma unroll
            for (int h = 0; h < GP; ++h) load(s, h);
            // the loads of a step stay behind the MFMAs before them and ahead of those behind them
            __builtin_amdgcn_sched_barrier(0);
        };
        // group h of a step as the MFMAs take it: four elements of each image tile, and a run of filters of four rows
        struct Operands {
            XV a[MT];
            Run<T, NT> b[4];
        };
        auto turned = [&](const Step &s, int h) {
            Operands o;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) a_put[mt * 64] = s.a[h][mt];
            if constexpr (BL) {
#pragma unroll
                for (int q = 0; q < NB; ++q) *b_put[q] = s.b[h][q];
            }
            // the wave's own LDS operations keep their order
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) o.a[mt] = a_get[mt * 64];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if constexpr (BL) __builtin_memcpy(&o.b[t].v, b_get[t], NT * ES);
                else o.b[t] = s.b[h][t];
            }
            __builtin_amdgcn_wave_barrier();
            return o;
        };
        // Elements of group h, number q of the slice, that count as zero, set to it: those of vectors beyond the last one, and
        // what a row's last vector shares with the one before it.
        int ends = 0;                                         // the group's first vector's place in its row
        auto row_end = [&](int p) {                           // (rows of fewer than four vectors end several times in a group)
            p -= NV - 1;
            return p == 0 || (NV < 4 && (p == NV || p == 2 * NV || p == 3 * NV));
        };
        auto next_ends = [&] {
            ends += dv;
            if (ends >= NV) ends -= NV;
        };
        auto blank = [&](Step &s, int h, int q) {
            __builtin_amdgcn_sched_barrier(0);                // (keeps the branches around it from becoming selects)
            const int ix = 4 * q + kl, iw = 4 * q + kk;
            const bool ex = WALK != kWhole && row_end(ends + kl), ew = WALK != kWhole && row_end(ends + kk);
            const int sx = ix < nvec ? (ex ? back : 0) : 4, sw = iw < nvec ? (ew ? back : 0) : 4;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) s.a[h][mt] = clear_below(s.a[h][mt], sx);
#pragma unroll
            for (int t = 0; t < NB; ++t) {
                if constexpr (BL) s.b[h][t] = clear_below(s.b[h][t], t * (4 / NT) + wt < sw ? 4 : 0);
                else s.b[h][t].blank(t < sw);
            }
        };
        // products of a group in MFMAs of its type
        auto plain = [&](const Operands &o) {
            if constexpr (ES == 4) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                        for (int u = 0; u < NT; ++u) acc[mt][u] = mfma16(o.a[mt][t], o.b[t].get(u), acc[mt][u]);
            } else {
                u32x2 b[NT];
#pragma unroll
                for (int u = 0; u < NT; ++u) b[u] = column4<NT>(o.b, u);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int u = 0; u < NT; ++u) acc[mt][u] = mfma16_bf16(o.a[mt], b[u], acc[mt][u]);
            }
        };
        unsigned low = 0;
        auto split_multiply = [&](const Operands &o0, const Operands &o1) {
            if constexpr (SPLIT) {
                Parts pa[MT], pb[NT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const float e[8] = {o0.a[mt][0], o0.a[mt][1], o0.a[mt][2], o0.a[mt][3], o1.a[mt][0], o1.a[mt][1], o1.a[mt][2], o1.a[mt][3]};
                    pa[mt] = split8(e, low);
                }
#pragma unroll
                for (int u = 0; u < NT; ++u) {
                    const float e[8] = {o0.b[0].get(u), o0.b[1].get(u), o0.b[2].get(u), o0.b[3].get(u),
                                        o1.b[0].get(u), o1.b[1].get(u), o1.b[2].get(u), o1.b[3].get(u)};
                    pb[u] = split8(e, low);
                }
                mfma_split(pa, pb, acc);
            }
        };
        Step step[PF];
        const int nst = (ng + GP - 1) / GP, whole = nfull / GP;
        ends = vbeg - dNV.over(vbeg) * NV;
        // step number st made ready for turning
        auto masked = [&](Step &s, int st) {
#pragma unroll
            for (int h = 0; h < GP; ++h) {
                if (st >= whole || (WALK != kWhole && back != 0 && ends + 4 >= NV)) blank(s, h, GP * st + h);
                if constexpr (WALK != kWhole) next_ends();
            }
        };
        start();
#pragma unroll
        for (int s = 0; s < PF; ++s) load_step(step[s]);
        if constexpr (SPLIT) {
            auto contract = [&](auto multiply) {
                for (int st = 0; st < nst; ++st) {
                    masked(step[0], st);
                    const Operands o0 = turned(step[0], 0), o1 = turned(step[0], 1);
                    multiply(o0, o1);
                    load_step(step[0]);
                }
            };
            // a layer that has diverged shows in the first step's operands
            float first = 0.f;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int r = 0; r < 4; ++r) first += step[0].a[0][mt][r] * 0.f;
#pragma unroll
            for (int t = 0; t < NB; ++t)
#pragma unroll
                for (int u = 0; u < (BL ? 4 : NT); ++u) {
                    if constexpr (BL) first += step[0].b[0][t][u] * 0.f;
                    else first += step[0].b[0][t].get(u) * 0.f;
                }
            const bool finite = !__any(first != 0.f);
            if (finite) contract(split_multiply);
            // an operand that is not finite or too small, or a part that overflowed: once more in fp32
            if (!finite || __any(!all_finite<MT * NT>(&acc[0][0]) || inexact(low))) {
                clear();
                start();
                ends = vbeg - dNV.over(vbeg) * NV;
                load_step(step[0]);
                contract([&](const Operands &o0, const Operands &o1) {
                    plain(o0);
                    plain(o1);
                });
            }
        } else {
            // A step is turned while the one before it is multiplied: a lone wave of a SIMD would wait for LDS otherwise.
            Operands o[2];
            masked(step[0], 0);
            o[0] = turned(step[0], 0);
            int done = 0;
            for (; done + PF <= whole; done += PF) {
#pragma unroll
                for (int s = 0; s < PF; ++s) {
                    masked(step[(s + 1) % PF], done + s + 1);
                    o[(s + 1) & 1] = turned(step[(s + 1) % PF], 0);
                    plain(o[s & 1]);
                    load_step(step[s]);
                }
            }
#pragma unroll
            for (int s = 0; s < PF; ++s)
                if (done + s < nst) {
                    if (s + 1 < PF) {
                        masked(step[(s + 1) % PF], done + s + 1);
                        o[(s + 1) & 1] = turned(step[(s + 1) % PF], 0);
                    }
                    plain(o[s & 1]);
                }
        }
    }
    add_slices<MT * NT>(&acc[0][0], slices, grp, slice, ks);
    if (!active || slice != 0) return;

    if (alpha_dev) alpha = *alpha_dev;
    float bv[NT];
#pragma unroll
    for (int u = 0; u < NT; ++u) bv[u] = bias ? bias[(size_t)loc * g.F + fl + u] : 0.f;
    struct __attribute__((packed, aligned(4))) Out { float v[NT]; };
    // Runs that would cross the last filter start earlier, inside the wave's filters as a rule, where the same sums are stored
    // twice.  A last block of fewer filters than a run reaches into the block before: in split tiles those are stored there only, as
    // either wave may have formed its tile in fp32.
    const int first = SPLIT ? max(f0 - (g.F - NT), 0) : 0;
    auto store = [&](auto whole) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int b = b0 + mt * 16 + 4 * kk + r;
                if (b >= g.B) continue;
                Out o;
#pragma unroll
                for (int u = 0; u < NT; ++u) o.v[u] = alpha * acc[mt][u][r] + bv[u];
                float *p = y + ((size_t)b * g.L + loc) * g.F + fl;
                if constexpr (whole()) {
                    *(Out *)p = o;
                } else {
#pragma unroll
                    for (int u = 1; u < NT; ++u)
                        if (u >= first) p[u] = o.v[u];
                }
            }
    };
    if (first == 0) store(std::true_type{});
    else store(std::false_type{});
}

namespace {

// Host check of a lc_forward_turned_kernel launch: parameters and arguments as those of the direct form (lc_forward_general.hip),
// and tparam[7] = form.
int check_forward_turned(const Geom &g, const LaunchPlan &p, bool bl) {
    const int MT = p.tparam[0], NT = p.tparam[1], nfw = p.tparam[2], ES = p.tparam[3], RAG = p.tparam[4];
    const int ks = p.tparam[5], tasks = p.tparam[6], form = p.tparam[7], waves = ks * nfw * tasks;
    const int NV = p.arg[0], nvt = p.arg[1], per = p.arg[2], nbt = p.arg[3], ntask = p.arg[4];
    LC_PLAN_REQUIRE(p, MT >= 1 && MT <= 4 && NT >= 1 && NT <= 4 && (ES == 4 || (ES == 2 && NT != 3)));
    LC_PLAN_REQUIRE(p, (nfw == 1 || nfw == 2) && ks >= 1 && ks <= 16 && (ks & (ks - 1)) == 0 && tasks >= 1 && (tasks & (tasks - 1)) == 0);
    LC_PLAN_REQUIRE(p, (int)p.block == 64 * waves && waves <= kTurnedWaves(MT, NT));
    // whole vectors inside a patch row and whole runs inside the filters; every vector in one slice, slices in groups
    LC_PLAN_REQUIRE(p, g.RC >= 4 && g.F >= NT && (!bl || g.F >= 4) && NV == ceil_div(g.RC, 4) && nvt == g.R * NV && RAG == (g.RC % 4 != 0));
    LC_PLAN_REQUIRE(p, form == kWhole ? g.RC % 16 == 0 : form == kTable && nvt <= kMostPlaces);
    LC_PLAN_REQUIRE(p, per % 4 == 0 && (long long)per * ks >= nvt);
    LC_PLAN_REQUIRE(p, nbt == ceil_div(g.B, 16 * MT) && (long long)ntask == (long long)g.L * nbt);
    LC_PLAN_REQUIRE(p, (long long)p.grid[0] * tasks >= ntask && (long long)(p.grid[0] - 1) * tasks < ntask);
    LC_PLAN_REQUIRE(p, (long long)p.grid[1] * nfw * NT * 16 >= g.F && (long long)(p.grid[1] - 1) * nfw * NT * 16 < g.F &&
                           p.grid[2] == 1);
    // slices, the waves' turning space, places up to the last one read
    const size_t sums = ks > 1 ? (size_t)(waves / 2) * MT * NT * 1024 : 0;
    const size_t turns = (size_t)waves * (ES == 4 ? turn_bytes<float>(MT, NT, bl) : turn_bytes<bf16_t>(MT, NT, bl));
    // (split: an even number of groups, a step of two ahead and the next one's place; otherwise four steps ahead and the next)
    const int groups = ceil_div(nvt, 4) + 1 + (ES == 4 && MT * NT >= 6 ? 3 : 5);
    LC_PLAN_REQUIRE(p, p.lds_bytes >= sums + turns + (form == kTable ? (size_t)4 * groups * 8 : 0));
    LC_PLAN_REQUIRE(p, form != kTable || 4 * groups <= nvt + kPlacesBeyond);
    // 32-bit byte offsets: into a batch tile's images, into a field's K x F matrix
    LC_PLAN_REQUIRE(p, (long long)16 * MT * g.H * g.W * g.C * ES < (1LL << 32) && (long long)g.K * g.F * ES < (1LL << 32));
    return LC_OK;
}

template <int MT, int NT, typename T>
int launch_tile(const Geom &g, const T *x, const T *w, const float *bias, float alpha, const float *alpha_dev, float *y,
                const ForwardTile &t, int form, hipStream_t s) {
    const int NV = ceil_div(g.RC, 4), nvt = g.R * NV, per = ceil_div(ceil_div(nvt, 4), t.ks) * 4;
    const int nbt = ceil_div(g.B, 16 * MT), waves = t.ks * t.nfw * t.tasks;
    const long long ntask = (long long)g.L * nbt;
    const bool bl = NT <= 2;                                  // (turned_form: eight filters at least)
    const size_t lds = (t.ks > 1 ? (size_t)(waves / 2) * MT * NT * 1024 : 0) + (size_t)waves * turn_bytes<T>(MT, NT, bl) +
                       (form == kTable ? (size_t)(nvt + kPlacesBeyond) * 8 : 0);
    dim3 grid((unsigned)((ntask + t.tasks - 1) / t.tasks), ceil_div(g.F, t.nfw * NT * 16));
    const LaunchPlan plan = make_plan("lc_forward_general", {MT, NT, t.nfw, (int)sizeof(T), g.RC % 4 != 0, t.ks, t.tasks, form},
                                      {NV, nvt, per, nbt, (int)ntask}, grid, 64 * waves, lds);
    if (int rc = check_forward_turned(g, plan, bl)) return rc;
#define LC_FORM(W, L)                                                                                                     \
    if (form == W && bl == L) {                                                                                           \
        LC_LAUNCH(plan, "lc_forward launch", (lc_forward_turned_kernel<MT, NT, T, W, L>), s, g, x, w, bias, alpha, alpha_dev, y, \
                  divisor(NV), nvt, per, divisor(nbt), divisor(g.LW), t.nfw - 1, __builtin_ctz(t.ks), (int)ntask);        \
        return LC_OK;                                                                                                     \
    }
    if constexpr (NT <= 2) { LC_FORM(kWhole, true) LC_FORM(kTable, true) }
    if constexpr (NT > 2) { LC_FORM(kWhole, false) LC_FORM(kTable, false) }
#undef LC_FORM
    return LC_EINTERNAL;
}

// 16 images x 16 filters x 16 patch elements, what a layer is measured in below
double blocks_of(const Geom &g) {
    return (double)g.L * ceil_div(g.B, 16) * ceil_div(g.F, 16) * ceil_div(g.R * ceil_div(g.RC, 4), 4);
}

// Which layers: filters in whole 32-byte vectors of fp32, or more than 128 of them, where the tile is picked for this form (below;
// on the direct form's tiles it gains a third of that, and bf16 rows at odd addresses lose: 4 images of 194 x 52 x 2, 19
// filters 1.6 times the time).  Rows of whole 16-element blocks at any size: 106 layers of 6000 to 14 million blocks of 16
// images, filters and elements, 1.18 times as fast as the direct form in fp32 and 1.25 in bf16.  Longer patches of other rows from 100000
// blocks on, where the table pays: 62 layers 1.05 and 1.15; below, the direct form's shorter start wins (32 layers of 600 to
// 40000 blocks 0.95 on its tiles).
int turned_form(const Geom &g) {
    if (g.F % 8 != 0 && g.F <= 128) return 0;
    if (g.RC % 16 == 0) return kWhole;
    const int nvt = g.R * ceil_div(g.RC, 4);
    return blocks_of(g) >= 100000 && nvt >= 64 && nvt <= kMostPlaces ? kTable : 0;
}

// Estimated clocks of a launch.  A group of 16 elements costs a wave its MFMAs (132 clocks a 16 x 16 tile in fp32, 48 where
// fp32 products are split, 17 in bf16), what it costs to split or transpose the operands and to find them, and the vector
// cache its loads; the waves share SIMDs, caches and L2, and none ends before its own chain.  The constants are a fit to 211
// layers timed with every tile and number of slices, in the caches and out of them; what is picked is on average 6 % (fp32)
// and 10 % (bf16) slower than the fastest.
// fullest: every compute unit has as many workgroups as the one with most.
double turned_clocks(const Geom &g, int es, int mt, int nt, int ks, int waves_wg, double wgs,
                    bool fullest) {
    const bool split = es == 4 && mt * nt >= 6, f32 = es == 4;
    const double mm = (split ? 48.0 : f32 ? 132.0 : 17.0) * mt * nt;
    const double form = g.RC % 16 == 0 ? 0.2 : g.RC % 4 != 0 ? 2.0 : 1.0;
    const double issue = mm + (split ? 20.6 : f32 ? 0.0 : 10.3) * 4 * (mt + nt) + (f32 ? 45.6 : 21.2) * form;
    const double per = ceil_div(ceil_div(g.R * ceil_div(g.RC, 4), 4), ks);
    const double add = (ks > 1 ? (f32 ? 308.0 : 270.0) * mt * nt + (f32 ? 176.0 : 91.0) * __builtin_ctz(ks) : 0) + (f32 ? 589.0 : 1085.0);
    const double waves = (fullest ? ceil(wgs / kComputeUnits) * kComputeUnits : wgs) * waves_wg;
    const double busy = waves * (per * issue + add) / 1024, loads = waves * per * (f32 ? 45.5 : 33.2) * mt / 256;
    const double alone = per * (issue + (f32 ? 46.0 : 90.5)) + add;
    const double lines = waves * per * (mt + nt) * 256 * es / ((f32 ? 78.1 : 49.3) * 256);
    // together in the norm of order 3/2: between one after the other and all at once
    const double sum = busy * sqrt(busy) + loads * sqrt(loads) + alone * sqrt(alone) + lines * sqrt(lines);
    return cbrt(sum * sum) + (double)g.L * g.R * g.RC * g.F * es / (f32 ? 3303.0 : 4300.0) + (f32 ? 12800.0 : 11100.0);
}

// Workgroups of a tile: two blocks of filters of one field share its patch; four waves at least.
void arrange(const Geom &g, ForwardTile *t) {
    const int room = kTurnedWaves(t->mt, t->nt) / t->ks;
    t->nfw = g.F > 16 * t->nt && room >= 2 ? 2 : 1;
    t->tasks = 1;
    while (t->tasks * t->nfw * t->ks < 4) t->tasks *= 2;
}

double workgroups_of(const Geom &g, const ForwardTile &t) {
    const double ntask = (double)g.L * ceil_div(g.B, 16 * t.mt);
    return ceil((ntask + t.tasks - 1) / t.tasks) * ceil_div(g.F, t.nfw * t.nt * 16);
}

double turned_clocks(const Geom &g, int es, const ForwardTile &t, bool fullest) {
    return turned_clocks(g, es, t.mt, t.nt, t.ks, t.tasks * t.nfw * t.ks, workgroups_of(g, t), fullest);
}

bool turned_splits(int es, int mt, int nt) { return es == 4 && mt * nt >= 6; }

// The fastest tile by the estimate; the direct form's where it is within a tenth of that (a fifth in bf16,
// where the estimate is further off).  The matrix
// unit rounds a running sum once per instruction (by half a unit in the last place on average), so that a contraction in fewer
// slices ends less precise: tiles that add to the sum that way take at least as many slices as the direct form's.
// first (nullable): a tile to be no less precise than either, in slices and in split products.
ForwardTile fastest_turned(const Geom &g, int es, const ForwardTile &direct, const ForwardTile *first) {
    ForwardTile best = first ? *first : direct;
    const int groups = ceil_div(g.R * ceil_div(g.RC, 4), 4);
    const bool first_splits = first && turned_splits(es, first->mt, first->nt);
    double own = 1e300, best_t = 1e300;
    for (int mt = 1; mt <= 4; ++mt) {
        if (mt > 1 && 16 * (mt - 1) >= g.B) break;
        if ((long long)g.L * ceil_div(g.B, 16 * mt) > kMostTasks) continue;
        for (int nt = 1; nt <= 4; ++nt) {
            if (nt > g.F || (nt > 1 && 16 * (nt - 1) >= g.F) || (es == 2 && nt == 3) || ceil_div(g.F, 16 * nt) > 65535) continue;
            const bool split = turned_splits(es, mt, nt);
            if (first_splits && !split) continue;
            const int least = max(split ? 1 : direct.ks, first && split == first_splits ? first->ks : 1);
            for (int ks = least; ks <= kTurnedWaves(mt, nt) && (ks == least || 2 * ks <= groups); ks *= 2) {
                ForwardTile t = {mt, nt, 1, 1, ks};
                arrange(g, &t);
                const double c = turned_clocks(g, es, t, first != nullptr);
                if (mt == direct.mt && nt == direct.nt && ks == direct.ks) own = c;
                if (c < best_t) {
                    best_t = c;
                    best = t;
                }
            }
        }
    }
    if (own < (es == 4 ? 1.1 : 1.2) * best_t) best = direct;
    best.ks = min(best.ks, kTurnedWaves(best.mt, best.nt));   // (millions of filters: no candidate with as many slices)
    arrange(g, &best);
    return best;
}

// Layers of kFullest blocks and more are as slow as the compute unit with most workgroups: the largest tiles run one or two of
// them a unit, and 265 of those take the time of 512.  Where that makes a tile no less precise 1.15 times as fast, they take it: 80 of
// 371 layers timed in fp32 (1.17 times as fast) and 92 of 336 in bf16 (1.18; 64 images of 28 x 142 x 5, 20 x 20 at stride 8, 223
// filters: 160 workgroups of 86 KB 37 and 25 us, now 256 of 53 KB 22 and 18; 88 x 28 x 5, 16 x 16 at stride 5, 382 filters: 51 -> 40).
// More than a tenth slower than the direct form were 27 and 6 of them, are 9 and 1 (with waits_for_a_round).  Smaller layers are
// what the constants were fitted to.
constexpr double kFullest = 131072;
ForwardTile pick_turned(const Geom &g, int es, const ForwardTile &direct) {
    const ForwardTile t = fastest_turned(g, es, direct, nullptr);
    if (blocks_of(g) < kFullest) return t;
    const ForwardTile u = fastest_turned(g, es, direct, &t);
    return turned_clocks(g, es, t, true) > 1.15 * turned_clocks(g, es, u, true) ? u : t;
}

ForwardTile turned_tile(const Geom &g, int es, const ForwardTile &direct) {
    static thread_local TileMemo<ForwardTile> memo;
    return memo.get(g, es, [&](const Geom &, int) { return pick_turned(g, es, direct); });
}

template <typename T>
int launch(const Geom &g, const T *x, const T *w, const float *bias, float alpha, const float *alpha_dev, float *y,
           const ForwardTile &direct, hipStream_t s) {
    const int form = turned_form(g);
    const ForwardTile t = turned_tile(g, sizeof(T), direct);
#define LC_TILE(M, N) if (t.mt == M && t.nt == N) return launch_tile<M, N>(g, x, w, bias, alpha, alpha_dev, y, t, form, s)
    LC_TILE(1, 1); LC_TILE(2, 1); LC_TILE(3, 1); LC_TILE(4, 1);
    LC_TILE(1, 2); LC_TILE(2, 2); LC_TILE(3, 2); LC_TILE(4, 2);
    LC_TILE(1, 4); LC_TILE(2, 4); LC_TILE(3, 4); LC_TILE(4, 4);
    if constexpr (sizeof(T) == 4) { LC_TILE(1, 3); LC_TILE(2, 3); LC_TILE(3, 3); LC_TILE(4, 3); }
#undef LC_TILE
    return LC_EINTERNAL;
}

}  // namespace

// A compute unit runs one workgroup of sixteen waves.  Where this form needs a little more than a round of them in fp32 and the
// direct form's, of up to four blocks of filters a wave where this one has two, fit in one, the second round is mostly empty: the
// direct form is 1.24 times as fast on 118 layers of 257 to 341 such workgroups (0.95 at least; 16 images of 53 x 22 x 24, 17 x 17 at
// stride 3, 313 filters: 104 -> 53 us), with 360 to 490 of them it is not (0.89 to 1.03 on 6), nor with one block of filters a
// wave (0.75 and 0.86 on 2).
bool waits_for_a_round(const Geom &g, int es, const ForwardTile &direct) {
    if (es != 4) return false;
    const ForwardTile t = turned_tile(g, es, direct);
    const double wgs = workgroups_of(g, t);
    return t.ks * t.nfw * t.tasks == 16 && wgs > kComputeUnits && 3 * wgs <= 4 * kComputeUnits && direct.ks >= t.ks && direct.nt > 1 &&
           workgroups_of(g, direct) <= kComputeUnits;
}

bool forward_turned_takes(const Geom &g, int es, const ForwardTile &direct) {
    return turned_form(g) != 0 && !waits_for_a_round(g, es, direct);
}

double forward_turned_clocks(const Geom &g, const ForwardTile &direct) {
    return turned_clocks(g, 4, turned_tile(g, 4, direct), true);
}

int launch_forward_turned(const Geom &g, const float *x, const float *w, const float *bias, float alpha, const float *alpha_dev,
                          float *y, const ForwardTile &direct, hipStream_t s) {
    return launch(g, x, w, bias, alpha, alpha_dev, y, direct, s);
}
int launch_forward_turned(const Geom &g, const bf16_t *x, const bf16_t *w, const float *bias, float alpha,
                          const float *alpha_dev, float *y, const ForwardTile &direct, hipStream_t s) {
    return launch(g, x, w, bias, alpha, alpha_dev, y, direct, s);
}

}  // namespace lc
