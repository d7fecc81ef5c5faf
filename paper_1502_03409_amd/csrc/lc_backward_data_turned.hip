// lc_backward_data with operands turned in LDS: the contraction of lc_backward_data_general.hip, its pixel blocks and its
// tasks, for layers whose filters fill groups of 16 (fp32) or 32 (bf16).
//
// What bounds the direct form is the vector cache, which takes a cycle per four neighbouring lanes of one line and a cycle per
// lane where neighbours read different rows: the MFMA's layout has sixteen images, or sixteen values' weight rows, in
// neighbouring lanes, 64 cycles a load for both operands.  Here a load gives four neighbouring lanes 64 bytes of one row, and
// the wave turns them in LDS.  A group of filters lies in one field, so that the field is the wave's: its place costs no
// vector instruction where it covers the whole pixel block (an fp32 MFMA holds the vector ALU's multipliers: every such
// instruction costs as much beside one as alone), a few where it covers a part of it.  Tiles of three blocks and more form fp32
// products on the bf16 matrix units (mfma_split).
#include <math.h>

#include <type_traits>

#include "lc_general.hpp"

namespace lc {

constexpr int kTurnedDataWaves = 8;   // per workgroup at most
template <typename T>
constexpr bool kTurnedDataSplit(int mt, int nt) { return sizeof(T) == 4 && mt * nt >= 3; }

// 16 bytes of a row: four fp32 or eight bf16 filters
template <typename T> struct Piece;
template <> struct Piece<float> { typedef f32x4 V; };
template <> struct Piece<bf16_t> { typedef u32x4 V; };
template <typename T>
__device__ __forceinline__ typename Piece<T>::V load_piece(gbytes base, unsigned off) {
    typedef __attribute__((address_space(1), aligned(sizeof(T)))) typename Piece<T>::V GV;
    return *(const GV *)(base + off);
}
__device__ __forceinline__ f32x4 product(f32x4 a, f32x4 b, f32x4 acc) {
#pragma unroll
    for (int t = 0; t < 4; ++t) acc = mfma16(a[t], b[t], acc);
    return acc;
}
__device__ __forceinline__ f32x4 product(u32x4 a, u32x4 b, f32x4 acc) { return mfma32_bf16(a, b, acc); }

template <int MT, int NT, typename T, bool MASK>
__global__ __launch_bounds__(64 * kTurnedDataWaves) void lc_bwd_data_turned_kernel(
    Geom g, const T *__restrict__ dy, const T *__restrict__ w, float *__restrict__ dx, int PR, int PC, Divisor dcbc, Divisor dnbt,
    Divisor dPCC, Divisor dC, Divisor dS, Divisor dFG, int lks, int ntask) {
    typedef typename Piece<T>::V PV;
    constexpr bool SPLIT = kTurnedDataSplit<T>(MT, NT);
    constexpr int ES = sizeof(T), V = 16 / ES, GW = 4 * V;    // filters a lane and a group
    constexpr int GP = SPLIT ? 2 : 1, PF = SPLIT ? 1 : 4;     // groups of a step, steps in flight
    extern __shared__ __attribute__((aligned(16))) f32x4 slices[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int m = lane & 15, kk = lane >> 4;
    // waves of a workgroup: slices of the contraction innermost, then tasks (pixel block, batch tile)
    const int ks = 1 << lks, slice = wave & (ks - 1), grp = wave >> lks;
    const int ltasks = 31 - __builtin_clz(blockDim.x >> 6) - lks;
    const int task = (remap_xcd(blockIdx.x, gridDim.x) << ltasks) + grp;
    const int n0 = blockIdx.y * (NT * 16), N = PR * PC * g.C, PCC = PC * g.C;
    const bool active = task < ntask;
    const int tk = min(task, ntask - 1);
    const int blk = dnbt.over(tk), b0 = (tk - blk * (int)dnbt.d) * (16 * MT);
    const int rb = dcbc.over(blk), r0 = rb * PR, c0 = (blk - rb * (int)dcbc.d) * PC;
    // the fields that touch the block
    const int i_lo = dS.over(max(0, r0 - g.R + g.S)), i_hi = min(g.LH - 1, dS.over(r0 + PR - 1));
    const int j_lo = dS.over(max(0, c0 - g.R + g.S)), j_hi = min(g.LW - 1, dS.over(c0 + PC - 1));
    const int na = i_hi - i_lo + 1, nap = j_hi - j_lo + 1, FG = (int)dFG.d;
    const int ngt = na > 0 && nap > 0 ? na * nap * FG : 0;    // groups of the block
    const int per = (ngt + ks - 1) >> lks, qbeg = slice * per, ng = max(min(per, ngt - qbeg), 0);
    const size_t dyimg = (size_t)g.L * g.F, first = (size_t)i_lo * g.LW + j_lo;

    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};

    if (ng > 0 && active) {
        const gbytes yp = (gbytes)(dy + (size_t)b0 * dyimg + first * g.F);
        const gbytes wp = (gbytes)(w + first * g.K * g.F);
        // Lane 4r + q loads piece kl = q ^ (r / 4) of row r (an image, or a value's weight row) and writes it to LDS, lane (r,kk)
        // reads it back; neither side meets a bank twice.
        PV *const turn = (PV *)(slices + (size_t)(ks > 1 ? (blockDim.x >> 7) * MT * NT * 64 : 0)) + wave * (MT + NT) * 64;
        const int row = lane >> 2, kl = (lane & 3) ^ (lane >> 4);
        PV *const put = turn + lane;
        const PV *const get = turn + 4 * m + (kk ^ (m >> 2));
        unsigned la[MT], lb[NT];                              // byte offsets of the lane's rows and piece
        int rr[NT], cc[NT];                                   // places of its values relative to field (i_lo, j_lo)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            la[mt] = (unsigned)((size_t)min(mt * 16 + row, g.B - 1 - b0) * dyimg + V * kl) * ES;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const int v = n0 + nt * 16 + row, vc = v < N ? v : 0;
            const int dr = dPCC.over(vc), rem = vc - dr * PCC, dc = dC.over(rem);
            rr[nt] = r0 + dr - i_lo * g.S;
            cc[nt] = c0 + dc - j_lo * g.S;
            lb[nt] = (unsigned)((rr[nt] * g.RC + cc[nt] * g.C + (rem - dc * g.C)) * g.F + V * kl) * ES;
        }
        // the last group of a field may be partly filled: its pieces end at the last filter, and what they share with others is
        // zero
        const int over = max(0, GW * (FG - 1) + V * kl - (g.F - V)), skip = min(over, V);
        const bool parted = MASK && g.F % GW != 0;
        const int arow = g.LW * g.K - g.S * g.RC, acol = g.K - g.S * g.C;
        struct Step {
            PV a[GP][MT], b[GP][NT];
            unsigned long long bad[GP][NT];                   // lanes whose value lies outside the field
            bool part[GP], tail[GP];
        };
        int fa, fp, fg, left;                                 // field of the next group, its number there, groups left
        auto start = [&] {
            const int fi = dFG.over(qbeg);
            fg = qbeg - fi * FG;
            fa = __builtin_amdgcn_readfirstlane((int)(((float)fi + 0.5f) * (1.0f / (float)nap)));
            fp = fi - fa * nap;
            left = ng;
        };
        auto load = [&](Step &s, int h) {
            const unsigned aoff = (unsigned)((fa * g.LW + fp) * g.F + GW * fg) * ES;
            const int boff = (fa * arow + fp * acol) * g.F + GW * fg;
            if constexpr (MASK) {
                const bool tail = parted && fg == FG - 1;
                // a field that contains the whole block contains its first and last pixel
                const int ra = fa * g.S, ca = fp * g.S, rf = r0 - i_lo * g.S - ra, cf = c0 - j_lo * g.S - ca;
                const bool part = rf < 0 || rf + PR > g.R || cf < 0 || cf + PC > g.R;
                s.tail[h] = tail;
                s.part[h] = part;
                const unsigned back = tail ? (unsigned)over * ES : 0u;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) s.a[h][mt] = load_piece<T>(yp, aoff + la[mt] - back);   // (together: never below 0)
                unsigned off[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    off[nt] = (unsigned)boff * ES + lb[nt] - back;
                    s.bad[h][nt] = 0;
                }
                if (part) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        const bool ok = ((unsigned)(rr[nt] - ra) < (unsigned)g.R) & ((unsigned)(cc[nt] - ca) < (unsigned)g.R);
                        off[nt] = ok ? off[nt] : 0u;
                        s.bad[h][nt] = __ballot(!ok);
                    }
                }
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) s.b[h][nt] = load_piece<T>(wp, off[nt]);
            } else {
                const gbytes ya = opaque(yp + aoff), wa = opaque(wp + (long long)boff * ES);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) s.a[h][mt] = load_piece<T>(ya, opaque(la[mt]));
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) s.b[h][nt] = load_piece<T>(wa, opaque(lb[nt]));
            }
            // (the last group is loaded again where there is none behind it, and never used)
            if (--left > 0 && ++fg == FG) {
                fg = 0;
                if (++fp == nap) {
                    fp = 0;
                    ++fa;
                }
            }
        };
        auto load_step = [&](Step &s) {
#pragma unroll
            for (int h = 0; h < GP; ++h) load(s, h);
            // the loads of a step stay behind the MFMAs before them and ahead of those behind them
            __builtin_amdgcn_sched_barrier(0);
        };
        struct Operands { PV a[MT], b[NT]; };
        // Group h of a step, as the MFMAs take it; values outside the field and what a field's last pieces share count as zero.
        auto turned = [&](Step &s, int h) {
            if constexpr (MASK) {
                if (s.part[h]) {
                    __builtin_amdgcn_sched_barrier(0);        // (keeps the branch from becoming selects)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) s.b[h][nt] = (s.bad[h][nt] >> lane) & 1 ? PV{} : s.b[h][nt];
                }
                if (s.tail[h]) {
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) s.a[h][mt] = clear_below(s.a[h][mt], skip);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) s.b[h][nt] = clear_below(s.b[h][nt], skip);
                }
            }
            Operands o;
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) put[mt * 64] = s.a[h][mt];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) put[(MT + nt) * 64] = s.b[h][nt];
            // the wave's own LDS operations keep their order
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) o.a[mt] = get[mt * 64];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) o.b[nt] = get[(MT + nt) * 64];
            __builtin_amdgcn_wave_barrier();
            return o;
        };
        auto plain = [&](const Operands &o) {
            if constexpr (ES == 4) {
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = mfma16(o.a[mt][t], o.b[nt][t], acc[mt][nt]);
            } else {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = mfma32_bf16(o.a[mt], o.b[nt], acc[mt][nt]);
            }
        };
        Step step[PF];
        start();
#pragma unroll
        for (int s = 0; s < PF; ++s) load_step(step[s]);
        if constexpr (SPLIT) {
            unsigned low = 0;
            auto contract = [&](auto multiply) {
                for (int q = 0; q < ng; q += 2) {
                    const Operands o0 = turned(step[0], 0);
                    Operands o1 = turned(step[0], 1);
                    if (q + 1 == ng) {                        // no second group: nothing is added
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt) o1.a[mt] = PV{};
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) o1.b[nt] = PV{};
                    }
                    multiply(o0, o1);
                }
            };
            // a layer that has diverged shows in the first group's operands
            float first = 0.f;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) first += step[0].a[0][mt][r] * 0.f;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) first += step[0].b[0][nt][r] * 0.f;
            }
            const bool finite = !__any(first != 0.f);
            if (finite) contract([&](const Operands &o0, const Operands &o1) {
                load_step(step[0]);                           // (ahead of the split, which runs beside the products then)
                Parts pa[MT], pb[NT];
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const float e[8] = {o0.a[mt][0], o0.a[mt][1], o0.a[mt][2], o0.a[mt][3], o1.a[mt][0], o1.a[mt][1], o1.a[mt][2], o1.a[mt][3]};
                    pa[mt] = split8(e, low);
                }
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const float e[8] = {o0.b[nt][0], o0.b[nt][1], o0.b[nt][2], o0.b[nt][3], o1.b[nt][0], o1.b[nt][1], o1.b[nt][2], o1.b[nt][3]};
                    pb[nt] = split8(e, low);
                }
                mfma_split(pa, pb, acc);
            });
            // an operand that is not finite or too small, or a part that overflowed: once more in fp32
            if (!finite || __any(!all_finite<MT * NT>(&acc[0][0]) || inexact(low))) {
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = (f32x4){0.f, 0.f, 0.f, 0.f};
                start();
                load_step(step[0]);
                contract([&](const Operands &o0, const Operands &o1) {
                    load_step(step[0]);
                    plain(o0);
                    plain(o1);
                });
            }
        } else {
            // A group is turned while the one before it is multiplied: a lone wave of a SIMD would wait for LDS otherwise.
            Operands o[2];
            o[0] = turned(step[0], 0);
            int done = 0;
            for (; done + PF <= ng; done += PF) {
#pragma unroll
                for (int s = 0; s < PF; ++s) {
                    o[(s + 1) & 1] = turned(step[(s + 1) % PF], 0);
                    plain(o[s & 1]);
                    load_step(step[s]);
                }
            }
#pragma unroll
            for (int s = 0; s < PF; ++s)
                if (done + s < ng) {
                    if (s + 1 < PF) o[(s + 1) & 1] = turned(step[(s + 1) % PF], 0);
                    plain(o[s & 1]);
                }
        }
    }
    add_slices<MT * NT>(&acc[0][0], slices, grp, slice, ks);
    if (!active || slice != 0) return;

    unsigned again = 0;                                       // bit mt*NT + nt: the tile holds a NaN
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int v = n0 + nt * 16 + m, vc = v < N ? v : 0, dr = dPCC.over(vc), rem = vc - dr * PCC;
        const int col = c0 + dC.over(rem);
        const bool stored = v < N && r0 + dr < g.H && col < g.W;
        float *o = dx + ((size_t)(r0 + dr) * g.W + c0) * g.C + rem;
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
    // The zero weights of a value outside a field make a NaN of an infinite or NaN dy of that field: such a tile is formed
    // again field by field, each field's part added only to the values it contains.  Where the fields tile the cells there are
    // no such weights.
    if constexpr (MASK) {
        if (again == 0 || (PR == g.S && PC == g.S && g.R % g.S == 0)) return;
        const int NVF = (g.F + V - 1) / V, last = V * NVF - g.F;
        while (again) {
            const int tile = __ffs(again) - 1, mt = tile / NT, nt = tile - mt * NT;
            again &= again - 1;
            const int v = n0 + nt * 16 + m, vc = v < N ? v : 0;
            const int dr = dPCC.over(vc), rem = vc - dr * PCC, dc = dC.over(rem);
            const int r1 = r0 + dr - i_lo * g.S, c1 = c0 + dc - j_lo * g.S;
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
                for (int f0 = 0; f0 < NVF; f0 += 4) {
                    const int fv = f0 + kk;
                    const bool in = fv < NVF;
                    const int sh = fv == NVF - 1 ? last : 0, skip = in ? sh : V;
                    const unsigned fo = (unsigned)(in ? V * fv - sh : 0) * ES;
                    const PV a = clear_below(load_piece<T>(yp, aoff + fo), skip);
                    const PV b = clear_below(load_piece<T>(wp, ok ? boff + fo : 0u), skip);
                    part = product(a, b, part);
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

// Host check of a lc_bwd_data_turned_kernel launch: parameters and arguments as those of the direct form
// (lc_backward_data_general.hip), and tparam[7] = 1.
int check_backward_data_turned(const Geom &g, const LaunchPlan &p, bool mask, int FG) {
    const int MT = p.tparam[0], NT = p.tparam[1], ES = p.tparam[2], ks = p.tparam[4], tasks = p.tparam[5];
    const int PR = p.arg[0], PC = p.arg[1], cbc = p.arg[2], nbt = p.arg[4], ntask = p.arg[5], V = 16 / ES;
    LC_PLAN_REQUIRE(p, MT >= 1 && MT <= 4 && NT >= 1 && NT <= 4 && (ES == 4 || ES == 2));
    LC_PLAN_REQUIRE(p, ks >= 1 && (ks & (ks - 1)) == 0 && tasks >= 1 && (tasks & (tasks - 1)) == 0);
    LC_PLAN_REQUIRE(p, (int)p.block == 64 * ks * tasks && (int)p.block <= 64 * kTurnedDataWaves);
    LC_PLAN_REQUIRE(p, PR >= g.S && PR % g.S == 0 && PC >= g.S && PC % g.S == 0 && cbc == ceil_div(g.W, PC));
    // no masks: every field of a block's rectangle covers all of the block, filters in whole groups
    LC_PLAN_REQUIRE(p, mask || (PR == g.S && PC == g.S && g.R % g.S == 0 && g.F % (4 * V) == 0));
    LC_PLAN_REQUIRE(p, g.F >= V && FG == ceil_div(g.F, 4 * V) && nbt == ceil_div(g.B, 16 * MT));
    const long long blocks = (long long)ceil_div(g.H, PR) * cbc, N = (long long)PR * PC * g.C;
    LC_PLAN_REQUIRE(p, (long long)ntask == blocks * nbt && N < (1LL << 31));
    LC_PLAN_REQUIRE(p, (long long)p.grid[0] * tasks >= ntask && (long long)(p.grid[0] - 1) * tasks < ntask);
    LC_PLAN_REQUIRE(p, (long long)p.grid[1] * NT * 16 >= N && (long long)(p.grid[1] - 1) * NT * 16 < N && p.grid[2] == 1);
    LC_PLAN_REQUIRE(p, p.lds_bytes >= (ks > 1 ? (size_t)(ks * tasks / 2) * MT * NT * 1024 : 0) + (size_t)ks * tasks * (MT + NT) * 1024);
    // the division of a field's number in fp32; 32-bit byte offsets: into a batch tile's dy, from a block's first field into w
    const long long nfr = PR / g.S + (g.R - 1) / g.S + 1, nfc = PC / g.S + (g.R - 1) / g.S + 1;
    LC_PLAN_REQUIRE(p, nfr * nfc * FG < (1LL << 20));
    LC_PLAN_REQUIRE(p, (long long)16 * MT * g.L * g.F * ES < (1LL << 32) && (nfr * g.LW + nfc) * g.K * g.F * ES < (1LL << 32) &&
                           (nfr * g.LW + nfc) * g.K * g.F < (1LL << 31));
    return LC_OK;
}

template <int MT, int NT, typename T>
int launch_tile(const Geom &g, const T *dy, const T *w, float *dx, const DataTile &t, int VW, bool plan_mask, hipStream_t s) {
    constexpr int GW = 64 / (int)sizeof(T);
    const int PR = g.S * t.qr, PC = g.S * t.qc, cbc = ceil_div(g.W, PC), FG = ceil_div(g.F, GW), nbt = ceil_div(g.B, 16 * MT);
    const long long ntask = (long long)ceil_div(g.H, PR) * cbc * nbt;
    const bool mask = !(t.qr == 1 && t.qc == 1 && g.R % g.S == 0 && g.F % GW == 0);
    const size_t lds = (t.ks > 1 ? (size_t)(t.ks * t.tasks / 2) * MT * NT * 1024 : 0) + (size_t)t.ks * t.tasks * (MT + NT) * 1024;
    dim3 grid((unsigned)((ntask + t.tasks - 1) / t.tasks), ceil_div(PR * PC * g.C, NT * 16));
    const LaunchPlan plan = make_plan("lc_bwd_data_general", {MT, NT, (int)sizeof(T), plan_mask, t.ks, t.tasks, VW, 1},
                                      {PR, PC, cbc, ceil_div(g.F, VW), nbt, (int)ntask}, grid, 64 * t.ks * t.tasks, lds);
    if (int rc = check_backward_data_turned(g, plan, mask, FG)) return rc;
    if (mask)
        LC_LAUNCH(plan, "lc_backward_data launch", (lc_bwd_data_turned_kernel<MT, NT, T, true>), s, g, dy, w, dx, PR, PC, divisor(cbc),
                  divisor(nbt), divisor(PC * g.C), divisor(g.C), divisor(g.S), divisor(FG), __builtin_ctz(t.ks), (int)ntask);
    else
        LC_LAUNCH(plan, "lc_backward_data launch", (lc_bwd_data_turned_kernel<MT, NT, T, false>), s, g, dy, w, dx, PR, PC, divisor(cbc),
                  divisor(nbt), divisor(PC * g.C), divisor(g.C), divisor(g.S), divisor(FG), __builtin_ctz(t.ks), (int)ntask);
    return LC_OK;
}

// Estimated clocks of a launch (G: groups of all pixel blocks together, most: of the block with most).  A group costs a wave its
// MFMAs (132 clocks a 16 x 16 tile in fp32, 48 where fp32 products are split, 17 in bf16), the splitting of the operands and,
// with masks, what finds the values outside a field; the waves share SIMDs, the vector cache and L2, and none ends before
// its own chain.  The constants are a fit to 161 layers timed with every tile, eight pixel blocks and four numbers of slices;
// what is picked is on average 6 % slower than the fastest.
double turned_clocks(const Geom &g, int es, const DataTile &t, double G, int most) {
    const bool f32 = es == 4, split = f32 && t.mt * t.nt >= 3, mask = !(t.qr == 1 && t.qc == 1 && g.R % g.S == 0 && g.F % (64 / es) == 0);
    const double N = (double)t.qr * t.qc * g.S * g.S * g.C, blocks = (double)ceil_div(g.H, g.S * t.qr) * ceil_div(g.W, g.S * t.qc);
    const double issue = (split ? 48.0 : f32 ? 132.0 : 17.0) * t.mt * t.nt + (split ? 89.0 : 0) * (t.mt + t.nt) +
                         (mask ? (f32 ? 45.0 : 64.0) * (t.mt + t.nt) : 0);
    const double add = (t.ks > 1 ? (f32 ? 388.0 : 353.0) * t.mt * t.nt + (f32 ? 71.0 : 0) * __builtin_ctz(t.ks) : 0) + (f32 ? 425.0 : 455.0);
    const double tiles = ceil_div(g.B, 16 * t.mt) * ceil(N / (16 * t.nt));
    const double busy = tiles * (G * issue + blocks * t.ks * add) / 1024, loads = tiles * G * (f32 ? 9.7 : 18.3) * (t.mt + t.nt) / 256;
    const double alone = ceil_div(most, t.ks) * (issue + (f32 ? 328.0 : 206.0)) + add;
    const double lines = tiles * G * (t.mt + t.nt) * 1024 / ((f32 ? 94.5 : 45.8) * 256);
    // together in the norm of order 3/2: between one after the other and all at once
    const double sum = busy * sqrt(busy) + loads * sqrt(loads) + alone * sqrt(alone) + lines * sqrt(lines);
    return cbrt(sum * sum) + (double)g.L * g.K * g.F * es * ceil_div(g.B, 16 * t.mt) / 3200 + 11000;
}

// The fastest tile by the estimate, where that is a tenth less than the direct form's takes here; grids of fewer than seven
// fields one way, whose blocks are mostly borders, keep the direct form's, whose estimate is of such (161 layers: 1.12 times
// as fast as the direct form in fp32 and 1.13 in bf16, 1.08 and 1.11 on its tiles).  Tiles that are not split take at least as
// many slices as the direct form's: a running sum is rounded once per matrix instruction, and fewer slices end less precise (45
// layers 1.28 times the direct form's error, 0.97 with as many; 1.10 times the time).
DataTile pick_turned(const Geom &g, int es, const DataTile &direct) {
    if (g.LH < 7 || g.LW < 7) return direct;
    const int FG = ceil_div(g.F, 64 / es);
    auto clocks = [&](const DataTile &t) {
        double fr, fc;
        int mr, mc;
        fields_across(g, t.qr, g.H, g.LH, &fr, &mr);
        fields_across(g, t.qc, g.W, g.LW, &fc, &mc);
        return turned_clocks(g, es, t, fr * fc * FG, mr * mc * FG);
    };
    const double own = clocks(direct);
    DataTile best = direct;
    double best_t = 1e300;
    static const int blocks[8][2] = {{1, 1}, {1, 2}, {2, 1}, {2, 2}, {1, 4}, {3, 3}, {4, 4}, {2, 4}};
    for (const auto &q : blocks) {
        const long long N = (long long)q[0] * q[1] * g.S * g.S * g.C;
        if (q[0] * q[1] > 1 && (N > 64 || q[0] > ceil_div(g.H, g.S) || q[1] > ceil_div(g.W, g.S))) continue;
        double fr, fc;
        int mr, mc;
        fields_across(g, q[0], g.H, g.LH, &fr, &mr);
        fields_across(g, q[1], g.W, g.LW, &fc, &mc);
        for (int mt = 1; mt <= 4; ++mt) {
            if (mt > 1 && 16 * (mt - 1) >= g.B) break;
            if ((double)ceil_div(g.H, g.S * q[0]) * ceil_div(g.W, g.S * q[1]) * ceil_div(g.B, 16 * mt) > (double)kMostTasks) continue;
            for (int nt = 1; nt <= 4; ++nt) {
                if (nt > 1 && 16 * (nt - 1) >= N) break;
                if ((N + 16 * nt - 1) / (16 * nt) > 65535) continue;
                const int least = es == 4 && mt * nt >= 3 ? 1 : direct.ks;
                for (int ks = least; ks <= kTurnedDataWaves && (ks == least || 2 * ks <= mr * mc * FG); ks *= 2) {
                    const DataTile t = {mt, nt, ks >= 4 ? 1 : 4 / ks, ks, q[0], q[1]};
                    const double c = turned_clocks(g, es, t, fr * fc * FG, mr * mc * FG);
                    if (c < best_t) {
                        best_t = c;
                        best = t;
                    }
                }
            }
        }
    }
    return own > 1.1 * best_t ? best : direct;
}

template <typename T>
int launch(const Geom &g, const T *dy, const T *w, float *dx, const DataTile &direct, int VW, hipStream_t s) {
    static thread_local TileMemo<DataTile> memo;
    const DataTile t = memo.get(g, sizeof(T), [&](const Geom &, int es) { return pick_turned(g, es, direct); });
    const bool plan_mask = !(t.qr == 1 && t.qc == 1 && g.R % g.S == 0 && g.F % VW == 0);
#define LC_TILE(M, N) if (t.mt == M && t.nt == N) return launch_tile<M, N>(g, dy, w, dx, t, VW, plan_mask, s)
    LC_TILE(1, 1); LC_TILE(2, 1); LC_TILE(3, 1); LC_TILE(4, 1);
    LC_TILE(1, 2); LC_TILE(2, 2); LC_TILE(3, 2); LC_TILE(4, 2);
    LC_TILE(1, 3); LC_TILE(2, 3); LC_TILE(3, 3); LC_TILE(4, 3);
    LC_TILE(1, 4); LC_TILE(2, 4); LC_TILE(3, 4); LC_TILE(4, 4);
#undef LC_TILE
    return LC_EINTERNAL;
}

}  // namespace

bool backward_data_turned_takes(const Geom &g, int es) {
    const int GW = 64 / es;
    const long long nf = 17 + (g.R - 1) / g.S;
    return g.F >= GW && 4 * ceil_div(g.F, GW) * GW <= 5 * g.F && (nf * g.LW + nf) * g.K * g.F < (1LL << 31);
}

int launch_backward_data_turned(const Geom &g, const float *dy, const float *w, float *dx, const DataTile &direct, int VW,
                                hipStream_t s) {
    return launch(g, dy, w, dx, direct, VW, s);
}
int launch_backward_data_turned(const Geom &g, const bf16_t *dy, const bf16_t *w, float *dx, const DataTile &direct, int VW,
                                hipStream_t s) {
    return launch(g, dy, w, dx, direct, VW, s);
}

}  // namespace lc
