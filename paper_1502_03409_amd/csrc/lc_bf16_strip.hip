// bf16 operands on the layers whose patch rows are not multiples of 16 values or whose filters come in blocks of 16
// or 32: lc_forward with the strip-sharing decomposition of the fp32 pipelined kernel
// (Sec. 3.1's untied fields overlap by R-S pixels, so a strip of adjacent fields shares the image rows it reads) and
// v_mfma_f32_16x16x16_bf16 in place of the fp32 matrix instruction.
//
// Workgroup = 4 adjacent fields of one field row, one per wave, x a batch tile of 16*MT images x 16*NT filters.  A chunk is
// CQ values of one patch row: the strip of x that the four fields share and each field's weight rows, both loaded into
// registers while the chunk before is computed and written to LDS between two barriers.  The contraction runs in blocks of
// 16 patch values: lane (m,kk) reads the four values 16 blk + 4 kk .. +3 of image m; lane (n,kk) reads the NT filters
// f0 + NT n .. of the four weight rows 16 blk + 4 kk .. +3 (the filters are the fast index of w, the patch values the
// slow one) and transposes them in registers into NT operands of four consecutive patch values each.  A chunk
// that is no multiple of 16 ends in a partial block: its lanes beyond the chunk feed zeros in both operands (the LDS
// holds the neighbouring field's pixels there, and the last weight row again: zeros on one side only would let an
// infinity or a NaN into fields that do not hold it).
//
// What bounds it is the number of loads a compute unit can have outstanding beyond L2, so they are few and wide: a lane
// takes 16 bytes of one weight row, an instruction whole lines (asked for as the NT filters of each lane, each line came in
// two to four pieces), and none is conditional.  Weight row r of a block lies in LDS at r % 4, r / 4: a wave's read of "row
// 4 kk + jj, filters NT n .." is 128 NT contiguous bytes.  128 images of 200 x 200 x 3, 20 x 20 at stride 4, 32 filters:
// 183 -> 107 us with operands out of the caches, 109 -> 72 with what fits them, against weights from global memory by the lane
// that multiplies them.  120 layers drawn from 17 to 256 images and 16 to 192 filters, half of them with 48 or 80 filters or at
// most 32 images: 1.54 times out of the caches (geometric mean, 1.02 to 2.5), 1.55 in them (1.06 to 2.4).  Blocks of filters of
// one strip follow each other: at the far ends of the launch 80 filters on 26 images of 79 x 90 x 8, 19 x 19 / 3 took 145 us in
// the caches (131 before the staged weights), side by side 67.
#include "lc_common.hpp"

namespace lc {
namespace {

constexpr int kStripSlots = 12;   // 8-byte staging registers per lane: chunk <= 12 * 256 * 8 B = 24 KB

// o[u] = (r[0].e_u, r[1].e_u, r[2].e_u, r[3].e_u): four rows of NT bf16 each -> NT operands of four rows
template <int NT>
__device__ __forceinline__ void rows_to_operands(const typename RawVec<bf16_t, NT>::V (&r)[4], u32x2 (&o)[NT]) {
    constexpr unsigned LO = 0x05040100u, HI = 0x07060302u;   // low / high halves of {src0:src1}
    if constexpr (NT == 1) {
        o[0] = (u32x2){(unsigned)r[0] | ((unsigned)r[1] << 16), (unsigned)r[2] | ((unsigned)r[3] << 16)};
    } else if constexpr (NT == 2) {
        o[0] = (u32x2){__builtin_amdgcn_perm(r[1], r[0], LO), __builtin_amdgcn_perm(r[3], r[2], LO)};
        o[1] = (u32x2){__builtin_amdgcn_perm(r[1], r[0], HI), __builtin_amdgcn_perm(r[3], r[2], HI)};
    } else {
        o[0] = (u32x2){__builtin_amdgcn_perm(r[1][0], r[0][0], LO), __builtin_amdgcn_perm(r[3][0], r[2][0], LO)};
        o[1] = (u32x2){__builtin_amdgcn_perm(r[1][0], r[0][0], HI), __builtin_amdgcn_perm(r[3][0], r[2][0], HI)};
        o[2] = (u32x2){__builtin_amdgcn_perm(r[1][1], r[0][1], LO), __builtin_amdgcn_perm(r[3][1], r[2][1], LO)};
        o[3] = (u32x2){__builtin_amdgcn_perm(r[1][1], r[0][1], HI), __builtin_amdgcn_perm(r[3][1], r[2][1], HI)};
    }
}

// OFF: byte offsets inside a batch tile of x, 64 bits where its images take 4 GB and more
template <int MT, int NT, int NB, int NS, int OCC, typename OFF>
__global__ __launch_bounds__(256, OCC) void lc_forward_bf16_staged_kernel(Geom g, const bf16_t *__restrict__ x,
                                                                       const bf16_t *__restrict__ w,
                                                                       const float *__restrict__ bias, float alpha,
                                                                       float *__restrict__ y, int strips_per_row,
                                                                       int CQ, int sq4, int RS, int nbt, int nslots) {
    typedef typename RawVec<bf16_t, NT>::V WV;    // NT consecutive filters of one weight row
    typedef typename FVec<NT>::T OV;              // NT consecutive outputs
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(1))) u32x4 *gw_ptr;
    typedef const __attribute__((address_space(1))) u32x2 *gx4_ptr;
    typedef const __attribute__((address_space(1))) char *gc_ptr;
    constexpr int NLOC = 4, BT = 16 * MT, NTHR = 64 * NLOC;
    constexpr int LPR = 2 * NT, RPL = 64 / LPR;              // lanes per weight row, rows per load
    constexpr int NL = (16 * NB + RPL - 1) / RPL;            // loads per wave and chunk
    constexpr int FB = 16 * NB * 16 * NT;                    // staged weights of a field, in values
    extern __shared__ __attribute__((aligned(16))) bf16_t xh[];      // [BT][RS] strip, then [NLOC][FB] weights
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 15, kk = lane >> 4;
    // blocks of filters, then batch tiles of one strip are neighbours in dispatch order on the same XCD: the blocks share
    // the strip, and lines of the weights where a line holds several blocks (grid.y > 1: too many workgroups for that)
    const int nfb = gridDim.y > 1 ? 1 : g.F / (16 * NT);
    const int t_id = remap_xcd(blockIdx.x, gridDim.x), t_fb = t_id / nfb;
    const int work = t_fb / nbt;
    const int i = work / strips_per_row, j0 = (work - i * strips_per_row) * NLOC;
    const int b0 = (t_fb - work * nbt) * BT;
    const int j = j0 + wave;
    const int f0 = (blockIdx.y + t_id - t_fb * nfb) * NT * 16;
    const bool active = j < g.LW;
    const int loc = i * g.LW + (active ? j : g.LW - 1);   // idle waves shadow the last field of the row
    const int SC = g.S * g.C, WC = g.W * g.C;
    const size_t img = (size_t)g.H * WC;

    f32x4 acc[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int u = 0; u < NT; ++u) acc[mt][u] = (f32x4){0.f, 0.f, 0.f, 0.f};

    // staging map: slot q of this thread copies 4-value vector number e = tid + NTHR*q of the [BT][sq4] chunk.  Lanes past
    // the chunk's end, images beyond B and values beyond the last field of the row repeat the nearest one that exists (goff,
    // loff: bytes), so that no load or store is conditional but for whole slots.
    const int vmax = (min(NLOC, g.LW - j0) - 1) * SC + CQ;   // values that the strip's fields read
    OFF goff[NS];
    unsigned loff[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        const int e = min(tid + NTHR * q, BT * sq4 - 1);
        const int b = e / sq4, v = min(4 * (e - b * sq4), vmax - 4);
        goff[q] = 2 * ((OFF)min(b, g.B - 1 - b0) * (OFF)img + v);
        loff[q] = 2u * (b * RS + v);
    }
    const gc_ptr xrow = (gc_ptr)(x + (size_t)b0 * img + (size_t)(i * g.S) * WC + j0 * SC);
    u32x2 st[NS];
    auto stage_load = [&](int kh, int sc) {
        const gc_ptr row = xrow + 2 * ((size_t)kh * WC + sc * CQ);
#pragma unroll
        for (int q = 0; q < NS; ++q)
            if (q < nslots) st[q] = *(gx4_ptr)(row + goff[q]);
    };
    auto stage_store = [&]() {
#pragma unroll
        for (int q = 0; q < NS; ++q)
            if (q < nslots) *(u32x2 *)((char *)xh + loff[q]) = st[q];
    };
    // weights: load q of this wave holds row RPL q + lane / LPR of the chunk, filters 8 (lane % LPR) ..; rows past
    // the chunk repeat its last one
    const gc_ptr wfield = (gc_ptr)(w + (size_t)loc * g.K * g.F + f0);
    bf16_t *wlds = xh + (size_t)BT * RS + wave * FB;
    u32x4 wr[NL];
    auto weights_load = [&](int kbase) {
        const gc_ptr base = wfield + 2 * (size_t)kbase * g.F;
#pragma unroll
        for (int q = 0; q < NL; ++q) {
            const int r = min(RPL * q + lane / LPR, CQ - 1);
            wr[q] = *(gw_ptr)(base + 2u * (unsigned)(r * g.F + 8 * (lane % LPR)));
        }
    };
    auto weights_store = [&]() {
#pragma unroll
        for (int q = 0; q < NL; ++q) {
            const int r = RPL * q + lane / LPR, at = (r & ~15) | ((r & 3) << 2) | ((r >> 2) & 3);
            if (16 * NB % RPL == 0 || r < 16 * NB) *(u32x4 *)(wlds + at * 16 * NT + 8 * (lane % LPR)) = wr[q];
        }
    };

    const bf16_t *xwin = xh + n * RS + wave * SC + 4 * kk;
    const bf16_t *wwin = wlds + kk * 16 * NT + n * NT;
    const int nsub = g.RC / CQ, nchunks = g.R * nsub;
    stage_load(0, 0);
    weights_load(0);
    int kh = 0, sc = 0;
    for (int c = 0; c < nchunks; ++c) {
        __syncthreads();                    // all waves are done reading the previous chunk
        stage_store();
        weights_store();
        __syncthreads();
        if (++sc == nsub) { sc = 0; ++kh; }
        if (c + 1 < nchunks) {
            stage_load(kh, sc);
            weights_load(kh * g.RC + sc * CQ);
        }
        __builtin_amdgcn_sched_barrier(0x2 | 0x4 | 0x8 | 0x80);   // the loads leave before the chunk's arithmetic
#pragma unroll
        for (int blk = 0; blk < NB; ++blk) {
            u32x2 a[MT], bo[NT];
            WV r[4];
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) r[jj] = *(const WV *)(wwin + blk * 256 * NT + jj * 64 * NT);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) a[mt] = *(const u32x2 *)(xwin + mt * 16 * RS + 16 * blk);
            rows_to_operands<NT>(r, bo);
            if (blk == NB - 1 && 16 * blk + 4 * kk >= CQ) {   // lanes past the end of the chunk
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) a[mt] = (u32x2){0u, 0u};
#pragma unroll
                for (int u = 0; u < NT; ++u) bo[u] = (u32x2){0u, 0u};
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int u = 0; u < NT; ++u) acc[mt][u] = mfma16_bf16(a[mt], bo[u], acc[mt][u]);
        }
    }

    if (!active) return;
    OV bv;
    if constexpr (NT == 1) bv = 0.f; else bv = (OV)(0.f);
    if (bias) bv = *(const OV *)(bias + (size_t)loc * g.F + f0 + NT * n);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int b = b0 + mt * 16 + 4 * kk + r;
            if (b >= g.B) continue;
            OV o;
            if constexpr (NT == 1) {
                o = alpha * acc[mt][0][r] + bv;
            } else {
#pragma unroll
                for (int u = 0; u < NT; ++u) o[u] = alpha * acc[mt][u][r] + bv[u];
            }
            *(OV *)(y + ((size_t)b * g.L + loc) * g.F + f0 + NT * n) = o;
        }
}

// 32-bit byte offsets inside a batch tile of x
bool strip_offsets_fit(const Geom &g, int BT) { return (long long)BT * g.H * g.W * g.C < (1LL << 31); }

// Host check of a lc_forward_bf16_staged_kernel launch.  tparam = {MT, NT, NB, NS, waves per SIMD, 64-bit offsets}; arg = {CQ,
// sq4, RS (bf16 values), batch tiles, strips per field row, slots}.
int check_forward_bf16_staged(const Geom &g, const LaunchPlan &p) {
    const int MT = p.tparam[0], NT = p.tparam[1], NB = p.tparam[2], NS = p.tparam[3];
    const int CQ = p.arg[0], sq4 = p.arg[1], RS = p.arg[2], nbt = p.arg[3], strips = p.arg[4], nslots = p.arg[5];
    const int BT = 16 * MT, SC = g.S * g.C, WC = g.W * g.C, sqc = 4 * sq4;
    LC_PLAN_REQUIRE(p, (NT == 1 || NT == 2 || NT == 4) && p.block == 256);
    // 8-byte accesses of four bf16 values in x, 16-byte ones of eight filters in w
    LC_PLAN_REQUIRE(p, g.RC % 4 == 0 && WC % 4 == 0 && SC % 4 == 0);
    LC_PLAN_REQUIRE(p, g.F % (NT * 16) == 0 && p.grid[2] == 1);
    // chunks of CQ values in NB blocks of 16 (the last one may be partial)
    LC_PLAN_REQUIRE(p, CQ > 0 && CQ % 4 == 0 && g.RC % CQ == 0 && NB == ceil_div(CQ, 16));
    LC_PLAN_REQUIRE(p, sqc == CQ + 3 * SC);
    LC_PLAN_REQUIRE(p, nslots <= NS && (long long)BT * sq4 <= (long long)nslots * 256);
    LC_PLAN_REQUIRE(p, (p.tparam[5] == 1 || strip_offsets_fit(g, BT)) && (long long)CQ * g.F < (1LL << 30));
    // a partial last block reads up to 12 values past a field's window; the weights behind the strip start on 16 bytes
    LC_PLAN_REQUIRE(p, RS % 8 == 0 && RS >= sqc + 16);
    LC_PLAN_REQUIRE(p, p.lds_bytes >= ((size_t)BT * RS + 4 * NB * 256 * NT) * sizeof(bf16_t));
    LC_PLAN_REQUIRE(p, strips == ceil_div(g.LW, 4) && nbt == ceil_div(g.B, BT));
    // blocks of filters: all in grid.x, or all in grid.y
    const int nfb = g.F / (NT * 16);
    LC_PLAN_REQUIRE(p, nfb <= 65535 && (p.grid[1] == 1 || (int)p.grid[1] == nfb));
    LC_PLAN_REQUIRE(p, (long long)p.grid[0] * p.grid[1] == (long long)strips * g.LH * nbt * nfb);
    return LC_OK;
}

// row stride in bf16 values: 16 bytes on or back modulo 128 bytes, so that the 16 image rows a wave reads at once start
// four banks apart, with at least 16 values of padding behind the staged strip
int strip_row_stride(int sqc) {
    int rs = (sqc + 16 + 7) & ~7;
    while (rs % 64 != 8 && rs % 64 != 56) rs += 8;
    return rs;
}
size_t strip_lds(const Geom &g, int BT, int CQ, int NT) {
    const int sqc = CQ + 3 * g.S * g.C;
    return ((size_t)BT * strip_row_stride(sqc) + (size_t)4 * ((CQ + 15) / 16) * 256 * NT) * sizeof(bf16_t);
}

// the largest chunk (a divisor of a patch row in whole 4-value vectors, at most 128 values) whose strip fits the staging
// registers and whose strip and weights fit lds bytes; 0 if none does
int strip_chunk(const Geom &g, int BT, int NT, size_t lds) {
    const int SC = g.S * g.C;
    for (int CQ = g.RC < 128 ? g.RC : 128; CQ >= 4; CQ -= 4) {   // (RC is a multiple of four)
        if (g.RC % CQ) continue;
        const long long sqc = CQ + 3LL * SC;
        if (BT * (sqc / 4) > kStripSlots * 256) continue;
        if (strip_lds(g, BT, CQ, NT) > lds || (long long)CQ * g.F >= (1LL << 30)) continue;
        return CQ;
    }
    return 0;
}

// Batch tile, filters per workgroup and chunk.  64-image tiles: several workgroups fit a compute unit and the second tile of
// a strip finds the weights in L2 (128 images in 8 waves that share the staged weights: 112 against 108 us on the 200 x 200
// layer, and up to 1.5 times slower on others).  Wide filter blocks read the strip fewer times; where they leave room for
// chunks of less than one block only (patch rows of 4 times a prime), or of less than a third of what narrower ones take (100
// values: 20 under 64 filters; 173 images of 168 x 100 x 4, 25 x 25 / 7, 192 filters 250 -> 158 us), narrower ones keep the row.
struct StripPick {
    int MT, NT, CQ;
};
StripPick strip_pick(const Geom &g) {
    const int MT = g.B > 32 ? 4 : 2, BT = 16 * MT;
    StripPick p = {MT, 0, 0};
    for (int NT : {4, 2, 1}) {
        if (g.F % (16 * NT)) continue;
        // LDS of two (64 filters, for their registers) or three workgroups a compute unit; two with 32 filters where three
        // would cut a row in three and more (40 layers 1.25 and 1.28 times, 1.07 at least; 99 images of 29 x 170 x 12, 7 x 7 / 3,
        // 96 filters 36.6 -> 32.7 us)
        int CQ = strip_chunk(g, BT, NT, (NT == 4 ? 80 : 53) * 1024);
        if (NT == 2 && CQ >= 16) {
            const int wide = strip_chunk(g, BT, NT, 80 * 1024);
            if (wide > 2 * CQ) CQ = wide;
        }
        if (CQ > (p.CQ < 16 ? p.CQ : 3 * p.CQ)) p.NT = NT, p.CQ = CQ;
    }
    return p;
}

template <int MT, int NT, int NB, int NS, typename OFF = unsigned>
int launch_strip_ns(const Geom &g, const bf16_t *x, const bf16_t *w, const float *bias, float alpha, float *y, int CQ,
                    hipStream_t s) {
    constexpr int BT = 16 * MT, OCC = NT == 4 ? 2 : 3;
    const int sqc = CQ + 3 * g.S * g.C, RS = strip_row_stride(sqc);
    const int strips = (g.LW + 3) / 4, nbt = (g.B + BT - 1) / BT, nslots = ceil_div(BT * (sqc / 4), 256);
    const long long nwg = (long long)strips * g.LH * nbt;
    if (nwg > 0x7fffffffLL) return LC_EUNSUPPORTED;
    // the runtime counts a dimension's threads in 32 bits: 2^24 workgroups of 256 and more keep the blocks of filters in y
    const int nfb = g.F / (NT * 16);
    const bool flat = nwg * nfb < (1 << 24);
    dim3 grid((unsigned)(flat ? nwg * nfb : nwg), flat ? 1 : nfb);
    auto kern = lc_forward_bf16_staged_kernel<MT, NT, NB, NS, OCC, OFF>;
    const LaunchPlan plan = make_plan("lc_forward_bf16_staged", {MT, NT, NB, NS, OCC, sizeof(OFF) == 8}, {CQ, sqc / 4, RS, nbt, strips, nslots},
                                      grid, 256, strip_lds(g, BT, CQ, NT));
    if (int rc = check_forward_bf16_staged(g, plan)) return rc;
    LC_LAUNCH(plan, "lc_forward (bf16 strip) launch", kern, s, g, x, w, bias, alpha, y, strips, CQ, sqc / 4, RS, nbt, nslots);
    return LC_OK;
}

template <int MT, int NT, int NB>
int launch_strip(const Geom &g, const bf16_t *x, const bf16_t *w, const float *bias, float alpha, float *y, int CQ,
                 hipStream_t s) {
    if (!strip_offsets_fit(g, 16 * MT))
        return launch_strip_ns<MT, NT, NB, kStripSlots, unsigned long long>(g, x, w, bias, alpha, y, CQ, s);
    if (16 * MT * (CQ + 3 * g.S * g.C) <= 6 * 4 * 256) return launch_strip_ns<MT, NT, NB, 6>(g, x, w, bias, alpha, y, CQ, s);
    return launch_strip_ns<MT, NT, NB, kStripSlots>(g, x, w, bias, alpha, y, CQ, s);
}

template <int MT, int NT>
int launch_strip_nb(const Geom &g, const bf16_t *x, const bf16_t *w, const float *bias, float alpha, float *y, int CQ,
                    hipStream_t s) {
    switch ((CQ + 15) / 16) {
        case 1: return launch_strip<MT, NT, 1>(g, x, w, bias, alpha, y, CQ, s);
        case 2: return launch_strip<MT, NT, 2>(g, x, w, bias, alpha, y, CQ, s);
        case 3: return launch_strip<MT, NT, 3>(g, x, w, bias, alpha, y, CQ, s);
        case 4: return launch_strip<MT, NT, 4>(g, x, w, bias, alpha, y, CQ, s);
        case 5: return launch_strip<MT, NT, 5>(g, x, w, bias, alpha, y, CQ, s);
        case 6: return launch_strip<MT, NT, 6>(g, x, w, bias, alpha, y, CQ, s);
        case 7: return launch_strip<MT, NT, 7>(g, x, w, bias, alpha, y, CQ, s);
        default:
            // 64 images with blocks of 64 filters: beyond strip_pick's LDS
            if constexpr (MT == 4 && NT == 4) return LC_EUNSUPPORTED;
            else return launch_strip<MT, NT, 8>(g, x, w, bias, alpha, y, CQ, s);
    }
}

// ------------------------------------------------------------------------------ backward weights
// dw[l,k,f] = beta dw + sum_b x[b, patch k of l] dy[b,l,f] with bf16 operands (the weight gradient of Eq. 1's terms).
// The decomposition of the fp32 kernel: a wave owns one location, G*64 patch elements and 16*NT filters, both
// operands come straight from global memory with lanes along the contiguous axis (4 patch elements of an image row,
// NT filters).  The contraction runs over the batch, 16 images per bf16 MFMA: lane (m,kk) loads its vectors for the
// four images 4 kk .. +3 of a step and transposes them in registers, so that operand t holds patch element
// kg + 4 m + t (operand u: filter f0 + NT m + u) of those four images.  Loads run PF steps ahead in a register ring.
template <int G, int NT, int PF>
__global__ __launch_bounds__(256, 4) void lc_bwd_weights_bf16_rows_kernel(Geom g, const bf16_t *__restrict__ x,
                                                                       const bf16_t *__restrict__ dy, float beta,
                                                                       float *__restrict__ out, int kblocks,
                                                                       int ntasks) {
    typedef typename RawVec<bf16_t, NT>::V BR;     // NT consecutive dy values as loaded
    typedef typename FVec<NT>::T BV;               // NT consecutive outputs
    // the patch vectors are only element-aligned in general (a field starts every S*C elements)
    typedef __attribute__((address_space(1), aligned(2))) u32x2 GAV;
    typedef __attribute__((address_space(1))) BR GBV;
    typedef const __attribute__((address_space(1))) bf16_t *gt_ptr;
    constexpr int KB = G * 64;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int m = lane & 15, kk = lane >> 4;
    const int task = remap_xcd(blockIdx.x, gridDim.x) * 4 + wave;
    if (task >= ntasks) return;
    const int loc = task / kblocks, k0 = (task - loc * kblocks) * KB;
    const int i = loc / g.LW, j = loc - i * g.LW;
    const int f0 = blockIdx.y * NT * 16;
    const size_t img = (size_t)g.H * g.W * g.C, dyimg = (size_t)g.L * g.F;

    // rows of the A tiles beyond K are loaded from a valid address (element 0 of the patch) and never stored
    gt_ptr xa[G];
#pragma unroll
    for (int gg = 0; gg < G; ++gg) {
        const int k = k0 + gg * 64 + 4 * m;
        const int kc = k < g.K ? k : 0;
        const int kh = kc / g.RC, rem = kc - kh * g.RC;
        xa[gg] = (gt_ptr)x + (size_t)(4 * kk) * img + ((i * g.S + kh) * g.W + j * g.S) * g.C + rem;
    }
    gt_ptr da = (gt_ptr)dy + (size_t)(4 * kk) * dyimg + (size_t)loc * g.F + f0 + NT * m;

    f32x4 acc[G][4][NT];
#pragma unroll
    for (int gg = 0; gg < G; ++gg)
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int u = 0; u < NT; ++u) acc[gg][t][u] = (f32x4){0.f, 0.f, 0.f, 0.f};

    u32x2 a[PF][G][4];
    BR bv[PF][4];
    auto load_step = [&](int ss) {      // one step = 16 images: this lane's four, then on to the next step
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
#pragma unroll
            for (int gg = 0; gg < G; ++gg) a[ss][gg][jj] = *(const GAV *)(xa[gg] + (size_t)jj * img);
            bv[ss][jj] = *(const GBV *)(da + (size_t)jj * dyimg);
        }
#pragma unroll
        for (int gg = 0; gg < G; ++gg) xa[gg] += 16 * img;
        da += 16 * dyimg;
    };
    auto mul_step = [&](int ss) {
        u32x2 bo[NT];
        rows_to_operands<NT>(bv[ss], bo);
#pragma unroll
        for (int gg = 0; gg < G; ++gg) {
            u32x2 ao[4];
            rows_to_operands<4>(a[ss][gg], ao);
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int u = 0; u < NT; ++u) acc[gg][t][u] = mfma16_bf16(ao[t], bo[u], acc[gg][t][u]);
        }
    };
    const int nsteps = g.B >> 4;             // B % (16*PF) == 0 on this path
#pragma unroll
    for (int ss = 0; ss < PF; ++ss) load_step(ss);
    for (int s0 = PF; s0 < nsteps; s0 += PF) {
#pragma unroll
        for (int ss = 0; ss < PF; ++ss) {
            mul_step(ss);
            load_step(ss);
            // the refill of slot ss stays right behind the MFMAs that consumed it
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int ss = 0; ss < PF; ++ss) mul_step(ss);

    float *ol = out + (size_t)loc * g.K * g.F + f0 + NT * m;
#pragma unroll
    for (int gg = 0; gg < G; ++gg)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int k = k0 + gg * 64 + 4 * (4 * kk + r) + t;
                if (k >= g.K) continue;
                BV *o = (BV *)(ol + (size_t)k * g.F);
                BV v;
                if constexpr (NT == 1) {
                    v = acc[gg][t][0][r];
                } else {
#pragma unroll
                    for (int u = 0; u < NT; ++u) v[u] = acc[gg][t][u][r];
                }
                if (beta != 0.f) v += beta * *o;
                *o = v;
            }
}

// Host check of a lc_bwd_weights_bf16_rows_kernel launch.  tparam = {G, NT, PF}; arg = {blocks of 64*G patch elements
// per field, wave tasks}.
int check_backward_weights_bf16_rows(const Geom &g, const LaunchPlan &p) {
    const int G = p.tparam[0], NT = p.tparam[1], PF = p.tparam[2];
    const int kblocks = p.arg[0], ntasks = p.arg[1];
    LC_PLAN_REQUIRE(p, p.block == 256 && (NT == 1 || NT == 2 || NT == 4));
    LC_PLAN_REQUIRE(p, g.RC % 4 == 0 && g.F % (NT * 16) == 0 && (int)p.grid[1] == g.F / (NT * 16) && p.grid[2] == 1);
    LC_PLAN_REQUIRE(p, PF >= 1 && g.B % (16 * PF) == 0);
    LC_PLAN_REQUIRE(p, kblocks == ceil_div(g.K, 64 * G) && (long long)ntasks == (long long)g.L * kblocks);
    LC_PLAN_REQUIRE(p, (long long)p.grid[0] * 4 >= ntasks && (long long)(p.grid[0] - 1) * 4 < ntasks);
    LC_PLAN_REQUIRE(p, (long long)g.H * g.W * g.C < (1LL << 31));
    return LC_OK;
}

template <int G, int NT, int PF>
int launch_rows(const Geom &g, const bf16_t *x, const bf16_t *dy, float beta, float *out, hipStream_t s) {
    constexpr int KB = G * 64;
    const int kblocks = (g.K + KB - 1) / KB;
    const long long ntasks = (long long)g.L * kblocks;
    if (ntasks > (1LL << 30)) return LC_EUNSUPPORTED;
    dim3 grid((unsigned)((ntasks + 3) / 4), g.F / (NT * 16));
    const LaunchPlan plan = make_plan("lc_bwd_weights_bf16_rows", {G, NT, PF}, {kblocks, (int)ntasks}, grid, 256, 0);
    if (int rc = check_backward_weights_bf16_rows(g, plan)) return rc;
    LC_LAUNCH(plan, "lc_backward_weights (bf16 rows) launch", (lc_bwd_weights_bf16_rows_kernel<G, NT, PF>), s, g, x, dy,
              beta, out, kblocks, (int)ntasks);
    return LC_OK;
}

// one step in flight and four waves per SIMD measured as fast as two steps and three waves (104 x 104 x 12 input, 10 x 10 fields, 32 filters, batch 128: 150 vs 153 us)
template <int G, int NT>
int launch_rows_pf(const Geom &g, const bf16_t *x, const bf16_t *dy, float beta, float *out, hipStream_t s) {
    return launch_rows<G, NT, 1>(g, x, dy, beta, out, s);
}

// The weight gradient with the patches shared through LDS.  In the kernel above every wave fetches its own
// 1200 x 128 patch, and those 8-byte loads are what binds it (same layer: 152 us, 88 us with the patch loads compiled out).
// Here a workgroup takes four adjacent fields and stages, per patch row, the image-row strip they share (as the
// forward kernel does; 2.5x fewer patch bytes on that layer, fetched once); wave = field.  Per patch row a wave contracts
// over the whole batch: lane (m,kk) reads the patch values 4 m .. +3 of the four images 16 s + 4 kk .. +3
// from LDS and transposes them in registers into four operands; the dy operands of all steps sit in registers for
// the whole kernel (batches up to 128 images).  The 64 x 16 NT tile of a patch row is stored as soon as it is
// complete.  Rows beyond the patch row read the neighbour's pixels: they only reach output rows that
// are not stored.  The patch rows are split over grid.z so that small layers still fill the chip.
// Unconditional staging loads and streamed stores: 127 -> 105 us on the 128 x 200 x 200 x 3 layer out of the caches, 108 -> 84
// in them; 60 drawn layers of up to 128 images 1.33 and 1.32 times (geometric mean, 1.03 at least) against a branch per load.
// OFF: byte offsets into x, 64 bits from 4 GB on.  NSTEP: steps of 16 images the batch may have; with eight for every batch the
// loads of dy asked for the last image again and again (29 images of 34 x 50 x 4, 13 x 13 / 2, 32 filters: 11.1 us, 8.8 with two).
template <int NT, bool STREAM, typename OFF, int NSTEP>
__global__ __launch_bounds__(256, 3) void lc_bwd_weights_bf16_strip_kernel(Geom g, const bf16_t *__restrict__ x,
                                                                         const bf16_t *__restrict__ dy, float beta,
                                                                         float *__restrict__ out, int strips_per_row,
                                                                         int sq4, int RS, int rows_per_wg) {
    typedef typename RawVec<bf16_t, NT>::V BR;     // NT consecutive dy values as loaded
    typedef typename FVec<NT>::T BV;               // NT consecutive outputs
    typedef const __attribute__((address_space(1))) BR *gb_ptr;
    typedef const __attribute__((address_space(1))) u32x2 *gx4_ptr;
    typedef const __attribute__((address_space(1))) char *gc_ptr;
    constexpr int BT = 16 * NSTEP, NLOC = 4, NTHR = 256;
    extern __shared__ __attribute__((aligned(16))) bf16_t xh[];      // [BT][RS] (+ 64 values of slack)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = lane & 15, kk = lane >> 4;
    const int work = remap_xcd(blockIdx.x, gridDim.x);
    const int i = work / strips_per_row, j0 = (work - i * strips_per_row) * NLOC;
    const int j = j0 + wave;
    const bool active = j < g.LW;
    const int loc = i * g.LW + (active ? j : g.LW - 1);   // idle waves shadow the last field of the row
    const int f0 = blockIdx.y * NT * 16;
    const int kh_lo = blockIdx.z * rows_per_wg, kh_hi = min(g.R, kh_lo + rows_per_wg);
    const int SC = g.S * g.C, WC = g.W * g.C;
    const size_t img = (size_t)g.H * WC, dyimg = (size_t)g.L * g.F;

    // dy operands of every step: images 16 s + 4 kk .. +3, filters f0 + NT m .. (zeros beyond the batch)
    const bf16_t *dyl = dy + (size_t)loc * g.F + f0 + NT * m;
    u32x2 bo[NSTEP][NT];
#pragma unroll
    for (int st = 0; st < NSTEP; ++st) {
        BR r[4];
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const int b = 16 * st + 4 * kk + jj;
            r[jj] = *(gb_ptr)(dyl + (size_t)min(b, g.B - 1) * dyimg);
            if (b >= g.B) r[jj] = BR{};
        }
        rows_to_operands<NT>(r, bo[st]);
    }

    // staging map: slot q copies 4-value vector number tid + 256 q of the [B][sq4] chunk; lanes past its end and values beyond
    // the last field of the row repeat the nearest one that exists (goff, loff: bytes), so that no load or store is
    // conditional but for whole slots.  Images beyond B are cleared once.
    const int nslots = (g.B * sq4 + NTHR - 1) / NTHR;
    const int vmax = (min(NLOC, g.LW - j0) - 1) * SC + g.RC;   // values that the strip's fields read
    OFF goff[kStripSlots];
    unsigned loff[kStripSlots];
#pragma unroll
    for (int q = 0; q < kStripSlots; ++q) {
        const int e = min(tid + NTHR * q, g.B * sq4 - 1);
        const int b = e / sq4, v = min(4 * (e - b * sq4), vmax - 4);
        goff[q] = 2 * ((OFF)b * (OFF)img + v);
        loff[q] = 2u * (b * RS + v);
    }
    for (int e = g.B * (RS >> 2) + tid; e < BT * (RS >> 2); e += NTHR) *(u32x2 *)(xh + 4 * e) = (u32x2){0u, 0u};
    const gc_ptr xrow = (gc_ptr)(x + (size_t)(i * g.S) * WC + j0 * SC);
    u32x2 st[kStripSlots];
    auto stage_load = [&](int kh) {
        const gc_ptr row = xrow + 2 * ((size_t)kh * WC);
#pragma unroll
        for (int q = 0; q < kStripSlots; ++q)
            if (q < nslots) st[q] = *(gx4_ptr)(row + goff[q]);
    };
    auto stage_store = [&]() {
#pragma unroll
        for (int q = 0; q < kStripSlots; ++q)
            if (q < nslots) *(u32x2 *)((char *)xh + loff[q]) = st[q];
    };

    const bf16_t *xwin = xh + (size_t)(4 * kk) * RS + wave * SC + 4 * m;
    float *ol = out + (size_t)loc * g.K * g.F + f0 + NT * m;
    const int nsteps = (g.B + 15) >> 4;
    if (kh_lo < kh_hi) stage_load(kh_lo);
    for (int kh = kh_lo; kh < kh_hi; ++kh) {
        __syncthreads();                    // all waves are done reading the previous patch row
        stage_store();
        __syncthreads();
        if (kh + 1 < kh_hi) stage_load(kh + 1);
        __builtin_amdgcn_sched_barrier(0x2 | 0x4 | 0x8 | 0x80);   // the loads leave before the row's arithmetic
        {
            f32x4 acc[4][NT];
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int u = 0; u < NT; ++u) acc[t][u] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int sp = 0; sp < NSTEP; ++sp) {
                if (sp < nsteps) {          // uniform
                    u32x2 r[4], ao[4];
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) r[jj] = *(const u32x2 *)(xwin + (size_t)(16 * sp + jj) * RS);
                    rows_to_operands<4>(r, ao);
#pragma unroll
                    for (int t = 0; t < 4; ++t)
#pragma unroll
                        for (int u = 0; u < NT; ++u) acc[t][u] = mfma16_bf16(ao[t], bo[sp][u], acc[t][u]);
                }
            }
            if (active) {
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const int kl = 4 * (4 * kk + r) + t;
                        if (kl >= g.RC) continue;
                        BV *o = (BV *)(ol + (size_t)(kh * g.RC + kl) * g.F);
                        BV v;
                        if constexpr (NT == 1) {
                            v = acc[t][0][r];
                        } else {
#pragma unroll
                            for (int u = 0; u < NT; ++u) v[u] = acc[t][u][r];
                        }
                        if (beta != 0.f) v += beta * *o;
                        if constexpr (STREAM) stream_store(v, o);
                        else *o = v;
                    }
            }
        }
    }
}

// row stride: 16 bytes past a multiple of 128 bytes, wide enough for the staged strip and for the 64 values of
// the last field (which reach past its patch row)
int wstrip_row_stride(const Geom &g, int sqc) {
    const int need = std::max(sqc, 3 * g.S * g.C + 64);
    return ((need - 8 + 63) / 64) * 64 + 8;
}

// Host check of a lc_bwd_weights_bf16_strip_kernel launch.  tparam = {NT, streamed stores, 64-bit offsets, steps of 16 images};
// arg = {strips per field row, sq4, RS (bf16 values), patch rows per workgroup}.
int check_backward_weights_bf16_strip(const Geom &g, const LaunchPlan &p) {
    const int NT = p.tparam[0];
    const int strips = p.arg[0], sq4 = p.arg[1], RS = p.arg[2], rows_per_wg = p.arg[3];
    const int SC = g.S * g.C, WC = g.W * g.C, sqc = 4 * sq4;
    LC_PLAN_REQUIRE(p, p.block == 256 && (NT == 1 || NT == 2 || NT == 4));
    LC_PLAN_REQUIRE(p, g.RC % 4 == 0 && SC % 4 == 0 && WC % 4 == 0 && g.B <= 16 * p.tparam[3] && p.tparam[3] <= 8);
    LC_PLAN_REQUIRE(p, g.F % (NT * 16) == 0 && (int)p.grid[1] == g.F / (NT * 16));
    // a patch row in a block of 64 values; the last field's block reads past its patch row inside the LDS row
    LC_PLAN_REQUIRE(p, g.RC <= 64);
    LC_PLAN_REQUIRE(p, sqc >= g.RC + 3 * SC && sqc <= 0xffff);
    LC_PLAN_REQUIRE(p, (long long)128 * sq4 <= (long long)kStripSlots * 256);
    LC_PLAN_REQUIRE(p, p.tparam[2] == 1 || strip_offsets_fit(g, g.B));
    LC_PLAN_REQUIRE(p, RS % 4 == 0 && RS >= sqc && RS >= 3 * SC + 64);
    LC_PLAN_REQUIRE(p, p.lds_bytes >= ((size_t)128 * RS + 64) * sizeof(bf16_t));
    LC_PLAN_REQUIRE(p, strips == ceil_div(g.LW, 4) && (long long)p.grid[0] == (long long)strips * g.LH);
    LC_PLAN_REQUIRE(p, rows_per_wg >= 1 && (long long)p.grid[2] * rows_per_wg >= g.R &&
                           (long long)(p.grid[2] - 1) * rows_per_wg < g.R);
    return LC_OK;
}

template <int NT, bool STREAM, typename OFF, int NSTEP>
int launch_wstrip_steps(const Geom &g, const bf16_t *x, const bf16_t *dy, float beta, float *out, hipStream_t s) {
    const int sqc = (g.RC + 3 * g.S * g.C + 3) & ~3;
    const int RS = wstrip_row_stride(g, sqc);
    const size_t lds = ((size_t)128 * RS + 64) * sizeof(bf16_t);
    auto kern = lc_bwd_weights_bf16_strip_kernel<NT, STREAM, OFF, NSTEP>;
    const int strips = (g.LW + 3) / 4;
    const long long nwork = (long long)strips * g.LH;
    if (nwork > 0x7fffffffLL) return LC_EUNSUPPORTED;
    // split the patch rows over grid.z until there are about four workgroups per compute unit
    int zsplit = 1;
    while (zsplit < g.R && nwork * (g.F / (NT * 16)) * zsplit < 4 * 256) ++zsplit;
    const int rows_per_wg = (g.R + zsplit - 1) / zsplit;
    dim3 grid((unsigned)nwork, g.F / (NT * 16), (g.R + rows_per_wg - 1) / rows_per_wg);
    const LaunchPlan plan = make_plan("lc_bwd_weights_bf16_strip", {NT, (int)STREAM, sizeof(OFF) == 8, NSTEP}, {strips, sqc / 4, RS, rows_per_wg}, grid, 256, lds);
    if (int rc = check_backward_weights_bf16_strip(g, plan)) return rc;
    LC_LAUNCH(plan, "lc_backward_weights (bf16 strip) launch", kern, s, g, x, dy, beta, out, strips, sqc / 4, RS,
              rows_per_wg);
    return LC_OK;
}

template <int NT, bool STREAM, typename OFF>
int launch_wstrip_as(const Geom &g, const bf16_t *x, const bf16_t *dy, float beta, float *out, hipStream_t s) {
    if constexpr (!STREAM)
        if (g.B <= 32) return launch_wstrip_steps<NT, STREAM, OFF, 2>(g, x, dy, beta, out, s);
    return g.B <= 64 ? launch_wstrip_steps<NT, STREAM, OFF, 4>(g, x, dy, beta, out, s)
                     : launch_wstrip_steps<NT, STREAM, OFF, 8>(g, x, dy, beta, out, s);
}

bool wstrip_supported(const Geom &g) {
    const int SC = g.S * g.C;
    if (g.RC % 4 || SC % 4 || (g.W * g.C) % 4 || g.F % 16 || g.B > 128 || g.RC > 64) return false;
    const int sqc = (g.RC + 3 * SC + 3) & ~3;
    if ((size_t)128 * (sqc / 4) > (size_t)kStripSlots * 256) return false;
    return ((size_t)128 * wstrip_row_stride(g, sqc) + 64) * sizeof(bf16_t) <= 48 * 1024 && sqc <= 0xffff;
}

// Streamed stores: whole lines (32 filters) of a gradient that is overwritten go past the caches where the reads of x weigh
// (128 images of 200 x 200 x 3: 99 -> 85 us); below 58 images the stores bind by themselves and the caches smooth them (32 of
// 48 x 29 x 4, 96 filters: 32 against 39), as they do with the half lines of 16 filters (72 of 54 x 108 x 4: 58 against 82).
template <int NT>
int launch_wstrip(const Geom &g, const bf16_t *x, const bf16_t *dy, float beta, float *out, hipStream_t s) {
    const bool fit = strip_offsets_fit(g, g.B);
    if constexpr (NT == 2)
        if (g.B >= 64 && beta == 0.f)
            return fit ? launch_wstrip_as<NT, true, unsigned>(g, x, dy, beta, out, s)
                       : launch_wstrip_as<NT, true, unsigned long long>(g, x, dy, beta, out, s);
    return fit ? launch_wstrip_as<NT, false, unsigned>(g, x, dy, beta, out, s)
               : launch_wstrip_as<NT, false, unsigned long long>(g, x, dy, beta, out, s);
}

}  // namespace

// Shapes: patch rows in whole 4-value vectors, filters in blocks of 16, and either batches in steps of 16 images or
// a shape the strip-sharing kernel takes (any batch up to 128: it stages the missing images as zeros).
bool bf16_strip_backward_weights_supported(const Geom &g) { return g.RC % 4 == 0 && g.F % 16 == 0 && wstrip_supported(g); }

bool bf16_rows_backward_weights_supported(const Geom &g) {
    return g.RC % 4 == 0 && g.F % 16 == 0 && (g.B % 16 == 0 || wstrip_supported(g));
}

int launch_backward_weights_bf16_rows(const Geom &g, const void *xv, const void *dyv, float beta, float *dw,
                                      hipStream_t s) {
    if (!bf16_rows_backward_weights_supported(g)) return LC_EUNSUPPORTED;
    const bf16_t *x = (const bf16_t *)xv, *dy = (const bf16_t *)dyv;
    if (wstrip_supported(g)) {
        if (g.F % 32 == 0) return launch_wstrip<2>(g, x, dy, beta, dw, s);
        return launch_wstrip<1>(g, x, dy, beta, dw, s);
    }
    if (g.F % 64 == 0) return launch_rows_pf<1, 4>(g, x, dy, beta, dw, s);
    if (g.F % 32 == 0) return launch_rows_pf<2, 2>(g, x, dy, beta, dw, s);
    return launch_rows_pf<2, 1>(g, x, dy, beta, dw, s);
}

// Shapes: patch rows, field offsets and image rows in whole 4-value vectors (8-byte accesses), filters in blocks of 16.
bool bf16_strip_forward_supported(const Geom &g) {
    const int SC = g.S * g.C;
    if (g.RC % 4 || SC % 4 || (g.W * g.C) % 4 || g.F % 16 || g.B <= 16) return false;
    const StripPick p = strip_pick(g);
    // (with 64-bit offsets rows in pieces of less than a block go to the kernels on bf16 storage: 64 images of 3400 x 3400 x 4,
    // 16 x 16 / 15, 32 filters in eights 2.6 ms there, 4.4 here; whole rows of 32 to 64 values 3.0 to 6.2 ms there, 2.1 to 2.7 here)
    return p.CQ >= (strip_offsets_fit(g, 16 * p.MT) ? 4 : 16);
}

// with the widest blocks of filters
long long bf16_strip_forward_workgroups(const Geom &g) {
    const int nt = g.F % 64 == 0 ? 4 : g.F % 32 == 0 ? 2 : 1, bt = g.B > 32 ? 64 : 32;
    return (long long)((g.LW + 3) / 4) * g.LH * ceil_div(g.B, bt) * (g.F / (16 * nt));
}

int launch_forward_bf16_strip(const Geom &g, const void *xv, const void *wv, const float *bias, float alpha, float *y,
                              hipStream_t s) {
    if (!bf16_strip_forward_supported(g)) return LC_EUNSUPPORTED;
    const bf16_t *x = (const bf16_t *)xv, *w = (const bf16_t *)wv;
    const StripPick p = strip_pick(g);
    if (p.MT == 4) {
        if (p.NT == 4) return launch_strip_nb<4, 4>(g, x, w, bias, alpha, y, p.CQ, s);
        if (p.NT == 2) return launch_strip_nb<4, 2>(g, x, w, bias, alpha, y, p.CQ, s);
        return launch_strip_nb<4, 1>(g, x, w, bias, alpha, y, p.CQ, s);
    }
    if (p.NT == 4) return launch_strip_nb<2, 4>(g, x, w, bias, alpha, y, p.CQ, s);
    if (p.NT == 2) return launch_strip_nb<2, 2>(g, x, w, bias, alpha, y, p.CQ, s);
    return launch_strip_nb<2, 1>(g, x, w, bias, alpha, y, p.CQ, s);
}

}  // namespace lc
