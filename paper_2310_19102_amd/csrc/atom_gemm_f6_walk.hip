// The packed group GEMM (atom_gemm_f6.hip: operands, unit images, exactness) for launches of many tiles.
//
// Tile 64 WR x 128, 2 WR wavefronts, each a 64 x 64 block of its own = four 32 x 32 sub-tiles; per sub-tile and INT4 group
// two FP6 MFMAs, the fp16 MFMA of the scale products and 16 fused multiply-adds.  WR = 4: one workgroup per compute
// unit, four LDS stages; WR = 2: two workgroups per compute unit, three stages each.
//
// What bounds it: no single pipe.  At steady clocks (1.8 GHz under the power limit, 2.38 GHz with operands of zeros, which
// run the same instructions) a step of the WR = 4 tile takes 1420 cycles; the matrix pipe needs 840 of them (24 MFMAs
// of 35 cycles per SIMD), the vector pipe 560, the vector memory path 640 (40 KB per step at 64 bytes per clock), and
// what leaves the L2 costs another 8 %.  Measured on a wavefront alone, every instruction it issues counts: so
//   * the multiply-adds of a sub-tile stand 4, 6 and 6 behind the three MFMAs of the next one (registers only: 484
//     cycles for 12 MFMAs and 64 multiply-adds, against 556 with 0, 8 and 8);
//   * a request is two scalar instructions and the load: one base address per operand, moved on by a step, and a
//     lane offset that serves every tile, because the last tile of a row or column of tiles is moved back so that
//     it is whole (what two tiles share they both compute, to the same bits);
//   * the weights are the row operand of the MFMA, so that a lane holds four consecutive columns of a row of Y and the
//     output staging is a quarter of the LDS writes.
// Against the walking kernel before this one (in turn on one card, half a second each): M = 4096, K = 8192, N = 57344: 1531 -> 1516 us;
// N = 10240: 272.5 -> 268.6 us; K = 28672, N = 8192: 718.9 -> 717.9 us (under the power limit, which decides there); M = 1024,
// K = 4096, N = 22016: 91.8 -> 83.8 us; M = 777, K = 5120, N = 13824 (WR = 2): 59.9 -> 57.6 us.  Wider tiles (64 x 96 per
// wavefront; 64 x 128 does not fit the registers) fetch fewer bytes and lose it again to the power limit and to partial rounds.
// A moved-back tile that leaves out the stores of what the tile before it stores is no faster (M = 192, N = 28672: 38.2 us, 37.9) and
// costs 1 % elsewhere.
//
// Workgroups walk tiles, and the stream of requests never stops at a tile's end.  The K loop's last NST steps have
// nothing of their own INT4 groups left to ask for: two of them fetch the two parts of the INT8 group, the others the
// first NST - 2 groups of the next tile; the stages of the INT8 group afterwards hold the output staging areas and then,
// behind one barrier, the next tile's other two groups.  vmcnt counts instructions in order, so the number of
// vector-memory instructions between two requests is the same in every wavefront and tile: XTRA stores (or, in a wavefront
// whose block is cut by M or N, which stores first and waits, and before the first tile, as many one-lane requests).

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include <type_traits>

#include "atom_gemm_f6.h"
#include "atom_launch.h"

namespace {

using namespace atom_gemm_f6;

template <int WR>
struct Walk {
    static constexpr int NJ    = 2;                           // units of weights of a tile = blocks of 32 columns of a wavefront
    static constexpr int NW    = 2 * WR;                      // wavefronts: WR rows x 2 columns
    static constexpr int NT    = 64 * NW;
    static constexpr int APART = round_kb(WR * IMG4);         // activation part of a stage, in whole requests
    static constexpr int WPART = round_kb(NJ * IMG4);
    static constexpr int STAGE = APART + WPART;
    static constexpr int NST   = WR == 4 ? 4 : 3;            // LDS stages
    static constexpr int NA    = APART / 1024, NB = WPART / 1024;
    static constexpr int KA    = (NA + NW - 1) / NW, KB = (NB + NW - 1) / NW;          // requests per wavefront and stage
    static constexpr int LPW   = KA + KB;
    static constexpr int NA8   = round_kb(WR * IMG8) / 1024, NB8 = round_kb(NJ * IMG8) / 1024;
    static constexpr int SPARE = NST * STAGE;                 // 16 bytes that are written and never read
    static constexpr int LDS   = SPARE + 64;
    static constexpr int OSTR  = 144;                         // output staging: bytes per row of 64 columns
    static constexpr int XTRA  = 8;                           // 16-byte stores per lane of a wavefront's block
    static_assert(1024 * NA8 <= STAGE && 1024 * NB8 <= STAGE, "a part of the INT8 group fits a stage");
    static_assert(NA8 <= LPW * NW && NB8 <= LPW * NW, "a part of the INT8 group is one stage's requests");
    static_assert(WR * 64 * OSTR <= STAGE, "half of the staging areas fit a stage");
    static_assert(LDS <= 160 * 1024 && (NST - 1) * LPW + XTRA <= 63, "LDS, vmcnt");
};

template <int WR>
__global__ __launch_bounds__(WR * 128, 2)
void w4a4_gemm_f6_walk_kernel(const F6Params p)
{
    using Gm = Walk<WR>;
    constexpr int NJ = Gm::NJ, NW = Gm::NW, NST = Gm::NST, STAGE = Gm::STAGE, LPW = Gm::LPW, XTRA = Gm::XTRA;
    constexpr int APART = Gm::APART, KA = Gm::KA;
    constexpr int T = 2 * NJ;                                 // sub-tiles of a wavefront
    using std::integral_constant;

    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WR, wn = wave / WR;
    const int r = lane & 31, g = lane >> 5;
    const int G4 = p.G4;

    // ---- the tiles of this workgroup: logical, logical + lstep, ... < lend of its XCD's contiguous share
    const int TM = (p.a_units + WR - 1) / WR, TN = (p.w_units + NJ - 1) / NJ;
    int logical, lstep, lend;
    {
        const int ntiles = TM * TN, nb = gridDim.x, xcd = blockIdx.x & 7;
        const int per = ntiles >> 3, rem = ntiles & 7;
        const int start = xcd * per + (xcd < rem ? xcd : rem);
        logical = start + (int)(blockIdx.x >> 3);
        lstep   = (nb - xcd + 7) >> 3;
        lend    = start + per + (xcd < rem ? 1 : 0);
        if (logical >= lend) return;
    }
    struct Tile { const uint8_t *a, *w; int au0, wu0; };
    auto tile_of = [&](int lt) __attribute__((always_inline)) -> Tile {
        const int band = 8 * TN, b = lt / band, rem = lt - b * band;
        const int hgt = TM - 8 * b < 8 ? TM - 8 * b : 8;      // M-tiles in this band
        const int tm = 8 * b + rem % hgt, tn = rem / hgt;
        Tile t;
        t.au0 = tm * WR < p.a_units - WR ? tm * WR : p.a_units - WR;
        t.wu0 = tn * NJ < p.w_units - NJ ? tn * NJ : p.w_units - NJ;
        t.a = p.a_pk + (int64_t)t.au0 * p.ustride;
        t.w = p.w_pk + (int64_t)t.wu0 * p.ustride;
        return t;
    };
    Tile cur_t = tile_of(logical), nxt_t = cur_t;

    // ---- loader: the activation (weight) part of a stage is the units' images one behind the other; piece j of a part is
    // its bytes [1024 j, 1024 j + 1024), moved by wavefront j % NW; lanes past the end of the part repeat its last 16 bytes
    // (they land in the padding)
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(smem), spare = lds0 + Gm::SPARE;
    uint32_t voff[LPW];
    auto part_off = [&](int j, int units, int img, int ln) __attribute__((always_inline)) -> uint32_t {
        int q = 64 * j + ln;                                   // 16-byte chunk of the part
        q = q < units * (img / 16) ? q : units * (img / 16) - 1;
        const int unit = q / (img / 16);
        return (uint32_t)unit * (uint32_t)p.ustride + 16u * (q - unit * (img / 16));
    };
#pragma unroll
    for (int k = 0; k < LPW; ++k)
        voff[k] = k < KA ? part_off(wave + NW * k, WR, IMG4, lane) : part_off(wave + NW * (k - KA), NJ, IMG4, lane);
    // request k of the group whose images start at a / w, into `stage`; !real: one lane, to where nobody reads
    auto request = [&](int k, const uint8_t *a, const uint8_t *w, int stage, bool real) __attribute__((always_inline)) {
        const bool act = k < KA;
        const int kk = act ? k : k - KA, n = act ? Gm::NA : Gm::NB, j = wave + NW * kk;
        const uint32_t dst = lds0 + stage * STAGE + (act ? 0 : APART) + 1024 * j;
        dma16_masked(j < n && real ? dst : spare, voff[k], act ? a : w, j < n && real ? ~0ull : 1ull);
    };
    auto request_now = [&](int k, const uint8_t *a, const uint8_t *w, int stage) __attribute__((always_inline)) {
        const bool act = k < KA;
        const int kk = act ? k : k - KA, n = act ? Gm::NA : Gm::NB, j = wave + NW * kk;
        const uint32_t dst = lds0 + stage * STAGE + (act ? 0 : APART) + 1024 * j;
        if (NW * (kk + 1) <= n) dma16(dst, voff[k], act ? a : w);
        else dma16_masked(j < n ? dst : spare, voff[k], act ? a : w, j < n ? ~0ull : 1ull);
    };
    // request k of a part of the INT8 group, into `stage`
    int lane_t = lane;
    auto request8 = [&](int k, int stage, bool act) __attribute__((always_inline)) {
        const int j = wave + NW * k, n = act ? Gm::NA8 : Gm::NB8;
        const uint8_t *base = (act ? cur_t.a : cur_t.w) + (int64_t)G4 * IMG4;
        if (NW * k >= n) dma16_masked(spare, 0u, base, 1ull);
        else dma16_masked(j < n ? lds0 + stage * STAGE + 1024 * j : spare, part_off(j, act ? WR : NJ, IMG8, lane_t), base, j < n ? ~0ull : 1ull);
    };
    auto dummy = [&]() __attribute__((always_inline)) { dma16_masked(spare, 0u, cur_t.a, 1ull); };

    // ---- fragment addresses inside a stage
    const uint32_t lane_off = lds0 + 1024 * g + 16 * r;
    const uint32_t a_off = wm * IMG4 + lane_off, b_off = APART + wn * IMG4 + lane_off;
    const uint32_t sa_off = lds0 + wm * IMG4 + SC4 + 8 * r, sb_off = lds0 + APART + wn * IMG4 + SC4 + 8 * r;
    typedef __attribute__((address_space(3))) const v4i *lds_v4i;
    typedef __attribute__((address_space(3))) const v2u *lds_v2u;
    auto read_pair = [&](uint32_t addr, int off) __attribute__((always_inline)) -> v12i {
        const v4i c0 = *(lds_v4i)(uintptr_t)(addr + off);
        const v4i c1 = *(lds_v4i)(uintptr_t)(addr + off + 2048);
        const v4i c2 = *(lds_v4i)(uintptr_t)(addr + off + 4096);
        const v8i lo = __builtin_shufflevector(c0, c1, 0, 1, 2, 3, 4, 5, 6, 7);
        const v8i hi = __builtin_shufflevector(c2, c2, 0, 1, 2, 3, -1, -1, -1, -1);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11);
    };
    auto read_scale = [&](uint32_t addr, int off) __attribute__((always_inline)) -> v2u {
        return *(lds_v2u)(uintptr_t)(addr + off);
    };

    v16f acc[T];                                               // sub-tile (i, j) at 2 j + i
    const v16f zf = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    v12i af[2], bf[2];
    v2u  sa[2], sb[2];
    v16f c[2], s[2];                                           // partial sums and scale products of two sub-tiles in flight
    uint32_t a_cur, b_cur, sa_cur, sb_cur;                     // lane addresses in the stage being read
    int cur = 0;

    auto scale_tile = [&](v2u tw, v2u tx) __attribute__((always_inline)) -> v16f {
        return __builtin_amdgcn_mfma_f32_32x32x8f16(__builtin_bit_cast(v4h, tw), __builtin_bit_cast(v4h, tx), zf, 0, 0, 0);
    };
    auto dequant = [&](v16f &a, const v16f &cc, const v16f &ss, int e0, int e1) __attribute__((always_inline)) {
#pragma unroll
        for (int e = e0; e < e1; ++e) a[e] = fmaf(cc[e], ss[e], a[e]);
        ATOM_F6_PIN(a);
    };
    auto set_stage = [&](int st) __attribute__((always_inline)) {
        a_cur = a_off + st * STAGE; b_cur = b_off + st * STAGE; sa_cur = sa_off + st * STAGE; sb_cur = sb_off + st * STAGE;
    };

    // One sub-tile = three slots of one MFMA each.  The fused multiply-adds of the sub-tile before are spread over all
    // three (4, 6, 6): the vector ALU then works in the shadow of every MFMA.  `req(slot)` issues the requests that
    // belong there.
    auto subtile = [&](auto t_c, bool next_stage_known, auto req) __attribute__((always_inline)) {
        constexpr int t = decltype(t_c)::value, i = t & 1, j = t >> 1, q = t & 1, pt = (t + T - 1) % T;
        if constexpr (i == 0) sb[j][0] = g == 0 ? sb[j][0] : 0u;        // (zero on one side keeps k-slots 4..7 empty)
        ATOM_F6_PIN(af[i]);
        ATOM_F6_PIN(bf[j]);
        c[q] = mfma_f6<0>(bf[j], af[i], zf);
        ATOM_F6_PIN(c[q]);
        // Fragment reads: what sub-tile 0 is the first to find free registers for, of the group being worked on; column
        // fragment 0 and row fragment 0 of the next group, after their last use, once its stage is known to be there.
        if constexpr (t == 0) {
            af[1] = read_pair(a_cur, 512);
            bf[1] = read_pair(b_cur, 512);
            sa[1] = read_scale(sa_cur, 256);
            sb[1] = read_scale(sb_cur, 256);
        } else if constexpr (t == 2) {
            if (next_stage_known) { bf[0] = read_pair(b_cur, 0); sb[0] = read_scale(sb_cur, 0); }
        } else if constexpr (t == 3) {
            if (next_stage_known) { af[0] = read_pair(a_cur, 0); sa[0] = read_scale(sa_cur, 0); }
        }
        req(0);
        dequant(acc[pt], c[q ^ 1], s[q ^ 1], 0, 4);
        ATOM_F6_SLOT_END();
        s[q] = scale_tile(sb[j], sa[i]);
        ATOM_F6_PIN(s[q]);
        req(1);
        dequant(acc[pt], c[q ^ 1], s[q ^ 1], 4, 10);
        ATOM_F6_SLOT_END();
        c[q] = mfma_f6<1>(bf[j], af[i], c[q]);
        ATOM_F6_PIN(c[q]);
        req(2);
        dequant(acc[pt], c[q ^ 1], s[q ^ 1], 10, 16);
        ATOM_F6_SLOT_END();
    };
    auto no_req = [](int) {};

    int base = 0;                                              // stage of the tile's group 0
    bool first = true;
    for (;;) {
        const int nlogical = logical + lstep;
        const bool more = nlogical < lend;
        nxt_t = tile_of(more ? nlogical : logical);
        asm volatile("" : "+v"(lane_t));                       // (what only a tile's end needs is derived from it there, and holds no registers before)
        if (first) {
#pragma unroll
            for (int v = 0; v < NST; ++v)
#pragma unroll
                for (int k = 0; k < LPW; ++k) request_now(k, cur_t.a + (int64_t)v * IMG4, cur_t.w + (int64_t)v * IMG4, v);
#pragma unroll
            for (int k = 0; k < XTRA; ++k) dummy();
            first = false;
        }
        __builtin_amdgcn_s_waitcnt(wait_imm((NST - 1) * LPW + XTRA));
        __syncthreads();
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = zf;
        c[0] = c[1] = s[0] = s[1] = zf;
        cur = base;
        set_stage(cur);
        af[0] = read_pair(a_cur, 0); bf[0] = read_pair(b_cur, 0);
        sa[0] = read_scale(sa_cur, 0); sb[0] = read_scale(sb_cur, 0);
        // the first group's sub-tile before the barrier
        subtile(integral_constant<int, 0>{}, false, no_req);
        const uint8_t *a_run = cur_t.a + NST * IMG4, *w_run = cur_t.w + NST * IMG4;    // the group to request next
        // One body: from the barrier of group u to the barrier of group u + 1.  At its start stage `cur` (group u) is read
        // to the end by every wavefront and group u + 1 has landed.  MODE: what stage `cur` is refilled with: 0 group
        // u + NST, 1 / 2 the activation / weight part of the INT8 group, 3 group v of the next tile.  LAST: no group follows.
        auto body = [&](int v, auto mode_c, auto loose_c, auto last_c) __attribute__((always_inline)) {
            constexpr int MODE = decltype(mode_c)::value, LOOSE = decltype(loose_c)::value;
            constexpr bool LAST = decltype(last_c)::value;
            if constexpr (!LAST) __builtin_amdgcn_s_waitcnt(wait_imm((NST - 2) * LPW + LOOSE));
            else                 __builtin_amdgcn_s_waitcnt(wait_imm(63));
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
            const int refill = cur;
            constexpr int NSLOT = LAST ? 9 : 3 * T;
            auto req_at = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
                for (int k = 0; k < LPW; ++k)
                    if (k * NSLOT / LPW == slot) {
                        if constexpr (MODE == 0)      request_now(k, a_run, w_run, refill);
                        else if constexpr (MODE == 1) request8(k, refill, true);
                        else if constexpr (MODE == 2) request8(k, refill, false);
                        else                          request(k, nxt_t.a + v * IMG4, nxt_t.w + v * IMG4, refill, more);
                    }
            };
            cur = cur + 1 == NST ? 0 : cur + 1;
            if constexpr (!LAST) set_stage(cur);
            subtile(integral_constant<int, 1>{}, !LAST, [&](int q) __attribute__((always_inline)) { req_at(q); });
            subtile(integral_constant<int, 2>{}, !LAST, [&](int q) __attribute__((always_inline)) { req_at(3 + q); });
            subtile(integral_constant<int, 3>{}, !LAST, [&](int q) __attribute__((always_inline)) { req_at(6 + q); });
            if constexpr (!LAST) subtile(integral_constant<int, 0>{}, false, [&](int q) __attribute__((always_inline)) { req_at(9 + q); });
            if constexpr (MODE == 0) { a_run += IMG4; w_run += IMG4; }
        };
        int stage8a, stage8w;
        {
            using I0 = integral_constant<int, 0>;
            using F = std::false_type;
            int u = 0;
            for (; u < NST - 1; ++u) body(0, I0{}, integral_constant<int, XTRA>{}, F{});
            for (; u + NST < G4; ++u) body(0, I0{}, I0{}, F{});
            stage8a = cur; body(0, integral_constant<int, 1>{}, I0{}, F{});
            stage8w = cur; body(0, integral_constant<int, 2>{}, I0{}, F{});
            if constexpr (NST == 4) body(0, integral_constant<int, 3>{}, I0{}, F{});
            body(NST - 3, integral_constant<int, 3>{}, I0{}, std::true_type{});
        }
        dequant(acc[T - 1], c[1], s[1], 0, 16);

        // ---- the INT8 group: INT8 MFMA, int32 tile converted to fp32, the same dequantisation
        {
            int ck[4];                                         // byte offset of chunk 2 kk + g of row r
            const int rt = lane_t & 31, gt = lane_t >> 5;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) ck[kk] = 128 * rt + 16 * (((2 * kk + gt) ^ rt ^ ((rt >> 3) & 1)) & 7);
            __builtin_amdgcn_s_waitcnt(wait_imm((NST - 2) * LPW));
            __syncthreads();
            const unsigned char *a8 = smem + stage8a * STAGE + wm * IMG8;
            const unsigned char *w8 = smem + stage8w * STAGE + wn * IMG8;
            v4i x[2][4];
            v2u xs[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) x[i][kk] = *reinterpret_cast<const v4i *>(a8 + ck[kk] + 4096 * i);
                xs[i] = *reinterpret_cast<const v2u *>(a8 + SC8 + 8 * r + 256 * i);
            }
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                v4i w[4];
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) w[kk] = *reinterpret_cast<const v4i *>(w8 + ck[kk] + 4096 * j);
                v2u ws = *reinterpret_cast<const v2u *>(w8 + SC8 + 8 * r + 256 * j);
                ws[0] = g == 0 ? ws[0] : 0u;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    v16i ci = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) ci = __builtin_amdgcn_mfma_i32_32x32x32_i8(w[kk], x[i][kk], ci, 0, 0, 0);
                    const v16f ss = scale_tile(ws, xs[i]);
                    v16f cf;
#pragma unroll
                    for (int e = 0; e < 16; ++e) cf[e] = (float)ci[e];
                    dequant(acc[2 * j + i], cf, ss, 0, 16);
                }
            }
        }
        __syncthreads();                                       // the two stages of the INT8 group are free

        // ---- store: a lane holds four consecutive columns of one row of Y at a time; the wavefront's block goes through LDS so
        // that global memory sees whole 128-byte rows
        constexpr int OSTR = Gm::OSTR;
        unsigned char *ot = smem + (wave < NW / 2 ? stage8a : stage8w) * STAGE + (wave % (NW / 2)) * (64 * OSTR);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v2h lo = __builtin_convertvector((v2f{acc[t][4 * q], acc[t][4 * q + 1]}), v2h);
                const v2h hi = __builtin_convertvector((v2f{acc[t][4 * q + 2], acc[t][4 * q + 3]}), v2h);
                *reinterpret_cast<v2u *>(ot + (32 * (t & 1) + r) * OSTR + (32 * (t >> 1) + 8 * q + 4 * g) * 2) =
                    v2u{__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi)};
            }
        __builtin_amdgcn_s_waitcnt(wait_imm(63));              // (LDS only: the wavefront reads what it wrote itself)
        const bool vec_ok = ((reinterpret_cast<uintptr_t>(p.y) | (uintptr_t)(p.ldy * 2)) & 15) == 0;
        const int64_t m_w = 64 * (int64_t)(cur_t.au0 + wm), n_w = 64 * (int64_t)(cur_t.wu0 + wn);
        uint16_t *const yb = p.y + m_w * p.ldy + n_w;
        auto request_two = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < LPW; ++k) request(k, nxt_t.a + (NST - 2) * IMG4, nxt_t.w + (NST - 2) * IMG4, stage8a, more);
#pragma unroll
            for (int k = 0; k < LPW; ++k) request(k, nxt_t.a + (NST - 1) * IMG4, nxt_t.w + (NST - 1) * IMG4, stage8w, more);
        };
        // (the same decision in all lanes; each arm passes the one barrier)
        if (vec_ok && m_w + 64 <= p.M && n_w + 64 <= p.N) {
            v4i ov[XTRA];
#pragma unroll
            for (int it = 0; it < XTRA; ++it) ov[it] = *reinterpret_cast<const v4i *>(ot + (it * 8 + (lane_t >> 3)) * OSTR + (lane_t & 7) * 16);
            __builtin_amdgcn_s_waitcnt(wait_imm(63));
            __syncthreads();                                   // every staging area is read: the two stages are free
            request_two();
            uint16_t *const yl = yb + (lane_t >> 3) * p.ldy + (lane_t & 7) * 8;
#pragma unroll
            for (int it = 0; it < XTRA; ++it) *reinterpret_cast<v4i *>(yl + it * 8 * p.ldy) = ov[it];
        } else {
            if (m_w < p.M && n_w < p.N)
                store_block_any<64, 64>(ot, OSTR, yb, p.ldy, (int)(p.M - m_w < 64 ? p.M - m_w : 64), (int)(p.N - n_w < 64 ? p.N - n_w : 64), lane_t);
            __syncthreads();
            __builtin_amdgcn_s_waitcnt(wait_imm(0));
            request_two();
#pragma unroll
            for (int k = 0; k < XTRA; ++k) dummy();
        }
        if (!more) {
            __builtin_amdgcn_s_waitcnt(wait_imm(0));           // (the last requests have landed before the LDS is given up)
            break;
        }
        logical = nlogical;
        cur_t = nxt_t;
        base = (base + G4 + 2) % NST;
    }
}

template <int WR>
hipError_t launch_cfg(const F6Params &p, hipStream_t stream)
{
    using Gm = Walk<WR>;
    auto kern = &w4a4_gemm_f6_walk_kernel<WR>;
    static atom_launch::LdsOptIn opt_in;   // one attribute call per kernel variant and device
    hipError_t err = atom_launch::ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(kern), Gm::LDS);
    if (err != hipSuccess) return err;
    const int64_t tiles = (int64_t)((p.a_units + WR - 1) / WR) * ((p.w_units + Gm::NJ - 1) / Gm::NJ);
    const int64_t slots = (int64_t)atom_launch::compute_units() * (2 * Gm::LDS <= 160 * 1024 ? 2 : 1);
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles < slots ? tiles : slots)), dim3(Gm::NT), Gm::LDS, stream, p);
    return hipGetLastError();
}

}  // namespace

namespace atom_gemm_f6 {

hipError_t launch_walk(const F6Params &p, int tile, hipStream_t stream)
{
    return tile == 0 ? launch_cfg<2>(p, stream) : launch_cfg<4>(p, stream);
}

}  // namespace atom_gemm_f6
