// The packed group GEMM (atom_gemm_f6.hip: operands, unit images, exactness) for launches of many tiles.
//
// WM x WN wavefronts, each with a block of 64 rows and 32 JW columns of its own = 2 JW sub-tiles of 32 x 32; per sub-tile and INT4
// group two FP6 MFMAs, the fp16 MFMA of the scale products between them, and then 16 fused multiply-adds.  Tiles (WM, WN, JW):
// 128 x 128 (2, 2, 2), two workgroups per compute unit with three LDS stages each; one workgroup of eight wavefronts per compute unit
// for 256 x 128 (4, 2, 2), four stages, and 256 x 192 (4, 2, 3), 128 x 384 (2, 4, 3) and 256 x 256 (4, 2, 4), three; 192 x 128 (3, 2, 2) has six
// wavefronts and four stages.
//
// What bounds it: the power limit, and behind it no single pipe.  With operands of zeros the same instructions run at 2.39 GHz,
// with real ones at 1.7 to 2.1, so what a step moves counts as much as what it issues.  M = 4096, K = 8192, N = 16384, 256 x 128: 434 us;
// without the loads 324, without the multiply-adds 371, without the scale products 374, without the fragment reads 416; with all loads
// served by the L2 416.  A third fewer bytes per multiply-add (256 x 256: 52 KB for 256 x 256 x 128, 40 KB for half of that) is the
// largest of what can be had: 446 -> 385 us (M = 4096, K = 28672, N = 8192: 709 -> 627).  The pipes, in cycles of a 256 x 256 step:
// 2260, of which the matrix pipe 1600, the vector pipe 1100, the barrier 200, the loads 290.
//   * One sub-tile at a time, with one tile of sums and one of scale products: with two wavefronts to a SIMD one's multiply-adds
//     run under the other's MFMAs, and nothing is gained by spreading them under its own (registers only, per sub-tile of
//     both wavefronts: 219 cycles, 252 with the multiply-adds 4, 6 and 6 behind the three MFMAs of the next sub-tile, at
//     real operands 132 and 146 ns).  The 32 registers less are what lets 64 x 128 fit a wavefront (253 registers, no spills).
//   * The FP6 MFMA without scales: the scaled form is two instruction words more (24 MFMAs and 128 multiply-adds 1175 -> 1107 cycles).
//   * The fragments that a sub-tile frees are read again right behind its last MFMA (JW = 2, 3: 1 to 3 % faster than behind the next
//     sub-tile's first one; JW = 4: 1.5 % slower).  Not kept: s_setprio around the multiply-adds (1 to 2 % slower with the loads in
//     place), the barrier between a sub-tile's MFMAs and its multiply-adds (1 to 8 % slower), non-temporal loads (25 % slower).
//   * A request is two scalar instructions and the load: one base address per operand, moved on by a step, and a
//     lane offset that serves every tile, because the last tile of a row or column of tiles is moved back so that
//     it is whole (what two tiles share they both compute, to the same bits).
//   * The weights are the row operand of the MFMA, so that a lane holds four consecutive columns of a row of Y and the
//     output staging is a quarter of the LDS writes.  JW = 3 takes one half of each of three units, its neighbour the other: all its
//     fragment reads then are at fixed distances, and it stores rows of 64 bytes instead of 128.
// Against the kernel before, which had the two smaller tiles (in turn on one card, weights from HBM): M = 4096, K = 8192, N = 16384:
// 446 -> 385 us; M = 1024, K = 4096, N = 22016: 94.6 -> 86.1 us (256 x 192), N = 12288: 54.4 -> 43.7 (128 x 384); M = 777, K = 5120,
// N = 13824: 64.8 -> 54.0 us (128 x 384); on the tiles that both have, 256 x 128 446 -> 431, 30.3 -> 28.9 (M = 512, N = 11008), 128 x 128
// within 1 % either way.  A moved-back tile that leaves out the stores of what the tile before it stores is no faster (M = 192,
// N = 28672: 38.2 us, 37.9) and costs 1 % elsewhere.
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

template <int WM, int WN, int JW>
struct Walk {
    static constexpr int NJ    = WN * JW / 2;                 // units of weights of a tile
    static constexpr int NW    = WM * WN;
    static constexpr int NT    = 64 * NW;
    static constexpr int APART = round_kb(WM * IMG4);         // activation part of a stage, in whole requests
    static constexpr int WPART = round_kb(NJ * IMG4);
    static constexpr int STAGE = APART + WPART;
    static constexpr int NST   = NW >= 6 && JW == 2 ? 4 : 3; // LDS stages
    static constexpr int NA    = APART / 1024, NB = WPART / 1024;
    static constexpr int NR    = NA + NB;                     // requests of a stage: those of the activations, then the weights'
    static constexpr int LPW   = (NR + NW - 1) / NW;
    static constexpr int NA8   = round_kb(WM * IMG8) / 1024, NB8 = round_kb(NJ * IMG8) / 1024;
    static constexpr int SPARE = NST * STAGE;                 // 16 bytes that are written and never read
    static constexpr int LDS   = SPARE + 64;
    static constexpr int OSTR  = 144;                         // output staging: bytes per row of 64 columns
    static constexpr int XTRA  = JW % 2 ? 4 : 8;              // 16-byte stores per lane of the last part of a wavefront's block
    static_assert(1024 * NA8 <= STAGE && 1024 * NB8 <= STAGE, "a part of the INT8 group fits a stage");
    static_assert(NA8 <= LPW * NW && NB8 <= LPW * NW, "a part of the INT8 group is one stage's requests");
    static_assert(WN % 2 == 0 && NW / 2 * 64 * OSTR <= STAGE, "half of the staging areas fit a stage");
    static_assert(LDS <= 160 * 1024 && (NST - 1) * LPW + XTRA <= 63, "LDS, vmcnt");
};

template <int WM, int WN, int JW>
__global__ __launch_bounds__(64 * WM * WN, 2)
void w4a4_gemm_f6_walk_kernel(const F6Params p)
{
    using Gm = Walk<WM, WN, JW>;
    constexpr int NJ = Gm::NJ, NW = Gm::NW, NST = Gm::NST, STAGE = Gm::STAGE, LPW = Gm::LPW, XTRA = Gm::XTRA;
    constexpr int APART = Gm::APART;
    constexpr int T = 2 * JW;                                 // sub-tiles of a wavefront
    constexpr bool ODD = JW % 2 != 0, EARLY = JW < 4;
    using std::integral_constant;

    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int r = lane & 31, g = lane >> 5;
    const int G4 = p.G4;

    // ---- the tiles of this workgroup: logical, logical + lstep, ... < lend of its XCD's contiguous share
    const int TM = (p.a_units + WM - 1) / WM, TN = (p.w_units + NJ - 1) / NJ;
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
        t.au0 = tm * WM < p.a_units - WM ? tm * WM : p.a_units - WM;
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
    int wave_t = wave;
    uint32_t voff[LPW];
    auto part_off = [&](int j, int units, int img, int ln) __attribute__((always_inline)) -> uint32_t {
        int q = 64 * j + ln;                                   // 16-byte chunk of the part
        q = q < units * (img / 16) ? q : units * (img / 16) - 1;
        const int unit = q / (img / 16);
        return (uint32_t)unit * (uint32_t)p.ustride + 16u * (q - unit * (img / 16));
    };
#pragma unroll
    for (int k = 0; k < LPW; ++k) {
        const int j = wave + NW * k;
        voff[k] = j < Gm::NA ? part_off(j, WM, IMG4, lane) : part_off(j - Gm::NA, NJ, IMG4, lane);
    }
    // request k of the group whose images start at a / w, into `stage`; !real: one lane, to where nobody reads
    auto request = [&](int k, const uint8_t *a, const uint8_t *w, int stage, bool real) __attribute__((always_inline)) {
        const int j = wave_t + NW * k;
        const uint32_t dst = lds0 + stage * STAGE + 1024 * j;
        dma16_masked(j < Gm::NR && real ? dst : spare, voff[k], j < Gm::NA ? a : w, j < Gm::NR && real ? ~0ull : 1ull);
    };
    auto request_now = [&](int k, const uint8_t *a, const uint8_t *w, int stage) __attribute__((always_inline)) {
        const int j = wave + NW * k;
        const uint32_t dst = lds0 + stage * STAGE + 1024 * j;
        if (NW * (k + 1) <= Gm::NR) dma16(dst, voff[k], NW * (k + 1) <= Gm::NA ? a : NW * k >= Gm::NA ? w : j < Gm::NA ? a : w);
        else dma16_masked(j < Gm::NR ? dst : spare, voff[k], w, j < Gm::NR ? ~0ull : 1ull);
    };
    // request k of a part of the INT8 group, into `stage`
    int lane_t = lane;
    auto request8 = [&](int k, int stage, bool act) __attribute__((always_inline)) {
        const int j = wave_t + NW * k, n = act ? Gm::NA8 : Gm::NB8;
        const uint8_t *base = (act ? cur_t.a : cur_t.w) + (int64_t)G4 * IMG4;
        if (NW * k >= n) dma16_masked(spare, 0u, base, 1ull);
        else dma16_masked(j < n ? lds0 + stage * STAGE + 1024 * j : spare, part_off(j, act ? WM : NJ, IMG8, lane_t), base, j < n ? ~0ull : 1ull);
    };
    auto dummy = [&]() __attribute__((always_inline)) { dma16_masked(spare, 0u, cur_t.a, 1ull); };

    // ---- fragment addresses inside a stage.  A wavefront's JW blocks of 32 columns: JW / 2 whole units, or, JW odd, one half each of
    // JW units (the other halves are its neighbour's)
    const int w_unit = ODD ? (wn >> 1) * JW : wn * (JW / 2), w_half = ODD ? wn & 1 : 0;
    const uint32_t lane_off = lds0 + 1024 * g + 16 * r;
    const uint32_t a_off = wm * IMG4 + lane_off, b_off = APART + w_unit * IMG4 + 512 * w_half + lane_off;
    const uint32_t sa_off = lds0 + wm * IMG4 + SC4 + 8 * r, sb_off = lds0 + APART + w_unit * IMG4 + 256 * w_half + SC4 + 8 * r;
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
    constexpr int NBF = ODD ? JW : 2;                          // column fragments held (of the next group's, the first goes to where this group's was)
    auto b_at = [](int j) constexpr { return ODD ? j * IMG4 : (j >> 1) * IMG4 + (j & 1) * 512; };
    auto sb_at = [](int j) constexpr { return ODD ? j * IMG4 : (j >> 1) * IMG4 + (j & 1) * 256; };
    v12i af[2], bf[NBF];
    v2u  sa[2], sb[NBF];
    v16f c, s;                                           // partial sums and scale products of two sub-tiles in flight
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

    auto read_a = [&](int i) __attribute__((always_inline)) { af[i] = read_pair(a_cur, 512 * i); sa[i] = read_scale(sa_cur, 256 * i); };
    auto read_b = [&](int j) __attribute__((always_inline)) { bf[j % NBF] = read_pair(b_cur, b_at(j)); sb[j % NBF] = read_scale(sb_cur, sb_at(j)); };
    // One sub-tile: three slots of one MFMA each, then its multiply-adds.  Fragment reads stand behind the last use of what they
    // replace, those of the next group in the two sub-tiles behind the barrier.  `req(slot)` issues the requests that belong there.
    auto subtile = [&](auto t_c, bool next_stage_known, auto req) __attribute__((always_inline)) {
        constexpr int t = decltype(t_c)::value, i = t & 1, j = t >> 1, jb = j % NBF;
        if constexpr (i == 0) sb[jb][0] = g == 0 ? sb[jb][0] : 0u;        // (zero on one side keeps k-slots 4..7 empty)
        ATOM_F6_PIN(af[i]);
        ATOM_F6_PIN(bf[jb]);
        c = mfma_f6<0>(bf[jb], af[i], zf);
        ATOM_F6_PIN(c);
        if constexpr (t == T - 2) {
            if (next_stage_known) read_b(0);
        }
        if constexpr (!EARLY) {
            if constexpr (t == 0) { read_a(1); read_b(1); }
            else if constexpr (i == 0 && j + 1 < JW) read_b(j + 1);
            else if constexpr (t == T - 1) {
                if (next_stage_known) read_a(0);
            }
        }
        req(0);
        ATOM_F6_SLOT_END();
        s = scale_tile(sb[jb], sa[i]);
        ATOM_F6_PIN(s);
        req(1);
        ATOM_F6_SLOT_END();
        c = mfma_f6<1>(bf[jb], af[i], c);
        ATOM_F6_PIN(c);
        if constexpr (!EARLY) {
        } else if constexpr (t == T - 2) {
            if (next_stage_known) read_a(0);
        } else if constexpr (t == T - 1) {
            if (next_stage_known) { read_a(1); read_b(1); }
        } else if constexpr (i == 1 && (t + 3) / 2 < JW) {
            read_b((t + 3) / 2);
        }
        req(2);
        ATOM_F6_SLOT_END();
        dequant(acc[t], c, s, 0, 16);
        ATOM_F6_SLOT_END();
    };
    auto no_req = [](int) {};
    // the sub-tiles of a group before its barrier (all reads of its stage are issued by then), and those behind it
    auto head = [&](auto req) __attribute__((always_inline)) {
        subtile(integral_constant<int, 0>{}, false, [&](int q) __attribute__((always_inline)) { req(q); });
        subtile(integral_constant<int, 1>{}, false, [&](int q) __attribute__((always_inline)) { req(3 + q); });
        if constexpr (JW >= 3) {
            subtile(integral_constant<int, 2>{}, false, [&](int q) __attribute__((always_inline)) { req(6 + q); });
            subtile(integral_constant<int, 3>{}, false, [&](int q) __attribute__((always_inline)) { req(9 + q); });
        }
        if constexpr (JW >= 4) {
            subtile(integral_constant<int, 4>{}, false, [&](int q) __attribute__((always_inline)) { req(12 + q); });
            subtile(integral_constant<int, 5>{}, false, [&](int q) __attribute__((always_inline)) { req(15 + q); });
        }
    };

    int base = 0;                                              // stage of the tile's group 0
#pragma unroll
    for (int v = 0; v < NST; ++v)
#pragma unroll
        for (int k = 0; k < LPW; ++k) request_now(k, cur_t.a + (int64_t)v * IMG4, cur_t.w + (int64_t)v * IMG4, v);
#pragma unroll
    for (int k = 0; k < XTRA; ++k) dummy();
    for (;;) {
        const int nlogical = logical + lstep;
        const bool more = nlogical < lend;
        nxt_t = tile_of(more ? nlogical : logical);
        asm volatile("" : "+v"(lane_t));                       // (what only a tile's end needs is derived from these two there, and
        asm volatile("" : "+s"(wave_t));                       // holds no registers before)
        __builtin_amdgcn_s_waitcnt(wait_imm((NST - 1) * LPW + XTRA));
        __syncthreads();
#pragma unroll
        for (int t = 0; t < T; ++t) acc[t] = zf;
        cur = base;
        set_stage(cur);
        read_a(0); read_b(0);
        if constexpr (EARLY) { read_a(1); read_b(1); }
        // the first group's sub-tiles before the barrier
        head(no_req);
        const uint8_t *a_run = cur_t.a + NST * IMG4, *w_run = cur_t.w + NST * IMG4;    // the group to request next
        // One body: from the barrier of group u, two sub-tiles before its end, to that of group u + 1.  At its start stage `cur` (group u) is
        // read to the end by every wavefront and group u + 1 has landed.  MODE: what stage `cur` is refilled with: 0 group
        // u + NST, 1 / 2 the activation / weight part of the INT8 group, 3 group v of the next tile.  LAST: no group follows.
        auto body = [&](int v, auto mode_c, auto loose_c, auto last_c) __attribute__((always_inline)) {
            constexpr int MODE = decltype(mode_c)::value, LOOSE = decltype(loose_c)::value;
            constexpr bool LAST = decltype(last_c)::value;
            if constexpr (!LAST) __builtin_amdgcn_s_waitcnt(wait_imm((NST - 2) * LPW + LOOSE));
            else                 __builtin_amdgcn_s_waitcnt(wait_imm(63));
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
            const int refill = cur;
            constexpr int NSLOT = LAST ? 6 : 3 * T;
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
            subtile(integral_constant<int, T - 2>{}, !LAST, [&](int q) __attribute__((always_inline)) { req_at(q); });
            subtile(integral_constant<int, T - 1>{}, !LAST, [&](int q) __attribute__((always_inline)) { req_at(3 + q); });
            if constexpr (!LAST) head([&](int q) __attribute__((always_inline)) { req_at(6 + q); });
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

        // ---- the INT8 group: INT8 MFMA, int32 tile converted to fp32, the same dequantisation
        {
            int ck[4];                                         // byte offset of chunk 2 kk + g of row r
            const int rt = lane_t & 31, gt = lane_t >> 5;
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) ck[kk] = 128 * rt + 16 * (((2 * kk + gt) ^ rt ^ ((rt >> 3) & 1)) & 7);
            __builtin_amdgcn_s_waitcnt(wait_imm((NST - 2) * LPW));
            __syncthreads();
            const unsigned char *a8 = smem + stage8a * STAGE + wm * IMG8;
            const unsigned char *w8 = smem + stage8w * STAGE + w_unit * IMG8;
            v4i x[2][4];
            v2u xs[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) x[i][kk] = *reinterpret_cast<const v4i *>(a8 + ck[kk] + 4096 * i);
                xs[i] = *reinterpret_cast<const v2u *>(a8 + SC8 + 8 * r + 256 * i);
            }
#pragma unroll
            for (int j = 0; j < JW; ++j) {
                v4i w[4];
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) w[kk] = *reinterpret_cast<const v4i *>(w8 + ck[kk] + 4096 * w_half + (ODD ? j * IMG8 : (j >> 1) * IMG8 + (j & 1) * 4096));
                v2u ws = *reinterpret_cast<const v2u *>(w8 + SC8 + 8 * r + 256 * w_half + (ODD ? j * IMG8 : (j >> 1) * IMG8 + (j & 1) * 256));
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
        const bool vec_ok = ((reinterpret_cast<uintptr_t>(p.y) | (uintptr_t)(p.ldy * 2)) & 15) == 0;
        const int64_t m_w = 64 * (int64_t)(cur_t.au0 + wm);
        auto request_two = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < LPW; ++k) request(k, nxt_t.a + (NST - 2) * IMG4, nxt_t.w + (NST - 2) * IMG4, stage8a, more);
#pragma unroll
            for (int k = 0; k < LPW; ++k) request(k, nxt_t.a + (NST - 1) * IMG4, nxt_t.w + (NST - 1) * IMG4, stage8w, more);
        };
        // the block goes out in parts of 64 columns (JW odd: two pieces of 32, and at last one), each through the wavefront's own
        // staging area
        constexpr int PARTS = (JW + 1) / 2;
#pragma unroll
        for (int h = 0; h < PARTS; ++h) {
            const int nj = JW - 2 * h < 2 ? 1 : 2;             // column blocks of this part
            const bool last = h == PARTS - 1;
#pragma unroll
            for (int t = 4 * h; t < 4 * h + 2 * nj; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v2h lo = __builtin_convertvector((v2f{acc[t][4 * q], acc[t][4 * q + 1]}), v2h);
                    const v2h hi = __builtin_convertvector((v2f{acc[t][4 * q + 2], acc[t][4 * q + 3]}), v2h);
                    *reinterpret_cast<v2u *>(ot + (32 * (t & 1) + r) * OSTR + (32 * ((t >> 1) & 1) + 8 * q + 4 * g) * 2) =
                        v2u{__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi)};
                }
            __builtin_amdgcn_s_waitcnt(wait_imm(63));          // (LDS only: the wavefront reads what it wrote itself)
            // first columns of the part's two blocks of 32
            const int64_t n_w = 64 * (int64_t)cur_t.wu0 + 64 * w_unit + (ODD ? 128 * h + 32 * w_half : 64 * h);
            constexpr int STEP = ODD ? 64 : 32;
            uint16_t *const yb = p.y + m_w * p.ldy + n_w;
            // (the same decision in all lanes; each arm passes the one barrier)
            if (vec_ok && m_w + 64 <= p.M && n_w + (nj - 1) * STEP + 32 <= p.N) {
                const int lpr = 4 * nj, rps = 64 / lpr;        // lanes per row, rows per step
                const int lr = lane_t / lpr, lc = lane_t % lpr;
                v4i ov[8];
#pragma unroll
                for (int it = 0; it < 64 / rps; ++it) ov[it] = *reinterpret_cast<const v4i *>(ot + (it * rps + lr) * OSTR + lc * 16);
                __builtin_amdgcn_s_waitcnt(wait_imm(63));
                if (last) {
                    __syncthreads();                           // every staging area is read: the two stages are free
                    request_two();
                }
                uint16_t *const yl = yb + lr * p.ldy + (lc >> 2) * STEP + (lc & 3) * 8;
#pragma unroll
                for (int it = 0; it < 64 / rps; ++it) *reinterpret_cast<v4i *>(yl + it * rps * p.ldy) = ov[it];
            } else {
                if (m_w < p.M) {
                    const int rows = (int)(p.M - m_w < 64 ? p.M - m_w : 64);
                    if constexpr (!ODD) {
                        if (n_w < p.N) store_block_any<64, 64>(ot, OSTR, yb, p.ldy, rows, (int)(p.N - n_w < 64 ? p.N - n_w : 64), lane_t);
                    } else {
                        for (int x = 0; x < nj; ++x) {
                            const int64_t n_x = n_w + STEP * x;
                            if (n_x < p.N) store_block_any<64, 32>(ot + 64 * x, OSTR, yb + STEP * x, p.ldy, rows, (int)(p.N - n_x < 32 ? p.N - n_x : 32), lane_t);
                        }
                    }
                }
                if (last) {
                    __syncthreads();
                    __builtin_amdgcn_s_waitcnt(wait_imm(0));
                    request_two();
#pragma unroll
                    for (int k = 0; k < XTRA; ++k) dummy();
                }
            }
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

template <int WM, int WN, int JW>
hipError_t launch_cfg(const F6Params &p, hipStream_t stream)
{
    using Gm = Walk<WM, WN, JW>;
    auto kern = &w4a4_gemm_f6_walk_kernel<WM, WN, JW>;
    static atom_launch::LdsOptIn opt_in;   // one attribute call per kernel variant and device
    hipError_t err = atom_launch::ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(kern), Gm::LDS);
    if (err != hipSuccess) return err;
    const int64_t tiles = (int64_t)((p.a_units + WM - 1) / WM) * ((p.w_units + Gm::NJ - 1) / Gm::NJ);
    const int64_t slots = (int64_t)atom_launch::compute_units() * (2 * Gm::LDS <= 160 * 1024 ? 2 : 1);
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles < slots ? tiles : slots)), dim3(Gm::NT), Gm::LDS, stream, p);
    return hipGetLastError();
}

}  // namespace

namespace atom_gemm_f6 {

hipError_t launch_walk(const F6Params &p, int tile, hipStream_t stream)
{
    switch (tile) {
    case 0:  return launch_cfg<2, 2, 2>(p, stream);
    case 1:  return launch_cfg<4, 2, 2>(p, stream);
    case 2:  return launch_cfg<4, 2, 3>(p, stream);
    case 3:  return launch_cfg<2, 4, 3>(p, stream);
    case 4:  return launch_cfg<4, 2, 4>(p, stream);
    case 5:  return launch_cfg<3, 2, 2>(p, stream);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace atom_gemm_f6
