// The packed group GEMM (atom_gemm_f6.hip: operands, unit images, exactness) for launches of few tiles.
//
// What bounds such a launch is not a pipe but what a wavefront can issue: with one wavefront per SIMD a step of the 128 x 128
// tile took 1020 cycles for 420 cycles of MFMAs, whatever was prefetched how far ahead, and tiles of 128 rows leave most
// compute units idle (M = 256, N = 4096: 64 tiles).  So here
//   * tiles are small (64 x 32 to 128 x 128) and a wavefront's block is 32 rows x 32 NJ columns, which puts up to two
//     wavefronts on every SIMD from one workgroup (four wavefronts and two workgroups for 64 x 64);
//   * a step's fragments are all in registers when it starts and the next group's are read meanwhile into a second
//     set, so nothing waits for LDS, and the stage just read is free at once;
//   * the loop is unrolled over the LDS stages, so that every LDS address is a register plus an immediate and a
//     request is one scalar addition and the load: 13 scalar instructions per step instead of 42.
// K = 4096, weights from HBM, general kernel and this one: M = 256, N = 4096 21.0 -> 11.7 us (64 x 64); M = 512, N = 4096
// 20.9 -> 15.3 us (64 x 128); M = 256, N = 12288 23.2 -> 21.0 us, M = 128, N = 22016 25.1 -> 22.9 us (128 x 128).
// Which tile a launch gets: pick_tile in atom_gemm_f6.hip, and launch_thin for the columns of the smaller two.

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include <type_traits>

#include "atom_gemm_f6.h"
#include "atom_launch.h"

namespace {

using namespace atom_gemm_f6;

template <int WR, int WC, int NJ, int STAGES>
struct Thin {
    static constexpr int NW    = WR * WC;
    static constexpr int NT    = 64 * NW;
    static constexpr int HW    = WC * NJ;                     // the tile's columns in half units
    static constexpr bool ODD  = HW % 2 == 1;                 // weights staged as halves of units instead of whole ones
    static constexpr int UA    = WR / 2;
    static constexpr int APART = round_kb(UA * IMG4);         // activation part of a stage, in whole requests
    static constexpr int WPART = round_kb(HW * (IMG4 / 2));
    static constexpr int STAGE = APART + WPART;
    static constexpr int NST   = STAGES;
    static constexpr int NA    = APART / 1024, NB = WPART / 1024;
    static constexpr int KA    = (NA + NW - 1) / NW, KB = (NB + NW - 1) / NW;          // requests per wavefront and stage
    static constexpr int LPW   = KA + KB;
    static constexpr int NA8   = round_kb(UA * IMG8) / 1024, NB8 = round_kb(HW * (IMG8 / 2)) / 1024;
    static constexpr int SPARE = NST * STAGE;                 // 16 bytes that are written and never read
    static constexpr int LDS   = SPARE + 64;
    static constexpr int OSTR  = 64 * NJ + 16;                // output staging: bytes per row of a wavefront's block
    static_assert(1024 * NA8 <= STAGE && 1024 * NB8 <= STAGE, "a part of the INT8 group fits a stage");
    static_assert(NA8 <= LPW * NW && NB8 <= LPW * NW, "a part of the INT8 group is one stage's requests");
    static_assert(NST % 2 == 0 && NST >= 4, "two fragment sets, two parts of the INT8 group");
    static_assert(NW * 32 * OSTR <= LDS && LDS <= 160 * 1024 && (NST - 1) * LPW <= 63, "LDS, vmcnt");
};

template <int WR, int WC, int NJ, int STAGES, int OCC>
__global__ __launch_bounds__(WR * WC * 64, OCC)
void w4a4_gemm_f6_thin_kernel(const F6Params p)
{
    using Gm = Thin<WR, WC, NJ, STAGES>;
    constexpr int NW = Gm::NW, NST = Gm::NST, STAGE = Gm::STAGE, LPW = Gm::LPW, UA = Gm::UA, HW = Gm::HW;
    constexpr int APART = Gm::APART, KA = Gm::KA;
    constexpr bool ODD = Gm::ODD;
    using std::integral_constant;

    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave % WR, wc = wave / WR;
    const int r = lane & 31, g = lane >> 5;
    const int G4 = p.G4;

    // M-tiles fastest, in bands of eight; the last tile of a row or column of tiles is moved back so that it is whole (what
    // two tiles share they both compute, to the same bits)
    const int TM = (p.a_units + UA - 1) / UA, TN = (2 * p.w_units + HW - 1) / HW;
    const int logical = xcd_contiguous_block_id();
    const int band = 8 * TN, bb = logical / band, rem = logical - bb * band;
    const int hgt = TM - 8 * bb < 8 ? TM - 8 * bb : 8;
    const int tm = 8 * bb + rem % hgt, tn = rem / hgt;
    const int au0 = tm * UA < p.a_units - UA ? tm * UA : p.a_units - UA;
    const int hw0 = tn * HW < 2 * p.w_units - HW ? tn * HW : 2 * p.w_units - HW;        // first half unit of weights
    const int wu0 = hw0 >> 1;
    const uint8_t *a_ptr = p.a_pk + (int64_t)au0 * p.ustride, *w_ptr = p.w_pk + (int64_t)wu0 * p.ustride;

    // ---- loader: the activation (weight) part of a stage is the units' images one behind the other; piece j of a
    // part is its bytes [1024 j, 1024 j + 1024), moved by wavefront j % NW; lanes past the end of the part
    // repeat its last 16 bytes (they land in the padding)
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(smem), spare = lds0 + Gm::SPARE;
    uint32_t voff[LPW];
    auto part_off = [&](int j, int units, int img) __attribute__((always_inline)) -> uint32_t {
        int q = 64 * j + lane;                                 // 16-byte chunk of the part
        q = q < units * (img / 16) ? q : units * (img / 16) - 1;
        const int unit = q / (img / 16);
        return (uint32_t)unit * (uint32_t)p.ustride + 16u * (q - unit * (img / 16));
    };
    // An odd number of half units: each half's codes and behind them its scales.  In an image they are the lower or upper half of every
    // piece of 1024 bytes (INT8: of 8192) of the codes and of the 512 bytes of scales.
    auto half_off = [&](int j, int img) __attribute__((always_inline)) -> uint32_t {
        const int codes = img == IMG4 ? SC4 : SC8, run = img == IMG4 ? 512 : 4096;
        int q = 64 * j + lane;                                 // 16-byte chunk of the part
        q = q < HW * (img / 32) ? q : HW * (img / 32) - 1;
        const int half = q / (img / 32), b = 16 * (q - half * (img / 32)), hw = (hw0 & 1) + half;
        return (uint32_t)(hw >> 1) * (uint32_t)p.ustride +
               (b < codes / 2 ? (uint32_t)(b / run * (2 * run) + run * (hw & 1) + b % run) : (uint32_t)(codes + 256 * (hw & 1) + b - codes / 2));
    };
    auto weight_off = [&](int j, int img) __attribute__((always_inline)) -> uint32_t {
        if constexpr (ODD) return half_off(j, img);
        else return part_off(j, HW / 2, img);
    };
#pragma unroll
    for (int k = 0; k < LPW; ++k)
        voff[k] = k < KA ? part_off(wave + NW * k, UA, IMG4) : weight_off(wave + NW * (k - KA), IMG4);
    // request k of a group whose images start `ahead` bytes behind a_ptr / w_ptr, into `stage`
    auto request = [&](int k, int ahead, int stage) __attribute__((always_inline)) {
        const bool act = k < KA;
        const int kk = act ? k : k - KA, n = act ? Gm::NA : Gm::NB, j = wave + NW * kk;
        const uint8_t *base = (act ? a_ptr : w_ptr) + ahead;
        const uint32_t dst = lds0 + stage * STAGE + (act ? 0 : APART) + 1024 * j;
        if (NW * (kk + 1) <= n) dma16(dst, voff[k], base);
        else dma16_masked(j < n ? dst : spare, voff[k], base, j < n ? ~0ull : 1ull);   // (no such piece: one lane, never read)
    };
    // request k of a part of the INT8 group, into `stage`
    auto request8 = [&](int k, int stage, bool act) __attribute__((always_inline)) {
        const int j = wave + NW * k, n = act ? Gm::NA8 : Gm::NB8;
        const uint8_t *base = (act ? p.a_pk + (int64_t)au0 * p.ustride : p.w_pk + (int64_t)wu0 * p.ustride) + (int64_t)G4 * IMG4;
        if (NW * k >= n) dma16_masked(spare, 0u, base, 1ull);
        else dma16_masked(j < n ? lds0 + stage * STAGE + 1024 * j : spare, act ? part_off(j, UA, IMG8) : weight_off(j, IMG8), base, j < n ? ~0ull : 1ull);
    };

    // ---- fragments
    const uint32_t lane_off = lds0 + 1024 * g + 16 * r;
    const int cb = wc * NJ;                                    // the wavefront's first block of 32 columns
    const uint32_t a_off = (wr >> 1) * IMG4 + 512 * (wr & 1) + lane_off;
    const uint32_t b_off = ODD ? lds0 + APART + cb * (IMG4 / 2) + 512 * g + 16 * r : APART + (cb >> 1) * IMG4 + 512 * (cb & 1) + lane_off;
    const uint32_t sa_off = lds0 + (wr >> 1) * IMG4 + 256 * (wr & 1) + SC4 + 8 * r;
    const uint32_t sb_off = ODD ? lds0 + APART + cb * (IMG4 / 2) + SC4 / 2 + 8 * r : lds0 + APART + (cb >> 1) * IMG4 + 256 * (cb & 1) + SC4 + 8 * r;
    typedef __attribute__((address_space(3))) const v4i *lds_v4i;
    typedef __attribute__((address_space(3))) const v2u *lds_v2u;
    auto read_pair = [&](uint32_t addr, int piece) __attribute__((always_inline)) -> v12i {
        const v4i c0 = *(lds_v4i)(uintptr_t)(addr);
        const v4i c1 = *(lds_v4i)(uintptr_t)(addr + piece);
        const v4i c2 = *(lds_v4i)(uintptr_t)(addr + 2 * piece);
        const v8i lo = __builtin_shufflevector(c0, c1, 0, 1, 2, 3, 4, 5, 6, 7);
        const v8i hi = __builtin_shufflevector(c2, c2, 0, 1, 2, 3, -1, -1, -1, -1);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11);
    };
    struct Frag { v12i a, b[NJ]; v2u sa, sb[NJ]; };
    auto read_frag = [&](int stage, Frag &f) __attribute__((always_inline)) {
        const uint32_t o = stage * STAGE;
        f.a = read_pair(a_off + o, 2048);
        f.sa = *(lds_v2u)(uintptr_t)(sa_off + o);
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            f.b[j] = read_pair(b_off + o + (ODD ? IMG4 / 2 : 512) * j, ODD ? 1024 : 2048);
            f.sb[j] = *(lds_v2u)(uintptr_t)(sb_off + o + (ODD ? IMG4 / 2 : 256) * j);
        }
    };

    v16f acc[NJ];
    const v16f zf = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    v16f c[2] = {zf, zf}, s[2] = {zf, zf};
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[j] = zf;
    auto scale_tile = [&](v2u tw, v2u tx) __attribute__((always_inline)) -> v16f {
        return __builtin_amdgcn_mfma_f32_32x32x8f16(__builtin_bit_cast(v4h, tw), __builtin_bit_cast(v4h, tx), zf, 0, 0, 0);
    };
    auto dequant = [&](v16f &a, const v16f &cc, const v16f &ss, int e0, int e1) __attribute__((always_inline)) {
#pragma unroll
        for (int e = e0; e < e1; ++e) a[e] = fmaf(cc[e], ss[e], a[e]);
        ATOM_F6_PIN(a);
    };

    // ---- One step: a group in stage ST whose fragments are in registers (set ST % 2).  The next group, in the next stage, is
    // read into the other set meanwhile, and stage ST, which everyone has read before the barrier, is refilled.  MODE: 0 the
    // group NST further on, 1 / 2 a part of the INT8 group, 3 nothing, 4 nothing and nothing to read (the last step).
    // WAIT: requests that may be outstanding when the next group has landed.
    Frag f[2];
    auto step = [&](auto st_c, auto mode_c, auto wait_c) __attribute__((always_inline)) {
        constexpr int ST = decltype(st_c)::value, MODE = decltype(mode_c)::value, WAIT = decltype(wait_c)::value;
        if constexpr (MODE != 4) {
            __builtin_amdgcn_s_waitcnt(wait_imm(WAIT));
            __syncthreads();
            __builtin_amdgcn_sched_barrier(0);
            read_frag((ST + 1) % NST, f[(ST + 1) % 2]);
        }
        Frag &x = f[ST % 2];
        auto req_at = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < LPW; ++k)
                if (k * 3 * NJ / LPW == slot) {
                    if constexpr (MODE == 0)      request(k, NST * IMG4, ST);
                    else if constexpr (MODE == 1) request8(k, ST, true);
                    else if constexpr (MODE == 2) request8(k, ST, false);
                }
        };
#pragma unroll
        for (int j = 0; j < NJ; ++j) x.sb[j][0] = g == 0 ? x.sb[j][0] : 0u;            // (zero on one side keeps k-slots 4..7 empty)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int q = NJ == 2 ? j : ST % 2, pj = NJ == 2 ? j ^ 1 : 0;
            ATOM_F6_PIN(x.a);
            ATOM_F6_PIN(x.b[j]);
            c[q] = mfma_f6<0>(x.b[j], x.a, zf);
            ATOM_F6_PIN(c[q]);
            req_at(3 * j);
            dequant(acc[pj], c[q ^ 1], s[q ^ 1], 0, 4);
            ATOM_F6_SLOT_END();
            s[q] = scale_tile(x.sb[j], x.sa);
            ATOM_F6_PIN(s[q]);
            req_at(3 * j + 1);
            dequant(acc[pj], c[q ^ 1], s[q ^ 1], 4, 10);
            ATOM_F6_SLOT_END();
            c[q] = mfma_f6<1>(x.b[j], x.a, c[q]);
            ATOM_F6_PIN(c[q]);
            req_at(3 * j + 2);
            dequant(acc[pj], c[q ^ 1], s[q ^ 1], 10, 16);
            ATOM_F6_SLOT_END();
        }
        if constexpr (MODE == 0) { a_ptr += IMG4; w_ptr += IMG4; }
    };

    // The first group goes to the stage from which the steps with a group to request end at the last stage: what
    // follows them then starts at stage 0, and every stage number is known at compile time.
    const int n = G4 - NST, first = (NST - n % NST) % NST;
#pragma unroll
    for (int v = 0; v < NST; ++v) {
        int st = first + v;
        st = st < NST ? st : st - NST;
#pragma unroll
        for (int k = 0; k < LPW; ++k) request(k, v * IMG4, st);
    }
    __builtin_amdgcn_s_waitcnt(wait_imm((NST - 1) * LPW));
    __syncthreads();
    constexpr integral_constant<int, (NST - 2) * LPW> kWait{};
    auto steps = [&](auto self, auto st_c, int from) __attribute__((always_inline)) -> void {
        constexpr int ST = decltype(st_c)::value;
        if constexpr (ST < NST) {
            if (ST == from && from != 0) read_frag(ST, f[ST % 2]);                     // (the very first group)
            if (ST >= from) step(st_c, integral_constant<int, 0>{}, kWait);
            self(self, integral_constant<int, ST + 1>{}, from);
        }
    };
    if (first != 0) steps(steps, integral_constant<int, 0>{}, first);
    else            read_frag(0, f[0]);
    for (int u = n / NST; u > 0; --u) steps(steps, integral_constant<int, 0>{}, 0);
    // (n groups requested since: NST steps are left)
    auto rest = [&](auto self, auto q_c) __attribute__((always_inline)) -> void {
        constexpr int q = decltype(q_c)::value;
        if constexpr (q < NST) {
            step(q_c, integral_constant<int, q == NST - 1 ? 4 : q == 0 ? 1 : q == 1 ? 2 : 3>{},
                 integral_constant<int, q <= NST - 2 ? (NST - 2 - q + (q < 2 ? q : 2)) * LPW : 0>{});
            self(self, integral_constant<int, q + 1>{});
        }
    };
    rest(rest, integral_constant<int, 0>{});
    dequant(acc[NJ - 1], c[1], s[1], 0, 16);                   // (NST is even: the last step's last result tile is number 1)
    constexpr int stage8a = 0, stage8w = 1;

    // ---- the INT8 group
    {
        __builtin_amdgcn_s_waitcnt(wait_imm(0));
        __syncthreads();
        const unsigned char *a8 = smem + stage8a * STAGE + (wr >> 1) * IMG8, *w8 = smem + stage8w * STAGE + (ODD ? cb * (IMG8 / 2) : (cb >> 1) * IMG8);
        const v2u xs = *reinterpret_cast<const v2u *>(a8 + SC8 + 8 * r + 256 * (wr & 1));
        int ck[4];                                             // byte offset of chunk 2 kk + g of row r
        v4i x[4];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            ck[kk] = 128 * r + 16 * (((2 * kk + g) ^ r ^ ((r >> 3) & 1)) & 7);
            x[kk] = *reinterpret_cast<const v4i *>(a8 + 4096 * (wr & 1) + ck[kk]);
        }
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
            const int half = (cb + j) & 1;
            const unsigned char *const wj = w8 + (ODD ? j * (IMG8 / 2) : 4096 * half);
            v2u ws = *reinterpret_cast<const v2u *>(ODD ? wj + SC8 / 2 + 8 * r : w8 + SC8 + 8 * r + 256 * half);
            ws[0] = g == 0 ? ws[0] : 0u;
            v16i ci = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
                ci = __builtin_amdgcn_mfma_i32_32x32x32_i8(*reinterpret_cast<const v4i *>(wj + ck[kk]), x[kk], ci, 0, 0, 0);
            const v16f ss = scale_tile(ws, xs);
            v16f cf;
#pragma unroll
            for (int e = 0; e < 16; ++e) cf[e] = (float)ci[e];
            dequant(acc[j], cf, ss, 0, 16);
        }
    }
    __syncthreads();

    // ---- store: a lane holds four consecutive columns of one row of Y at a time (the weights are the row operand of the
    // MFMA); through LDS so that global memory sees whole row pieces
    constexpr int OSTR = Gm::OSTR;
    unsigned char *ot = smem + wave * (32 * OSTR);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const v2h lo = __builtin_convertvector((v2f{acc[j][4 * q], acc[j][4 * q + 1]}), v2h);
            const v2h hi = __builtin_convertvector((v2f{acc[j][4 * q + 2], acc[j][4 * q + 3]}), v2h);
            *reinterpret_cast<v2u *>(ot + r * OSTR + (32 * j + 8 * q + 4 * g) * 2) =
                v2u{__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi)};
        }
    __builtin_amdgcn_s_waitcnt(wait_imm(63));                  // (LDS only: the wavefront reads what it wrote itself)
    store_block<32, 32 * NJ, true>(ot, OSTR, p.y, p.ldy, (int64_t)au0 * 64 + 32 * wr, (int64_t)(hw0 + cb) * 32, p.M, p.N, lane);
}

template <int WR, int WC, int NJ, int STAGES, int OCC>
hipError_t launch_cfg(const F6Params &p, hipStream_t stream)
{
    using Gm = Thin<WR, WC, NJ, STAGES>;
    auto kern = &w4a4_gemm_f6_thin_kernel<WR, WC, NJ, STAGES, OCC>;
    static atom_launch::LdsOptIn opt_in;   // one attribute call per kernel variant and device
    hipError_t err = atom_launch::ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(kern), Gm::LDS);
    if (err != hipSuccess) return err;
    const int64_t tiles = (int64_t)((p.a_units + Gm::UA - 1) / Gm::UA) * ((2 * p.w_units + Gm::HW - 1) / Gm::HW);
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(Gm::NT), Gm::LDS, stream, p);
    return hipGetLastError();
}

}  // namespace

namespace atom_gemm_f6 {

// What a compute unit can have in flight is bounded, so from memory a step costs what its tile fetches (a unit of 64 rows or columns is
// 6.6 KB of a group) and more stages help as far as about 60 KB of requests.  Hence, of a launch of up to one tile per compute unit, the smallest
// tile that keeps it one: 64 x 64 becomes 64 x 32 where there are compute units for twice the tiles, 64 x 128 becomes 64 x 96.
// Weights from HBM, us, 64 x 64 with four stages and 64 x 32 with six: M = 128, K = 4096, N = 4096 10.9 -> 9.0; K = 11008, N = 4096 24.3 -> 18.5; K =
// 8192, N = 1000 (256 rows) 16.3 -> 12.9; out of the last-level cache 7.9 -> 7.6, 16.8 -> 14.4, 12.6 -> 11.5.  64 x 96 for 64 x 128: M = 320, K = 11008,
// N = 4096 31.3 -> 28.9; M = 128, K = 8192, N = 10000 27.2 -> 25.1.  64 x 64 with six stages for four: M = 256, K = 4096, N = 4096 11.1 -> 10.5; K =
// 11008 24.6 -> 23.0.  Six stages are also longer code to fetch, 0.4 us, which fewer groups don't repay: from the cache K = 2048, N = 3000 5.6 -> 5.85 (64 x 32)
// and 5.8 -> 6.4 (64 x 64), K = 1280, N = 4096 4.7 -> 5.0 and 4.9 -> 5.3, K = 2560 6.1 -> 6.1 and 6.3 -> 6.7; from HBM 7.0 -> 6.3 and 7.1 -> 6.9, 5.6 -> 5.3
// and 5.7 -> 5.7, 8.0 -> 7.0 and 8.1 -> 7.9.  What HBM gives these two beyond 64 x 32 is little or less than nothing out of the last-level cache, so they stand
// where neither loses: 64 x 64 with six stages from 47 groups on (front end and GEMM, warm: M = 192, K = 5120, N = 4096 13.7 -> 14.0; K = 6144 16.0 -> 16.0, K = 11008 24.3 -> 24.0), 64
// x 96 from 31 groups on up to seven eighths of the compute units (M = 320, K = 5120, N = 4096 18.1 -> 17.7, M = 128, K = 4096, N = 9000 14.6 -> 14.4; but K = 3072, M = 300, N =
// 4500 14.5 -> 14.9, K = 5120, M = 65, N = 12288, 256 tiles, 17.4 -> 17.8).  128 x 96 on twelve wavefronts for 128 x 128 spilled and was 1.04 to 1.08 of it at K = 4096, 5120.
static int thin_form(int64_t au, int64_t wu, int64_t G4, int tile, int64_t cus)
{
    const int64_t t64 = au * wu, t96 = au * ((2 * wu + 2) / 3);
    if (tile == 0) return G4 >= 15 && 2 * t64 <= cus ? 326 : G4 >= 47 && t64 <= cus ? 646 : 644;
    if (tile == 1) return G4 >= 31 && t96 <= cus - cus / 8 ? 964 : 1284;
    return 0;
}

hipError_t launch_thin(const F6Params &p, int tile, hipStream_t stream)
{
    switch (thin_form(p.a_units, p.w_units, p.G4, tile, atom_launch::compute_units())) {
    case 326:  return launch_cfg<2, 1, 1, 6, 2>(p, stream);
    case 646:  return launch_cfg<2, 2, 1, 6, 2>(p, stream);
    case 644:  return launch_cfg<2, 2, 1, 4, 3>(p, stream);
    case 964:  return launch_cfg<2, 3, 1, 4, 2>(p, stream);
    case 1284: return launch_cfg<2, 4, 1, 4, 2>(p, stream);
    default:   return launch_cfg<4, 2, 2, 4, 2>(p, stream);
    }
}

}  // namespace atom_gemm_f6

// The columns and stages of a tile of 64 rows (0: 64 x 64, 1: 64 x 128), 10 times the one and the other, as their test asks it.
extern "C" int atom_internal_packed_thin_form(int64_t M, int64_t N, int32_t K, int32_t tile, int64_t cus)
{
    return atom_gemm_f6::thin_form((M + 63) / 64, (N + 63) / 64, (K - 128) >> 7, tile, cus);
}
