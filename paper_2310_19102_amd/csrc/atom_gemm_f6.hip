// Group GEMM on pre-tiled operands with the INT4 groups carried in FP6 (Section 4.2 of the
// paper, steps 1-3; the arithmetic is that of atom_gemm.hip).
//
// gfx950 has no INT4 matrix instruction, and on the INT8 one a 4-bit code costs as much as an
// 8-bit code.  It does have v_mfma_f32_32x32x64_f8f6f4, which runs FP6 operands at twice the INT8
// rate, and the E3M2 variant of FP6 represents every integer in [-8, 8] exactly.  An INT4 code is
// therefore re-encoded (not re-quantised) as the E3M2 number of the same value; the products of a
// group are integers of at most 7 bits, their sum over the 128 channels of a group is below 2^14,
// and the instruction's fp32 accumulation of such values is exact (checked on the hardware against
// integer sums, with accumulator inputs up to 2^23).  So the fp32 result tile IS the group's
// integer partial sum P[m, n, g], and step 2 needs no integer-to-float conversion: one fused
// multiply-add per element and group against the tile of scale products.  The 128 outlier channels
// stay INT8 on the INT8 MFMA.
//
// Operands come in an opaque tiled layout (pack_rows_kernel below writes it, from the canonical
// q4 / q8 / scale arrays; weights once, offline; activations per call into the workspace).  A
// "unit" is 64 rows; for every unit the images of its groups follow each other, each image being
// byte for byte what one LDS stage holds for that unit and group, so the K loop's loader is a
// linear copy global -> LDS by global_load_lds_dwordx4 (no registers, no address arithmetic, whole
// cache lines).
//   INT4 group image, 6656 bytes: lane (row r, half g) of the two FP6 MFMAs of a group holds the
//     channels 32 g .. 32 g + 31 (first MFMA) and 64 + 32 g .. 64 + 32 g + 31 (second) of its row:
//     2 x 24 = 48 bytes of FP6, stored as three 16-byte chunks c = 0, 1, 2 at
//     2048 c + 1024 g + 16 r, so that one 128-bit fragment read of a wavefront is one contiguous
//     kilobyte (bank-conflict free) and every address of a step is the lane's base plus an
//     immediate; the fp16 scale of row r, zero-extended to 64 bits (the operand of the fp16 MFMA
//     that forms the scale products: the scale in its first element, zeros behind), at 6144 + 8 r.
//   INT8 group image, 8704 bytes: 16-byte chunk c of row r at 128 r + 16 ((c ^ r ^ (r/8 % 2)) % 8),
//     scale at 8192 + 8 r.
// Rows past the end of the matrix hold zero codes and zero scales.
//
// Three GEMM kernels share this layout and arithmetic, and give the same bits: groups are added in ascending
// order, the INT8 group(s) last, each by one fmaf: the accumulation chain of the definition.
//   atom_gemm_f6_thin.hip: launches of few tiles (one row of 32 x 32 blocks per wavefront).
//   atom_gemm_f6_walk.hip: launches of many tiles (64 x 64 per wavefront, workgroups that walk tiles).
//   w4a4_gemm_f6_kernel below: everything those two do not take (several INT8 groups, fewer than seven
//     INT4 groups) and the dump of the integer sums.  256 x 128 (or 128 x 128, 64 x 128) tile, wavefront tile 64 x 64 = four
//     32 x 32 sub-tiles, NST LDS stages.  Per INT4 group and sub-tile: two FP6 MFMAs (64 channels each) and one
//     fp16 MFMA that forms the 32 x 32 tile of scale products a_scale[m] * w_scale[n] (rank 1, exact in fp32), then 16
//     fused multiply-adds per lane.

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include <type_traits>

#include "atom_gemm_f6.h"
#include "atom_internal.h"
#include "atom_launch.h"

namespace {

using namespace atom_gemm_f6;

// ------------------------------------------------------------------------------------------
// Packing: canonical rows -> unit images.
// ------------------------------------------------------------------------------------------
struct PackParams {
    const uint8_t *q4; const int8_t *q8; const uint16_t *scale;
    uint8_t *out;
    int64_t rows;                         // valid rows
    int     units, G4, G8, O;
    int64_t ustride;                      // bytes per unit = G4 * IMG4 + G8 * IMG8
};

// The 32 codes of 16 bytes as FP6 E3M2 numbers: a code with its top bit flipped is 8 more than its value and, in the mantissa of
// an fp16 number of exponent 10, reads as 1032 more; the conversion is a plain one (scale 1, every code is representable).
__device__ __forceinline__ v6u codes_to_fp6(const v4u &w)
{
    typedef unsigned v16u __attribute__((ext_vector_type(16)));
    v16u h;
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        const uint32_t even = w[d] & 0x0F0F0F0Fu, odd = (w[d] >> 4) & 0x0F0F0F0Fu;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t pair = __builtin_amdgcn_perm(odd, even, 0x0C000C00u | (unsigned)i | (unsigned)(4 + i) << 16);
            h[4 * d + i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(v2h, pair ^ 0x64086408u) - v2h{(_Float16)1032.0f, (_Float16)1032.0f});
        }
    }
    return __builtin_amdgcn_cvt_scalef32_pk32_bf6_f16(__builtin_bit_cast(v32h, h), 1.0f);
}

// One workgroup: NG INT4 groups of a unit, or one INT8 group of it.  Bound by memory where there is much of it (4.2 to 5.5 TB/s read and written).
// 4 NG lanes read the 64 NG bytes that a row has in those groups; the images are put together in LDS and leave as whole kilobytes.  (A
// workgroup per group whose lanes took a row each read half a line of every row, and the other half was fetched by another XCD.)  Before
// and now, us: 57344 x 8192 172.2, 114.7; 13824 x 5120 27.3, 22.5; 4096 x 28672 44.7, 34.4; 4096 x 8192 16.1, 12.8; 1024 x 4096 4.5, 4.1.
// The units of a second operand, if any, follow the first one's (grid.y).
template <int NG>
__global__ __launch_bounds__(256)
void pack_rows_kernel(const PackParams first, const PackParams second_op)
{
    const bool two = (int)blockIdx.y >= first.units;           // the same decision in every lane
    const PackParams &p = two ? second_op : first;
    constexpr int LPR = 4 * NG, RPL = 256 / LPR, NL = 64 / RPL;       // lanes per row, rows per load, loads
    __shared__ __align__(16) unsigned char img[NG * IMG4];
    const int     G    = p.G4 + p.G8, parts = (p.G4 + NG - 1) / NG;
    const int64_t K4h  = (int64_t)p.G4 * 64;          // bytes of a canonical q4 row
    const int     unit = (int)blockIdx.y - (two ? first.units : 0), t = threadIdx.x;
    const int64_t m0   = (int64_t)unit * 64;
    uint8_t *const uout = p.out + (int64_t)unit * p.ustride;
    if ((int)blockIdx.x < parts) {
        const int g0 = NG * blockIdx.x, ng = p.G4 - g0 < NG ? p.G4 - g0 : NG;
        // thread t: rows t / LPR + RPL j, piece t % LPR of the row (four per group: 32 consecutive channels, 16 canonical bytes,
        // 24 bytes of FP6; piece q of a group is half q % 2 of MFMA q / 2)
        const int row = t / LPR, gi = (t >> 2) % NG, half = t & 1, second = (t >> 1) & 1;
        const bool here = gi < ng;
        v4u w[NL];
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const int64_t m = m0 + row + RPL * j;
            w[j] = v4u{0u, 0u, 0u, 0u};
            if (here && m < p.rows) w[j] = *reinterpret_cast<const v4u *>(p.q4 + m * K4h + (int64_t)g0 * 64 + 16 * (t % LPR));
        }
        const int srow = t / NG, sg = t % NG;
        uint32_t sbits = 0;
        if (srow < 64 && sg < ng && m0 + srow < p.rows) sbits = p.scale[(m0 + srow) * G + g0 + sg];
        unsigned char *const dst = img + gi * IMG4 + 1024 * half;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            const v6u f = codes_to_fp6(w[j]);
            unsigned char *const d = dst + 16 * (row + RPL * j);
            // the first MFMA's 24 bytes: chunk 0 and the front of chunk 1; the second's: the back of chunk 1 and chunk 2
            *reinterpret_cast<v4u *>(d + (second ? 4096 : 0)) = second ? v4u{f[2], f[3], f[4], f[5]} : v4u{f[0], f[1], f[2], f[3]};
            *reinterpret_cast<v2u *>(d + 2048 + (second ? 8 : 0)) = second ? v2u{f[0], f[1]} : v2u{f[4], f[5]};
        }
        if (srow < 64) *reinterpret_cast<v2u *>(img + sg * IMG4 + SC4 + 8 * srow) = v2u{sbits, 0u};
        __syncthreads();
        uint8_t *const out = uout + (int64_t)g0 * IMG4;
        for (int i = t; i < ng * (IMG4 / 16); i += 256)
            *reinterpret_cast<v4u *>(out + 16 * i) = *reinterpret_cast<const v4u *>(img + 16 * i);
    } else {
        // two chunks per thread: chunk ids t and t + 256 of the 512; row id / 8, slot id % 8
        const int g8 = blockIdx.x - parts;
        uint8_t *const out = uout + (int64_t)p.G4 * IMG4 + (int64_t)g8 * IMG8;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int id = t + 256 * half, row = id >> 3, slot = id & 7;
            const int chunk = (slot ^ row ^ ((row >> 3) & 1)) & 7;
            const int64_t m = m0 + row;
            v4u w = {0u, 0u, 0u, 0u};
            uint32_t sbits = 0;
            if (m < p.rows) {
                w = *reinterpret_cast<const v4u *>(p.q8 + m * p.O + (int64_t)g8 * 128 + chunk * 16);
                sbits = p.scale[m * G + p.G4 + g8];
            }
            *reinterpret_cast<v4u *>(out + 16 * id) = w;
            if (slot == 0) *reinterpret_cast<v2u *>(out + SC8 + 8 * row) = v2u{sbits, 0u};
        }
    }
}

// ------------------------------------------------------------------------------------------
// The GEMM
// ------------------------------------------------------------------------------------------
template <int WM>
struct F6Geom {
    static constexpr int NWAVE = WM * 2;
    static constexpr int NT    = NWAVE * 64;
    static constexpr int NST   = WM == 4 ? 4 : 3;                 // LDS stages
    static constexpr int APART = round_kb(WM * IMG4);              // activation units of a stage (padded to whole DMA instructions)
    static constexpr int STAGE = APART + round_kb(2 * IMG4);
    static constexpr int NA    = APART / 1024, NI = STAGE / 1024; // DMA instructions per stage: NA for activations
    static constexpr int LPW   = (NI + NWAVE - 1) / NWAVE;        // at most, per wavefront
    static constexpr int APART8 = round_kb(WM * IMG8);
    static constexpr int STAGE8 = APART8 + round_kb(2 * IMG8);
    static constexpr int NA8   = APART8 / 1024, NI8 = STAGE8 / 1024;
    static constexpr int LPW8  = (NI8 + NWAVE - 1) / NWAVE;
    static constexpr int OSTRIDE = 144;                            // output staging: bytes per row of a wavefront's 64 x 64 fp16 tile
    static constexpr int OUT   = NWAVE * 64 * OSTRIDE;
    static constexpr int SPARE = NST * STAGE;                      // a kilobyte that is written and never read
    static constexpr int LDS0  = NST * STAGE + 1024 > STAGE8 ? NST * STAGE + 1024 : STAGE8;
    static constexpr int LDS   = LDS0 > OUT ? LDS0 : OUT;
};

template <int WM, bool DBG>
__global__ __launch_bounds__(WM * 128, 2)
void w4a4_gemm_f6_kernel(const F6Params p)
{
    using Gm = F6Geom<WM>;
    constexpr int NWAVE = Gm::NWAVE, NST = Gm::NST, STAGE = Gm::STAGE, APART = Gm::APART;
    constexpr int NA = Gm::NA, NI = Gm::NI, LPW = Gm::LPW;

    extern __shared__ __align__(16) unsigned char smem[];

    const int tid  = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int r = lane & 31, g = lane >> 5;

    const int G4 = p.G4;
    // tile of this workgroup: M-tiles fastest, in bands of up to eight M-tiles so that the tiles an
    // XCD works on at one time share both activation and weight units in its L2
    const int TM = (p.a_units + WM - 1) / WM, TN = (p.w_units + 1) / 2;
    const int logical = xcd_contiguous_block_id();
    constexpr int LPWc = Gm::LPW;
    struct Tile {
        int a_valid, w_valid;
        const uint8_t *a_tile, *w_tile;
        int64_t m_w, n_w;
        uint32_t voff[LPWc];
    };
    auto tile_of = [&](int lt) __attribute__((always_inline)) -> Tile {
        Tile t;
        const int band = 8 * TN, b = lt / band, rem = lt - b * band;
        const int hgt = TM - 8 * b < 8 ? TM - 8 * b : 8;          // M-tiles in this band
        const int tm = 8 * b + rem % hgt, tn = rem / hgt;
        const int au0 = tm * WM, wu0 = tn * 2;
        t.a_valid = p.a_units - au0 < WM ? p.a_units - au0 : WM;
        t.w_valid = p.w_units - wu0 < 2 ? p.w_units - wu0 : 2;
        t.a_tile = p.a_pk + (int64_t)au0 * p.ustride;
        t.w_tile = p.w_pk + (int64_t)wu0 * p.ustride;
        t.m_w = (int64_t)au0 * 64 + wm * 64;
        t.n_w = (int64_t)wu0 * 64 + wn * 64;
#pragma unroll
        for (int k = 0; k < LPW; ++k) {
            const int j0 = wave + NWAVE * k, j = j0 < NI ? j0 : wave;
            const bool isa = j < NA;
            int q = 64 * (isa ? j : j - NA) + lane;             // 16-byte chunk within the part
            const int nq = (isa ? WM : 2) * (IMG4 / 16);
            q = q < nq ? q : nq - 1;
            int unit = q / (IMG4 / 16);
            const int off = q - unit * (IMG4 / 16);
            const int valid = isa ? t.a_valid : t.w_valid;
            unit = unit < valid ? unit : valid - 1;               // ragged tiles repeat their last unit
            t.voff[k] = (uint32_t)unit * (uint32_t)p.ustride + 16u * off;
        }
        return t;
    };
    const Tile T = tile_of(logical);

    // ---- loader: DMA instruction j of a stage fills LDS bytes [1024 j, 1024 j + 1024) of the
    // stage; j < NA: activation units, else weight units.  Wavefront w issues j = w, w + NWAVE, ...
    // Lanes past the end of a part repeat its last chunk (they land in the padding).
    // Every wavefront issues LPW instructions per stage, so that the waits below are the same
    // immediate in every wavefront and no branch sits inside a K-step: a wavefront without an
    // LPW-th block repeats its first block into a spare kilobyte that nobody reads.
    const uint32_t vzero = 0;
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(smem), spare = lds0 + Gm::SPARE;
    // instruction k of the request of group v into stage `stage`
    auto request_one = [&](int k, int v, int stage) __attribute__((always_inline)) {
        const int j0 = wave + NWAVE * k, j = j0 < NI ? j0 : wave;
        // (selected with a mask, not with ?: -- the compiler turns that into a branch)
        const uint32_t mk = NWAVE * (k + 1) <= NI ? ~0u : 0u - (uint32_t)(j0 < NI);
        const uint32_t dst = spare + ((lds0 + stage * STAGE + 1024 * j - spare) & mk);
        dma16(dst, T.voff[k], (j < NA ? T.a_tile : T.w_tile) + (int64_t)v * IMG4);
    };
    // Past the last INT4 group the same number of instructions is issued, so that the count a wait
    // refers to never changes: every lane reads the tile's first 16 bytes (one cache line per
    // instruction) into the spare kilobyte.
    auto request_dummy = [&]() __attribute__((always_inline)) { dma16(spare, vzero, T.a_tile); };
    // Instruction k of the request of the first INT8 group, activation part (NA8 instructions) or
    // weight part, into stage `stage`: issued in place of the dummies of two of the last steps,
    // whose stages are free by then, so that the group has landed when the K loop ends.
    // (Here an image starts on a multiple of kU8 = 9 KB of the stage and is moved by nine
    // instructions of its own, so that everything but the lane's chunk is the same in all lanes.)
    auto request_int8 = [&](int k, int stage, bool act) __attribute__((always_inline)) {
        const int j = wave + NWAVE * k;
        const bool real = j < 9 * (act ? WM : 2);
        const int unit = j / 9, jin = j - 9 * unit;               // (uniform)
        const int valid = act ? T.a_valid : T.w_valid;
        const int src_unit = unit < valid ? unit : valid - 1;     // ragged tiles repeat their last unit
        int chunk = 64 * jin + lane;                            // 16-byte chunk of the image; its last instruction is half empty
        chunk = chunk < IMG8 / 16 ? chunk : IMG8 / 16 - 1;
        const uint32_t vo = (uint32_t)src_unit * (uint32_t)p.ustride + 16u * chunk;
        const uint32_t dst = real ? lds0 + stage * STAGE + unit * kU8 + 1024 * jin : spare;
        dma16(dst, vo, (act ? T.a_tile : T.w_tile) + (int64_t)G4 * IMG4);
    };

    // ---- fragment addresses: one register per operand (and one per operand for the scales) holds
    // the lane's address inside the stage of the coming group; everything a step reads is that
    // plus an immediate.  The registers move on by one stage per step.
    const uint32_t lane_off = lds0 + 1024 * g + 16 * r;
    const uint32_t a_off = wm * IMG4 + lane_off, b_off = APART + wn * IMG4 + lane_off;
    const uint32_t sa_off = lds0 + wm * IMG4 + SC4 + 8 * r, sb_off = lds0 + APART + wn * IMG4 + SC4 + 8 * r;

    // the 48 bytes of sub-tile row (column) block i of a unit: the operands of its two MFMAs
    // (addresses are 32-bit LDS addresses, the workgroup's base included)
    typedef __attribute__((address_space(3))) const v4i *lds_v4i;
    typedef __attribute__((address_space(3))) const v2u *lds_v2u;
    auto read_pair = [&](uint32_t addr, int i) __attribute__((always_inline)) -> v12i {
        const v4i c0 = *(lds_v4i)(uintptr_t)(addr + 512 * i);
        const v4i c1 = *(lds_v4i)(uintptr_t)(addr + 512 * i + 2048);
        const v4i c2 = *(lds_v4i)(uintptr_t)(addr + 512 * i + 4096);
        const v8i lo = __builtin_shufflevector(c0, c1, 0, 1, 2, 3, 4, 5, 6, 7);
        const v8i hi = __builtin_shufflevector(c2, c2, 0, 1, 2, 3, -1, -1, -1, -1);
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11);
    };
    // scale operand of rows 32 i + r: {fp16 bits, 0, 0, 0}
    auto read_scale = [&](uint32_t addr, int i) __attribute__((always_inline)) -> v2u {
        return *(lds_v2u)(uintptr_t)(addr + 256 * i);
    };

    v16f acc[4];
    const v16f zf = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};

    auto scale_tile = [&](v2u ta, v2u tb) __attribute__((always_inline)) -> v16f {
        return __builtin_amdgcn_mfma_f32_32x32x8f16(__builtin_bit_cast(v4h, ta), __builtin_bit_cast(v4h, tb), zf, 0, 0, 0);
    };
    // steps 2 and 3 for elements e0 .. e1-1 of sub-tile (i, j) of group grp
    auto dequant = [&](int grp, int i, int j, const v16f &c, const v16f &s, int e0, int e1) __attribute__((always_inline)) {
#pragma unroll
        for (int e = e0; e < e1; ++e) acc[2 * i + j][e] = fmaf(c[e], s[e], acc[2 * i + j][e]);
        if (DBG && grp >= 0) {
#pragma unroll
            for (int e = e0; e < e1; ++e) {
                const int64_t m = T.m_w + 32 * i + 8 * (e >> 2) + 4 * g + (e & 3), n = T.n_w + 32 * j + r;
                if (m < p.M && n < p.N) p.partials[(m * p.N + n) * (p.G4 + p.G8) + grp] = (int32_t)c[e];
            }
        }
    };

    v12i af0, bf0;
    v2u sa[2], sb[2];
    v16f c_pend, s_pend;
    int  u_pend;
    int cur;
    uint32_t a_cur, b_cur;
    // ---- prologue: the first NST groups are requested, the first one has landed
    {
#pragma unroll
        for (int v = 0; v < NST; ++v) {
            if (v < G4) {
#pragma unroll
                for (int k = 0; k < LPW; ++k) request_one(k, v, v);
            } else {
#pragma unroll
                for (int k = 0; k < LPW; ++k) request_dummy();
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(wait_imm((NST - 1) * LPW));
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = zf;
    cur = 0; a_cur = a_off; b_cur = b_off;
    // carried from step to step: the fragments of sub-tile row 0 / column 0 and the scale operands of
    // the coming step, and the integer and scale tiles of the last sub-tile of the step before
    af0 = read_pair(a_cur, 0); bf0 = read_pair(b_cur, 0);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        sa[i] = read_scale(sa_off, i);
        sb[i] = read_scale(sb_off, i);
        sb[i][0] = g == 0 ? sb[i][0] : 0u;     // zero on one side keeps k-slots 4..7 of the fp16 MFMA empty
    }
    c_pend = zf; s_pend = zf;
    u_pend = -1;

    // One K-step = one INT4 group.  Twelve slots of one MFMA each, fenced so that the compiler keeps
    // their order.  Sub-tiles in the order (0,0) (1,0) (0,1) (1,1): column fragments 0 are free after
    // the second sub-tile and row fragments 0 after the third, and are refilled from the next stage.
    // Of the three slots of a sub-tile the first carries the step's memory instructions and address
    // updates, the other two eight fused multiply-adds each of the sub-tile before (its last MFMA
    // is two slots back by then): the vector ALU has about as much to do as the matrix pipe, and an
    // in-order wavefront that meets more than 32 cycles of vector work between two MFMAs holds
    // the matrix pipe up.  The barrier comes after the third slot: group u+1 has landed (each
    // wavefront waited for its own share before it) and every read of stage u is complete (issued
    // in the first slot), so from there on stage u is refilled with group u + NST, spread over
    // three slots: issued in one burst the requests fill the address queue and hold up MFMAs.
    // A step has no branch (one inside it lets the compiler sink MFMAs past the barrier): MODE says
    // at compile time what the step requests: 0 group u + NST, 1 nothing (dummies), 2 / 3 the
    // activation / weight part of the first INT8 group.
    auto step = [&](int u, auto mode_c) __attribute__((always_inline)) {
        constexpr int MODE = decltype(mode_c)::value;
        const int nxt = cur + 1 == NST ? 0 : cur + 1;
        // lane addresses in the next stage (they become the current ones of the next step)
        const uint32_t a_nxt = a_off + nxt * STAGE, b_nxt = b_off + nxt * STAGE;
        const uint32_t sa_nxt = sa_off + nxt * STAGE, sb_nxt = sb_off + nxt * STAGE;
        v12i af1, bf1;
        v16f c0, c1, c2, c3, s0, s1, s2, s3;
        v2u nsa[2], nsb[2];
        int kreq = 0;                           // DMA instructions of this step issued so far
        auto dma_slot = [&](int n) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < n; ++q, ++kreq) {
                if (kreq < LPW) {
                    if constexpr (MODE == 0)      request_one(kreq, u + NST, cur);
                    else if constexpr (MODE == 2) request_int8(kreq, cur, true);
                    else if constexpr (MODE == 3) request_int8(kreq, cur, false);
                    else                          request_dummy();
                }
            }
        };
        constexpr int PER = (LPW + 2) / 3;      // per slot, over the three memory slots behind the barrier
        // slot 0
        ATOM_F6_PIN(af0);
        c0 = mfma_f6<0>(af0, bf0, zf);
        ATOM_F6_PIN(c0);
        af1 = read_pair(a_cur, 1);
        bf1 = read_pair(b_cur, 1);
        ATOM_F6_SLOT_END();
        // slot 1
        ATOM_F6_PIN(sa[0]);
        s0 = scale_tile(sa[0], sb[0]);
        ATOM_F6_PIN(s0);
        dequant(u_pend, 1, 1, c_pend, s_pend, 0, 8);
        ATOM_F6_PIN(acc[3]);
        ATOM_F6_SLOT_END();
        // slot 2
        c0 = mfma_f6<1>(af0, bf0, c0);
        ATOM_F6_PIN(c0);
        dequant(u_pend, 1, 1, c_pend, s_pend, 8, 16);
        ATOM_F6_PIN(acc[3]);
        ATOM_F6_SLOT_END();
        __builtin_amdgcn_s_waitcnt(wait_imm((NST - 2) * LPW));
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        // slot 3
        ATOM_F6_PIN(af1);
        ATOM_F6_PIN(bf0);
        c1 = mfma_f6<0>(af1, bf0, zf);
        ATOM_F6_PIN(c1);
        dma_slot(PER);
        ATOM_F6_SLOT_END();
        // slot 4
        ATOM_F6_PIN(sa[1]);
        s1 = scale_tile(sa[1], sb[0]);
        ATOM_F6_PIN(s1);
        dequant(u, 0, 0, c0, s0, 0, 8);
        ATOM_F6_PIN(acc[0]);
        ATOM_F6_SLOT_END();
        // slot 5
        c1 = mfma_f6<1>(af1, bf0, c1);
        ATOM_F6_PIN(c1);
        dequant(u, 0, 0, c0, s0, 8, 16);
        ATOM_F6_PIN(acc[0]);
        ATOM_F6_SLOT_END();
        // slot 6
        ATOM_F6_PIN(bf1);
        c2 = mfma_f6<0>(af0, bf1, zf);
        ATOM_F6_PIN(c2);
        bf0 = read_pair(b_nxt, 0);
        dma_slot(PER);
        ATOM_F6_SLOT_END();
        // slot 7
        ATOM_F6_PIN(sb[1]);
        s2 = scale_tile(sa[0], sb[1]);
        ATOM_F6_PIN(s2);
        dequant(u, 1, 0, c1, s1, 0, 8);
        ATOM_F6_PIN(acc[2]);
        ATOM_F6_SLOT_END();
        // slot 8
        c2 = mfma_f6<1>(af0, bf1, c2);
        ATOM_F6_PIN(c2);
        dequant(u, 1, 0, c1, s1, 8, 16);
        ATOM_F6_PIN(acc[2]);
        ATOM_F6_SLOT_END();
        // slot 9
        ATOM_F6_PIN(af1);
        c3 = mfma_f6<0>(af1, bf1, zf);
        ATOM_F6_PIN(c3);
        af0 = read_pair(a_nxt, 0);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            nsa[i] = read_scale(sa_nxt, i);
            nsb[i] = read_scale(sb_nxt, i);
        }
        dma_slot(LPW);                          // whatever is left
        ATOM_F6_SLOT_END();
        // slot 10
        ATOM_F6_PIN(sa[1]);
        s3 = scale_tile(sa[1], sb[1]);
        ATOM_F6_PIN(s3);
        dequant(u, 0, 1, c2, s2, 0, 8);
        ATOM_F6_PIN(acc[1]);
        ATOM_F6_SLOT_END();
        // slot 11
        c3 = mfma_f6<1>(af1, bf1, c3);
        ATOM_F6_PIN(c3);
        dequant(u, 0, 1, c2, s2, 8, 16);
        ATOM_F6_PIN(acc[1]);
        ATOM_F6_PIN(nsa[0]); ATOM_F6_PIN(nsa[1]); ATOM_F6_PIN(nsb[0]); ATOM_F6_PIN(nsb[1]);   // (keeps the wait for these reads down here)
        sa[0] = nsa[0]; sa[1] = nsa[1];
        sb[0] = nsb[0]; sb[1] = nsb[1];
        sb[0][0] = g == 0 ? sb[0][0] : 0u; sb[1][0] = g == 0 ? sb[1][0] : 0u;
        ATOM_F6_SLOT_END();
        c_pend = c3; s_pend = s3; u_pend = u;
        cur = nxt; a_cur = a_nxt; b_cur = b_nxt;
    };
    // The last NST steps have nothing of the K loop left to request.  Two of them fetch the first
    // INT8 group instead (its two parts fit a stage each), which then costs no round trip of its own.
    static_assert(9 * WM <= LPW * NWAVE && 9 * 2 <= LPW * NWAVE && WM * kU8 <= STAGE && 2 * kU8 <= STAGE, "a part per step and stage");
    const bool pre8 = p.G8 >= 1 && G4 >= NST;
    int stage8a = 0, stage8w = 0;
    {
        using std::integral_constant;
        int u = 0;
        for (; u + NST < G4; ++u) step(u, integral_constant<int, 0>{});
        if (pre8) {
            stage8a = cur; step(u++, integral_constant<int, 2>{});
            stage8w = cur; step(u++, integral_constant<int, 3>{});
        }
        for (; u < G4; ++u) step(u, integral_constant<int, 1>{});
    }
    dequant(u_pend, 1, 1, c_pend, s_pend, 0, 16);

    // ---- the INT8 groups: INT8 MFMA, int32 tile converted to fp32, the same dequantisation
    {
        constexpr int NA8 = Gm::NA8, NI8 = Gm::NI8, LPW8 = Gm::LPW8, APART8 = Gm::APART8;
        uint32_t voff8[LPW8];
#pragma unroll
        for (int k = 0; k < LPW8; ++k) {
            const int j = wave + NWAVE * k;
            const bool isa = j < NA8;
            int q = 64 * (isa ? j : j - NA8) + lane;
            const int nq = (isa ? WM : 2) * (IMG8 / 16);
            q = q < nq ? q : nq - 1;
            int unit = q / (IMG8 / 16);
            const int off = q - unit * (IMG8 / 16);
            const int valid = isa ? T.a_valid : T.w_valid;
            unit = unit < valid ? unit : valid - 1;
            voff8[k] = (uint32_t)unit * (uint32_t)p.ustride + 16u * off;
        }
        int ck[4];                                                 // byte offset of chunk 2 kk + g of row r
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) ck[kk] = 128 * (lane & 31) + 16 * (((2 * kk + (lane >> 5)) ^ (lane & 31) ^ (((lane & 31) >> 3) & 1)) & 7);
        __builtin_amdgcn_s_waitcnt(wait_imm(0));                    // the requests of the K loop's last steps
        for (int g8 = 0; g8 < p.G8; ++g8) {
            const bool here = pre8 && g8 == 0;                     // requested during the K loop, in two stages
            const int a_unit8 = here ? stage8a * STAGE + wm * kU8 : wm * IMG8;
            const int b_unit8 = here ? stage8w * STAGE + wn * kU8 : APART8 + wn * IMG8;
            __syncthreads();                                       // every read of the LDS contents so far is done
            if (!here) {
                const uint8_t *ab = T.a_tile + (int64_t)G4 * IMG4 + (int64_t)g8 * IMG8;
                const uint8_t *wb = T.w_tile + (int64_t)G4 * IMG4 + (int64_t)g8 * IMG8;
#pragma unroll
                for (int k = 0; k < LPW8; ++k) {
                    const int j = wave + NWAVE * k;
                    if (j < NI8) dma16(lds0 + 1024 * j, voff8[k], j < NA8 ? ab : wb);
                }
                __builtin_amdgcn_s_waitcnt(wait_imm(0));
                __syncthreads();
            }
            v2u qa[2], qb[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                qa[i] = *reinterpret_cast<const v2u *>(smem + a_unit8 + SC8 + 8 * r + 256 * i);
                qb[i] = *reinterpret_cast<const v2u *>(smem + b_unit8 + SC8 + 8 * r + 256 * i);
                qb[i][0] = g == 0 ? qb[i][0] : 0u;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    v16i ci = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) {
                        const v4i a = *reinterpret_cast<const v4i *>(smem + a_unit8 + ck[kk] + 4096 * i);
                        const v4i b = *reinterpret_cast<const v4i *>(smem + b_unit8 + ck[kk] + 4096 * j);
                        ci = __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, ci, 0, 0, 0);
                    }
                    const v16f s = scale_tile(qa[i], qb[j]);
                    v16f cf;
#pragma unroll
                    for (int e = 0; e < 16; ++e) cf[e] = (float)ci[e];
                    dequant(G4 + g8, i, j, cf, s, 0, 16);
                }
        }
    }
    __syncthreads();                                               // LDS is free

    // ---- store: the 64 x 64 fp16 tile of a wavefront goes through LDS so that global memory sees
    // whole 128-byte rows (a lane holds one column of the MFMA layout).
    constexpr int OSTRIDE = Gm::OSTRIDE;
    unsigned char *ot = smem + wave * (64 * OSTRIDE);
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int row = 32 * (t >> 1) + 8 * (e >> 2) + 4 * g + (e & 3);
            const int col = 32 * (t & 1) + r;
            *reinterpret_cast<uint16_t *>(ot + row * OSTRIDE + col * 2) = __half_as_ushort(__float2half_rn(acc[t][e]));
        }
    __builtin_amdgcn_s_waitcnt(wait_imm(0));                   // the wavefront reads only what it wrote itself
    store_block<64, 64, true>(ot, OSTRIDE, p.y, p.ldy, T.m_w, T.n_w, p.M, p.N, lane);
}

template <int WM, bool DBG>
hipError_t launch_f6_cfg(const F6Params &p, hipStream_t stream)
{
    using Gm = F6Geom<WM>;
    static_assert(Gm::LDS <= 160 * 1024, "LDS of a compute unit");
    static_assert(Gm::LPW * (Gm::NST - 1) <= 63, "vmcnt is a 6-bit counter");
    const int64_t TM = (p.a_units + WM - 1) / WM, TN = (p.w_units + 1) / 2;
    auto kern = &w4a4_gemm_f6_kernel<WM, DBG>;
    static atom_launch::LdsOptIn opt_in;   // one attribute call per kernel variant and device
    hipError_t err = atom_launch::ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(kern), Gm::LDS);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(kern, dim3((unsigned)(TM * TN)), dim3(Gm::NT), Gm::LDS, stream, p);
    return hipGetLastError();
}

}  // namespace

namespace atom_internal {

// Tile of a launch: 0, 1, 2 = thin 64 x 64, 64 x 128, 128 x 128; 3 to 8 = walking 128 x 128, 256 x 128, 256 x 192, 128 x 384,
// 256 x 256, 192 x 128; -1: the general kernel.
//
// Among the first five the estimate is the time per INT4 group in units of 10 ns: rounds of tiles over the compute units times
// what a tile's step takes.  Thin tiles win where large ones leave compute units without work; beyond the first round (64 x 64: the
// third) they pay prologue and store in the open and fetch more bytes per multiply-add than the walking ones.  Two lines
// beside that, both at K = 4096 / 11008, weights from HBM:
//   * 128 x 128 with hardly more tiles than compute units: the few that share one cost less than a full second round (M = 384,
//     N = 11008, 258 tiles: 27.5 / 59.2 us, 256 x 128 30.4 / 64.8; M = 896, N = 4992, 273 tiles: 28.1 / 58.6 and 29.5 / 62.6).  With
//     how many tiles that ends differs with the rows of tiles (after 264, 264, 275, 270 and 280 tiles of 3, 4, 5, 6 and 8 rows:
//     M = 512, N = 8576, 268 tiles: 32.9 / 73.8 us, 256 x 128 30.1 / 64.1); with two rows 258 tiles are slow already;
//   * three units of rows: the general kernel leaves the fourth unit of its two rows of tiles out of its requests, the walking one
//     moves the last tile back and fetches three units twice (M = 192, K = 8192, N = 28672: 66.6 us, walking 71.9; N = 57344:
//     130 / 139).  From 17 groups on both yield to tiles of 192 rows.
//
// Where 256 x 128 (or, of three units, the general kernel) comes out and as many rows of tiles of 192 cover M, those are taken from 17 groups on: the same
// number of tiles with three quarters of the work each.  On six wavefronts, two SIMDs with two and two with one, that is not worth
// three quarters of the time, so nowhere else.  Weights from HBM, us: M = 192, K = 4096, N = 22016 36.0 -> 30.7 (general), K = 5120, N = 27648
// 47.3 -> 41.2, K = 8192, N = 57344 131 -> 117; M = 320, K = 5120, N = 13824 39.1 -> 36.5 (256 x 128), M = 384, K = 4096, N = 12288 31.7 -> 29.2,
// M = 576, K = N = 8192 51.3 -> 51.7 (from the cache 49.9 -> 45.7).
//
// Against the tile that then stands, the three wide ones, which fetch fewer bytes per multiply-add and cover the output in fewer
// rounds, by an estimate of the whole time (fit_ns), fitted to 969 sizes (M = 65 to 4096, K = 2304 to 14336, N = 1000 to 28672): taken at 360 of them,
// where the time is 0.76 to 1.02 of the other tile's (0.890 on average); over all of them what is taken is 1.0005
// of the best of the candidates (at 6 above 1.02: M = 707, K = 8192, N = 12288 1.044, M = 2061, K = 4096, N = 8409 1.040).  With up to sixteen groups the
// wide tiles' prologues and stores take what their steps gain (16 groups, M = 2304, N = 8200: 47.7 us on 128 x 128, 50.2 at best on
// a wide one; seven, M = 1100, N = 16300: 32.4, 33.8; M = 1700, N = 2870: 15.3, 17.7).
// Every tile on these sizes and what the rule takes: profiles/w4a4_gemm_f6_tiles.txt.
//
// ns of a round, and per group of a full round, of a part of one that is all there is, and of one behind full rounds (both: with hardly a tile, and what they
// grow by up to one per compute unit).  A part behind full rounds costs less: workgroups that walk don't wait for each other, so it starts in the gaps
// that they leave (128 x 128 in two rounds and eight tiles, and 256 x 192, which one cost for both takes: M = 1536, K = 4096, N = 11008 71.4, 73.9; M = 759, N = 22016 77.1, 78.7).
struct TileTime { int ua, uw, round, full, alone, alone_share, behind, behind_share; };

// Estimated time of a launch in ns, weights from HBM.  128 x 128 tiles walk two to a compute unit, so a full round is two of them to each, and
// a last round of more than one to each approaches it.
static int64_t fit_ns(int tile, int64_t au, int64_t wu, int64_t G4, int64_t cus)
{
    static const TileTime time[9] = {
        {1, 1, 0, 200, 200, 40, 160, 100},    {1, 2, 900, 320, 270, 70, 260, 130},  {2, 2, 1900, 470, 390, 60, 340, 160}, {2, 2, 4100, 860, 460, 40, 180, 250},
        {4, 2, 6400, 740, 540, 170, 340, 430}, {4, 3, 7400, 1070, 650, 340, 630, 440}, {2, 6, 7900, 1070, 760, 210, 630, 430}, {4, 4, 8200, 1370, 910, 260, 860, 190},
        {3, 2, 4800, 620, 520, 90, 460, 170}};
    const TileTime &t = time[tile];
    const int64_t tiles = ((au + t.ua - 1) / t.ua) * ((wu + t.uw - 1) / t.uw), slots = tile == 3 ? 2 * cus : cus;
    const int64_t full = tiles / slots, rest = tiles % slots;
    const int64_t last = rest == 0 ? 0 : rest > cus ? t.full - 250 * (slots - rest) / cus
                       : full == 0 ? t.alone + t.alone_share * rest / cus : t.behind + t.behind_share * rest / cus;
    return 4000 + (full + (rest != 0)) * t.round + G4 * (full * t.full + last);
}

// `us`: the estimate of the tile taken, operands out of the last-level cache: for the wide tiles and those of 192 rows fit_ns less what the cache gives and, one launch
// behind the other, the call's own 4 us do not show (by tile from 1 us above fit_ns to 4 us below it).
static int pick_tile(int64_t au, int64_t wu, int64_t G4, int64_t cus, float *us = nullptr)
{
    struct { int ua, uw, rounds, first, more; } const tile[5] = {
        {1, 1, 3, 13, 21}, {1, 2, 1, 21, 37}, {2, 2, 1, 37, 60}, {2, 2, 1, 45, 0}, {4, 2, 1, 79, 79}};
    int best = -1;
    int64_t least = INT64_MAX;
    for (int i = 0; i < 5; ++i) {
        if (au < tile[i].ua || wu < tile[i].uw) continue;
        const int64_t rows = (au + tile[i].ua - 1) / tile[i].ua, tiles = rows * ((wu + tile[i].uw - 1) / tile[i].uw);
        const int64_t n = (tiles + cus - 1) / cus;
        const int64_t cost = n <= tile[i].rounds ? n * tile[i].first
                           : i == 3 && n == 2 && rows >= 3 && tiles - cus < 3 * (rows < 8 ? rows : 8) ? 72
                           : i == 3 ? n * 45 - n / 2 * 3       // (two workgroups per compute unit: the pair costs a little less)
                                    : n * tile[i].more;
        if (cost < least) { least = cost; best = i; }
    }
    if (us) *us = 5.0f + 0.0093f * (float)least * (float)(G4 + 2);
    const bool general = best == 3 && au == 3;
    if (G4 < 17 || best < 0) return general ? -1 : best;
    if (general || (best == 4 && (au + 2) / 3 == (au + 3) / 4)) best = 8;
    int64_t ns = fit_ns(best, au, wu, G4, cus);
    for (int i = 5; i < 8; ++i) {
        static const int ua[3] = {4, 2, 4}, uw[3] = {3, 6, 4};
        if (au < ua[i - 5] || wu < uw[i - 5]) continue;
        const int64_t wide = fit_ns(i, au, wu, G4, cus);
        if (wide < ns) { ns = wide; best = i; }
    }
    if (us && best >= 5) *us = 0.001f * (float)ns - 1.5f;
    return best;
}

// The same for the sizes of a call without a dump; -1: the general kernel.
static int tile_of_launch(int64_t M, int64_t N, int K, int O, int64_t cus)
{
    const int G4 = (K - O) >> 7, G8 = O >> 7;
    return G8 == 1 && G4 >= 7 ? pick_tile((M + 63) / 64, (N + 63) / 64, G4, cus) : -1;
}

size_t f6_packed_bytes(int64_t rows, int K, int O)
{
    const int64_t units = (rows + 63) / 64;
    const int G4 = (K - O) >> 7, G8 = O >> 7;
    return (size_t)(units * ((int64_t)G4 * IMG4 + (int64_t)G8 * IMG8));
}

static PackParams pack_params(const void *q4, const void *q8, const void *scale, int64_t rows, int K, int O, void *out)
{
    PackParams p;
    p.q4 = static_cast<const uint8_t *>(q4); p.q8 = static_cast<const int8_t *>(q8);
    p.scale = static_cast<const uint16_t *>(scale);
    p.out = static_cast<uint8_t *>(out);
    p.rows = rows;
    p.units = (int)((rows + 63) / 64);
    p.G4 = (K - O) >> 7; p.G8 = O >> 7; p.O = O;
    p.ustride = (int64_t)p.G4 * IMG4 + (int64_t)p.G8 * IMG8;
    return p;
}

static hipError_t launch_pack(const PackParams &p, const PackParams &q, hipStream_t stream)
{
    const unsigned units = (unsigned)(p.units + q.units);
    // One group to a workgroup up to eleven of them per compute unit, where the time is that of a round (1024 x 4096 4.1 us, with four groups
    // 4.8; 1024 x 11008 5.9, 6.8; 13824 x 1664, 2592 of them, 7.4, 8.2; 8192 x 3072, 2944 of them, 8.3, 8.4; 4096 x 8192, 4032 of them, 11.1, 10.4), and where
    // four would leave most of a row's last workgroup idle (152064 rows of 256: 11.3, 17.9; 16384 of 1280: 6.4, 8.8)
    if ((int64_t)p.G4 * units <= 2816 || p.G4 < 4 || (p.G4 % 4 == 1 && p.G4 < 12))
        hipLaunchKernelGGL(pack_rows_kernel<1>, dim3((unsigned)(p.G4 + p.G8), units), dim3(256), 0, stream, p, q);
    else
        hipLaunchKernelGGL(pack_rows_kernel<4>, dim3((unsigned)((p.G4 + 3) / 4 + p.G8), units), dim3(256), 0, stream, p, q);
    return hipGetLastError();
}

hipError_t launch_f6_pack(const void *q4, const void *q8, const void *scale, int64_t rows, int K, int O,
                          void *out, hipStream_t stream)
{
    PackParams none{};
    return launch_pack(pack_params(q4, q8, scale, rows, K, O, out), none, stream);
}

hipError_t launch_f6_pack_both(const GemmArgs &a, void *a_out, void *w_out, hipStream_t stream)
{
    return launch_pack(pack_params(a.a_q4, a.a_q8, a.a_scale, a.M, a.K, a.O, a_out),
                       pack_params(a.w_q4, a.w_q8, a.w_scale, a.N, a.K, a.O, w_out), stream);
}

float f6_product_us(int64_t M, int64_t N, int K, int O, int64_t cus)
{
    const int G4 = (K - O) >> 7;
    if (O != 128 || G4 < 7) return 0.0f;
    float us;
    pick_tile((M + 63) / 64, (N + 63) / 64, G4, cus, &us);
    return us;                                                   // (operands that were just written: out of the last-level cache)
}

hipError_t launch_f6_gemm(const void *a_pk, int64_t M, const void *w_pk, int64_t N, int K, int O, void *y,
                          int64_t ldy, int32_t *partials, hipStream_t stream)
{
    F6Params p;
    p.a_pk = static_cast<const uint8_t *>(a_pk); p.w_pk = static_cast<const uint8_t *>(w_pk);
    p.y = static_cast<uint16_t *>(y); p.partials = partials;
    p.M = M; p.N = N; p.ldy = ldy;
    p.a_units = (int)((M + 63) / 64); p.w_units = (int)((N + 63) / 64);
    p.G4 = (K - O) >> 7; p.G8 = O >> 7;
    p.ustride = (int64_t)p.G4 * IMG4 + (int64_t)p.G8 * IMG8;
    const int pick = partials ? -1 : tile_of_launch(M, N, K, O, atom_launch::compute_units());
    if (pick >= 0) return pick < 3 ? launch_thin(p, pick, stream) : launch_walk(p, pick - 3, stream);
    // 256-row tiles halve the weight traffic per row but want at least four rounds of tiles over the
    // 256 compute units; 128-row tiles run two workgroups per compute unit, which hides one's prologue,
    // barriers and store behind the other's K loop
    const int64_t tiles256 = ((M + 255) / 256) * ((N + 127) / 128);
    if (M > 128 && tiles256 >= 1024) return partials ? launch_f6_cfg<4, true>(p, stream) : launch_f6_cfg<4, false>(p, stream);
    if (M > 64) return partials ? launch_f6_cfg<2, true>(p, stream) : launch_f6_cfg<2, false>(p, stream);
    return partials ? launch_f6_cfg<1, true>(p, stream) : launch_f6_cfg<1, false>(p, stream);
}

}  // namespace atom_internal

// For the tests of the tiles: which one a call takes on a card of `cus` compute units.
extern "C" int atom_internal_packed_tile(int64_t M, int64_t N, int32_t K, int32_t O, int64_t cus)
{
    return atom_internal::tile_of_launch(M, N, K, O, cus);
}
