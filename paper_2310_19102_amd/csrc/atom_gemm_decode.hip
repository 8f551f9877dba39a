// Weight-streaming variants of the group GEMM for decode-sized M (up to 256 rows).
//
// Same arithmetic as atom_gemm.hip (Section 4.2 of the paper, steps 1-3), except
// that the per-group terms of one output are summed in a fixed tree (eight K-slices,
// each in ascending group order, then slices 0..7) instead of one ascending chain.
//
// At these sizes the kernel is bound by reading the packed weights once from HBM
// (Section 3 of the paper: small-batch dense layers are memory-bound), so the
// layout of the work follows the weight bytes:
//   * a workgroup (8 wavefronts) owns 16 output channels = 16 weight rows, all of K;
//     N/16 workgroups keep every CU busy even at N = 4096;
//   * wavefront w owns a contiguous run of groups of those rows (split-K inside the
//     workgroup); it fetches its weight bytes with one 128-bit load per lane and
//     group (16 rows x 64 bytes per instruction, four groups in flight) and never
//     shares them, so no LDS staging and no barrier sits on the streaming path;
//   * the activation codes (M x K/2 bytes, L2-resident) are fetched per wavefront
//     in the same MFMA register layout (at M <= 16 in the common case: the real rows
//     only, through a copy in LDS); rows >= M are zeros or never stored;
//   * the contraction is the INT8 MFMA 16x16x64: one 128-channel INT4 group is two
//     MFMAs (even-position and odd-position codes after the nibble widening), an
//     INT8 group is two MFMAs of 64 channels;
//   * each wavefront dequantises its own groups into fp32 (convert, scale product,
//     fused multiply-add), the eight partial tiles meet in LDS once, at the end.
//
// MFMA 16x16x64 i8 layout: lane l supplies row (l & 15) of its operand and the
// 16 bytes of K-chunk (l >> 4); the result has column (l & 15) in lane l and rows
// 4*(l >> 4) + e in register e = 0..3.  Activations are the row operand.

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include <type_traits>

#include "atom_gemm_common.h"
#include "atom_gemm_decode_staged.h"
#include "atom_launch.h"

namespace {

using namespace atom_gemm;

using namespace atom_decode_staged;        // NW, NT, TN and the helpers shared with the one-launch decode linear

// The general kernel.
// RB: 16-row blocks of activations (M <= 16 * RB)
// VS: the wavefronts' runs are whole blocks of four groups (G even), so the four scales of a
//     batch are one 8-byte load per row (instead of four 2-byte loads that several wavefronts
//     request from the same lines); needs 4-byte aligned scale arrays
// ONE8: there is exactly one INT8 group (O = 128, the set-up of the paper), the last group of the
//     last wavefront's run.  The second 64 bytes of its rows then have registers of their own, and
//     the slots hold one 16-byte piece each.
// The common decoding case (ONE8, G a multiple of four, 8-byte aligned scale rows) has kernels of
// its own below; this one takes everything else.
template <int RB, bool VS, bool ONE8 = false>
__global__ __launch_bounds__(NT, 1)
void w4a4_gemm_decode_kernel(const GemmParams p)
{
    __shared__ float red[NW][RB][4][64];   // [slice][row block][register][lane]
    // groups whose loads are in flight together per wavefront (register budget)
    constexpr int DEPTH = (RB >= 4 && !ONE8) ? 2 : 4;

    const int tid  = threadIdx.x;
    const int lane = tid & 63;
    // (told to be the same in every lane: the INT4 / INT8 decisions below then are scalar branches;
    // as lane-dependent ones they became exec-masked regions, and the compiler waited for the loads
    // of a slot at the end of its region before it issued the next slot's: four memory round trips
    // per wavefront instead of one)
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, kc = lane >> 4;

    const int K4 = p.K - p.O, G = p.K >> 7, G4 = K4 >> 7;
    const int64_t n0 = (int64_t)blockIdx.x * TN;

    // this wavefront's run of groups
    // (VS: in whole blocks of four groups, so that a batch's four scales are one 8-byte piece of
    // a scale row that starts on a multiple of four; the last block of K may be a partial one)
    const int nblk    = VS ? (G + 3) >> 2 : G;
    const int g_begin = (VS ? 4 : 1) * (int)((int64_t)wave * nblk / NW);
    const int g_end   = min(G, (VS ? 4 : 1) * (int)((int64_t)(wave + 1) * nblk / NW));

    // weight row of this lane (clamped: rows >= N are computed and never stored)
    int64_t wr = n0 + col;
    wr = wr < p.N ? wr : p.N - 1;
    const uint8_t  *w4 = p.w_q4 + wr * (K4 >> 1) + kc * 16;
    const int8_t   *w8 = p.w_q8 + wr * p.O + kc * 16;
    const uint16_t *ws = p.w_scale + wr * G;
    // activation rows of this lane as the MFMA row operand (row = col index here)
    const uint8_t *a4[RB];
    const int8_t  *a8[RB];
    bool a_ok[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int64_t m = 16 * rb + col;
        a_ok[rb] = m < p.M;
        const int64_t mc = a_ok[rb] ? m : 0;
        a4[rb] = p.a_q4 + mc * (K4 >> 1) + kc * 16;
        a8[rb] = p.a_q8 + mc * p.O + kc * 16;
    }
    // ONE8 addresses every load as scalar base + 32-bit byte offset (arrays below 4 GiB: host),
    // one register per stream instead of a 64-bit pointer per load
    constexpr uint32_t GSTEP = 64u;                      // from one group's piece to the next, and to the second half of the INT8 group
    const uint32_t w4o = (uint32_t)(wr * (K4 >> 1)) + kc * 16;
    const uint32_t w8o = (uint32_t)(wr * p.O) + kc * 16;
    uint32_t a4o[RB], a8o[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int64_t mc = a_ok[rb] ? 16 * rb + col : 0;
        a4o[rb] = (uint32_t)(mc * (K4 >> 1)) + kc * 16;
        a8o[rb] = (uint32_t)(mc * p.O) + kc * 16;
    }
    const uint8_t *w8b = reinterpret_cast<const uint8_t *>(p.w_q8), *a8b = reinterpret_cast<const uint8_t *>(p.a_q8);
    // rows of the result held by this lane: 16*rb + 4*kc + e
    float acc[RB][4];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[rb][e] = 0.0f;

    const v4i zi = {0, 0, 0, 0};

    // Groups are processed in batches of DEPTH.  Every load of a batch (weight codes,
    // weight scales, activation codes, activation scales) is issued before the first is
    // used, so a wavefront pays the memory latency once per batch, not once per group.
    for (int gb = g_begin; gb < g_end; gb += DEPTH) {
        constexpr int HALVES = ONE8 ? 1 : 2;
        uint4    wq[DEPTH][HALVES];       // [group][half]: an INT4 group uses half 0 only
        uint4    aq[DEPTH][RB][HALVES];
        uint4    wx, ax[RB];              // ONE8: the second half of the INT8 group (untouched elsewhere)
        uint16_t wsc[DEPTH];
        uint16_t asc[DEPTH][RB][4];
        uint2    wvs, avs[RB][4];         // VS: the four scales of the batch stay packed until they are used
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int  g    = gb + d;
            const bool live = g < g_end;
            const int  gc   = live ? g : g_end - 1;         // dead slots re-read the last group
            const bool is4  = gc < G4;
            // (an INT4 slot leaves its second half alone: writing zeros there made the compiler wait
            // for every load in flight, since one of an earlier batch might still target the register)
            if constexpr (ONE8) {         // one load per slot: array and offset are scalar selects
                wq[d][0] = *reinterpret_cast<const uint4 *>((is4 ? p.w_q4 : w8b) + (is4 ? w4o + (uint32_t)gc * GSTEP : w8o));
            } else if (is4) {
                wq[d][0] = *reinterpret_cast<const uint4 *>(w4 + (size_t)gc * 64);
            } else {
                wq[d][0] = *reinterpret_cast<const uint4 *>(w8 + (size_t)(gc - G4) * 128);
                wq[d][1] = *reinterpret_cast<const uint4 *>(w8 + (size_t)(gc - G4) * 128 + 64);
            }
            if constexpr (!VS) wsc[d] = ws[gc];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                // rows >= M load row 0 (no lane-dependent branch around a load) and are zeroed below
                if constexpr (ONE8) {
                    aq[d][rb][0] = *reinterpret_cast<const uint4 *>((is4 ? p.a_q4 : a8b) + (is4 ? a4o[rb] + (uint32_t)gc * 64u : a8o[rb]));
                } else if (is4) {
                    aq[d][rb][0] = *reinterpret_cast<const uint4 *>(a4[rb] + (size_t)gc * 64);
                } else {
                    aq[d][rb][0] = *reinterpret_cast<const uint4 *>(a8[rb] + (size_t)(gc - G4) * 128);
                    aq[d][rb][1] = *reinterpret_cast<const uint4 *>(a8[rb] + (size_t)(gc - G4) * 128 + 64);
                }
                if constexpr (!VS) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int64_t m = 16 * rb + 4 * kc + e;
                        asc[d][rb][e] = m < p.M ? p.a_scale[m * G + gc] : (uint16_t)0;
                    }
                }
            }
        }
        if constexpr (ONE8) {
            // Unconditional (a branch around these loads made the compiler wait for them inside it):
            // a batch without the INT8 group reads the first piece of its first group once more.
            const bool has8 = g_end > G4 && gb + DEPTH >= g_end;
            const int  g0   = gb < G4 ? gb : G4 - 1;
            wx = *reinterpret_cast<const uint4 *>((has8 ? w8b : p.w_q4) + (has8 ? w8o + GSTEP : w4o + (uint32_t)g0 * GSTEP));
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                ax[rb] = *reinterpret_cast<const uint4 *>((has8 ? a8b : p.a_q4) + (has8 ? a8o[rb] + 64u : a4o[rb] + (uint32_t)g0 * 64u));
        }
        if constexpr (VS) {
            static_assert(!VS || DEPTH == 4, "a batch is four groups");
            // (32-bit element offsets on the scalar bases: M * G and N * G are far below 2^31)
            // A row of scales starts on an even element (G even) and its four-blocks on 4-byte
            // boundaries: two 4-byte loads, the second one held inside the row where the last block
            // of K has two groups only (its slots are dead).
            const int g2 = gb + 2 <= G - 2 ? gb + 2 : G - 2;
            // (scalar base + 32-bit byte offset per lane, like the codes)
            auto load4 = [&](const uint16_t *base, uint32_t row) {
                const uint8_t *sb  = reinterpret_cast<const uint8_t *>(base);
                const uint32_t off = row * (uint32_t)(2 * G);
                return make_uint2(*reinterpret_cast<const uint32_t *>(sb + 2 * gb + off),
                                  *reinterpret_cast<const uint32_t *>(sb + 2 * g2 + off));
            };
            wvs = load4(p.w_scale, (uint32_t)wr);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int64_t m = 16 * rb + 4 * kc + e;
                    // rows >= M: row 0 is read (no lane-dependent branch around a load), zeros are used
                    uint2 av = load4(p.a_scale, (uint32_t)(m < p.M ? m : 0));
                    if (m >= p.M) av = make_uint2(0, 0);
                    avs[rb][e] = av;
                }
        }
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int g = gb + d;
            if (g >= g_end) break;
            const bool is4 = g < G4;
            v4i b0, b1;
            if (is4) { b0 = widen_lo(wq[d][0]); b1 = widen_hi(wq[d][0]); }
            else     { b0 = __builtin_bit_cast(v4i, wq[d][0]); b1 = __builtin_bit_cast(v4i, ONE8 ? wx : wq[d][HALVES - 1]); }
            // 2^-8 of the nibble widening folded into the weight scale (exact)
            // scale number d of a packed four
            const int sidx = d;
            auto unpack = [&](const uint2 &v) { return (uint16_t)((sidx < 2 ? v.x : v.y) >> (16 * (sidx & 1))); };
            const float wsf = half_bits_to_float(VS ? unpack(wvs) : wsc[d]) * (is4 ? (1.0f / 256.0f) : 1.0f);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                v4i x0, x1;
                if (is4) { x0 = widen_lo(aq[d][rb][0]); x1 = widen_hi(aq[d][rb][0]); }
                else     { x0 = __builtin_bit_cast(v4i, aq[d][rb][0]); x1 = __builtin_bit_cast(v4i, ONE8 ? ax[rb] : aq[d][rb][HALVES - 1]); }
                if (!a_ok[rb]) { x0 = zi; x1 = zi; }
                v4i c = __builtin_amdgcn_mfma_i32_16x16x64_i8(x0, b0, zi, 0, 0, 0);
                c = __builtin_amdgcn_mfma_i32_16x16x64_i8(x1, b1, c, 0, 0, 0);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[rb][e] = fmaf((float)c[e], half_bits_to_float(VS ? unpack(avs[rb][e]) : asc[d][rb][e]) * wsf, acc[rb][e]);
            }
        }
    }

    // the eight K-slices meet in LDS and are added in slice order
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int e = 0; e < 4; ++e) red[wave][rb][e][lane] = acc[rb][e];
    __syncthreads();
    for (int idx = tid; idx < RB * 4 * 64; idx += NT) {
        const int l = idx & 63, e = (idx >> 6) & 3, rb = idx >> 8;
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += red[w][rb][e][l];
        const int64_t m = 16 * rb + 4 * (l >> 4) + e;
        const int64_t n = n0 + (l & 15);
        if (m < p.M && n < p.N) p.y[m * p.ldy + n] = __half_as_ushort(__float2half_rn(s));
    }
}

// The cases decoding runs in, written out on their own: RB blocks of 16 activation rows per
// workgroup (blockIdx.y says which 16 RB rows of up to 256), O = 128 (one INT8 group, the last group of K), 32-bit offsets, and either G a
// multiple of four with 8-byte aligned scale rows (TAIL = 3: the last block of four is three INT4
// groups and the INT8 group; the four scales of a batch are one 8-byte load) or G = 4 j + 2 with
// 4-byte aligned scale rows (TAIL = 1: the last block is one INT4 group and the INT8 group; two
// 4-byte loads).  Same sums in the same order as w4a4_gemm_decode_kernel<RB, true,
// true> (eight K-slices of whole four-group blocks, ascending inside a slice, slices added
// 0..7), so the two agree bit for bit.  What differs is the vector work per weight byte and the
// bytes the vector memory path returns to registers (64 per clock and CU), which set the pace here:
//   * a batch is four INT4 groups; the batch that holds the INT8 group (the last block of K, in
//     the last wavefront) is code of its own: no per-slot case analysis, no second half of an INT8 group
//     loaded where there is none;
//   * rows >= M are not zeroed in the operand: an MFMA row depends on its own operand row only, and
//     those rows are never stored;
//   * the accumulator holds 256 x the sum (the nibble widening's factor stays in; the INT8 group's
//     scale products are multiplied by 256 instead, an exact scaling): one multiplication per
//     wavefront at the end instead of one per group;
//   * the scale products of a group and row block are one fp16 MFMA (activation scales of the
//     operand rows against the weight scales of the columns, both in k-slot 0: the result has the
//     layout of the integer tile; a product of two fp16 numbers is exact in fp32), so a lane loads
//     one 8-byte piece of activation scales per batch and row block, not four;
//   * CB blocks of 16 output channels per workgroup share the activation operand: what a
//     workgroup reads of the activations does not depend on how many channels it covers, and with
//     32 rows and more these reads, all of them hits in the L2, are most of what the L2 delivers
//     (about 8 TB/s to all CUs together in these kernels, whatever the shape).  The rows come as
//     whole rows (a load instruction brings four rows of 256 contiguous bytes) and reach the
//     operand layout through a region of LDS of the wavefront's own, like the rows of the staged
//     kernel, one row block at a time.
template <int RB, int CB, bool TILED, int TAIL>
__global__ __launch_bounds__(NT, RB * CB <= 2 ? 4 : 2)     // 128 registers do for two row blocks of one channel block
void w4a4_gemm_decode16_kernel(const GemmParams p)
{
    // per wavefront: 16 staged rows of activation codes (one row block at a time), later its partial sums
    constexpr int WREG = CB * RB * 1024 > kStageWave ? CB * RB * 1024 : kStageWave;
    __shared__ __align__(16) unsigned char stage[NW * WREG];

    const int tid  = threadIdx.x;
    const int lane = tid & 63;
    const int col = lane & 15, kc = lane >> 4;

    const int K4 = p.K - 128, G = p.K >> 7;
    // blockIdx.y: which 16 RB rows of the activations
    const int row0 = (int)blockIdx.y * (16 * RB);
    const int M = min((int)p.M - row0, 16 * RB);          // rows of this workgroup
    const int64_t n0 = (int64_t)blockIdx.x * (TN * CB);
    constexpr bool A8 = TAIL == 3;
    const int nblk    = (G + 3) >> 2;
    const int wave    = slice_of_wave(__builtin_amdgcn_readfirstlane(tid >> 6), p.swap_slices);
    const int g_begin = 4 * (int)((int64_t)wave * nblk / NW);
    const int g_end   = min(G, 4 * (int)((int64_t)(wave + 1) * nblk / NW));

    constexpr uint32_t GSTEP = TILED ? 1024u : 64u;
    const uint32_t nb16 = (uint32_t)((p.N + TN - 1) / TN);
    uint32_t w4o[CB], w8o[CB], wso[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        int64_t wr = n0 + TN * cb + col;                  // clamped: columns >= N are computed and never stored
        wr = wr < p.N ? wr : p.N - 1;
        uint32_t b16 = (uint32_t)blockIdx.x * CB + cb;    // block of 16 channels in the tiled arrays, clamped likewise
        b16 = b16 < nb16 ? b16 : nb16 - 1;
        w4o[cb] = TILED ? b16 * (uint32_t)((G - 1) * 1024) + lane * 16 : (uint32_t)(wr * (K4 >> 1)) + kc * 16;
        w8o[cb] = TILED ? b16 * 2048u + lane * 16 : (uint32_t)(wr * 128) + kc * 16;
        wso[cb] = (uint32_t)wr * (uint32_t)G;
    }
    const uint8_t *w8b = reinterpret_cast<const uint8_t *>(p.w_q8), *a8b = reinterpret_cast<const uint8_t *>(p.a_q8);
    // operand row 16 rb + col of this lane (rows >= M read row 0): INT8 codes and scales
    uint32_t a8o[RB], aso[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const uint32_t ar = row0 + (16 * rb + col < M ? 16 * rb + col : 0);
        a8o[rb] = ar * 128u + kc * 16;
        aso[rb] = ar * (uint32_t)G;
    }
    // staging of the INT4 activation codes: instruction (rb, i) moves rows 16 rb + 4 i .. + 3, lane -> row
    // 16 rb + 4 i + kc, 16-byte chunk `col` of the row's 256 bytes (four groups); rows >= M repeat row M - 1
    uint32_t srow[RB][4];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 16 * rb + 4 * i + kc;
            srow[rb][i] = (uint32_t)(row0 + (r < M ? r : M - 1)) * (uint32_t)(K4 >> 1) + col * 16;
        }
    unsigned char *mine = stage + wave * WREG;
    unsigned char *st_w = mine + kc * kStageRow + col * 16;                    // + 4 i kStageRow
    const unsigned char *st_r = mine + col * kStageRow + kc * 16;              // + 64 d

    float acc[CB][RB][4];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[cb][rb][e] = 0.0f;
    const v4i   zi = {0, 0, 0, 0};
    const v4f32 zf = {0.0f, 0.0f, 0.0f, 0.0f};

    auto batch = [&](int gb, auto has8_c) __attribute__((always_inline)) {
        constexpr bool HAS8 = decltype(has8_c)::value;
        // Every load of the batch is issued before the first is used, the activation rows first: they
        // come from the L2, the weights from HBM, and loads return in order.  In the batch with the
        // INT8 group the chunks of a row past the INT4 groups repeat the last one.
        constexpr int NG4 = HAS8 ? TAIL : 4;               // INT4 groups of the batch
        // (named registers, not an array: the array stayed in scratch memory)
        uint4 s00, s01, s02, s03, s10, s11, s12, s13, s20, s21, s22, s23, s30, s31, s32, s33;
        const uint32_t back = HAS8 && col >= 4 * NG4 ? (uint32_t)(col - (4 * NG4 - 1)) * 16u : 0u;
        auto stage_load = [&](int rb, int i) __attribute__((always_inline)) {
            return *reinterpret_cast<const uint4 *>(p.a_q4 + (srow[rb][i] + (uint32_t)gb * 64u - back));
        };
        s00 = stage_load(0, 0); s01 = stage_load(0, 1); s02 = stage_load(0, 2); s03 = stage_load(0, 3);
        if constexpr (RB > 1) { s10 = stage_load(1, 0); s11 = stage_load(1, 1); s12 = stage_load(1, 2); s13 = stage_load(1, 3); }
        if constexpr (RB > 2) {
            s20 = stage_load(2, 0); s21 = stage_load(2, 1); s22 = stage_load(2, 2); s23 = stage_load(2, 3);
            s30 = stage_load(3, 0); s31 = stage_load(3, 1); s32 = stage_load(3, 2); s33 = stage_load(3, 3);
        }
        uint2 avs[RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) avs[rb] = load_scales<A8>(p.a_scale, aso[rb], gb, G);
        uint4 a8lo[RB], a8hi[RB];
        if constexpr (HAS8) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                a8lo[rb] = *reinterpret_cast<const uint4 *>(a8b + a8o[rb]);
                a8hi[rb] = *reinterpret_cast<const uint4 *>(a8b + (a8o[rb] + 64u));
            }
        }
        // (keeps the activation rows ahead of the weights in the order of the requests)
        __builtin_amdgcn_sched_barrier(0);
        uint2 wvs[CB];
        uint4 wq[CB][4], wx[CB];
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) {
            wvs[cb] = load_scales<A8>(p.w_scale, wso[cb], gb, G);
#pragma unroll
            for (int d = 0; d < NG4; ++d) wq[cb][d] = *reinterpret_cast<const uint4 *>(p.w_q4 + (w4o[cb] + (uint32_t)(gb + d) * GSTEP));
            if constexpr (HAS8) {
                wq[cb][TAIL] = *reinterpret_cast<const uint4 *>(w8b + w8o[cb]);
                wx[cb]       = *reinterpret_cast<const uint4 *>(w8b + (w8o[cb] + GSTEP));
            }
        }
        // (the fence keeps the loads here: left alone the compiler spreads them between the MFMAs
        // to save registers, which turns one memory round trip per batch into several)
        __builtin_amdgcn_sched_barrier(0);
        // one row block at a time through the wavefront's region (LDS instructions of a wavefront
        // execute in order: the next block's writes come after this block's reads)
        uint4 aq[RB][4];
        auto through_lds = [&](auto rbc, const uint4 &r0, const uint4 &r1, const uint4 &r2, const uint4 &r3) __attribute__((always_inline)) {
            constexpr int rb = decltype(rbc)::value;
            *reinterpret_cast<uint4 *>(st_w)                  = r0;
            *reinterpret_cast<uint4 *>(st_w + 4 * kStageRow)  = r1;
            *reinterpret_cast<uint4 *>(st_w + 8 * kStageRow)  = r2;
            *reinterpret_cast<uint4 *>(st_w + 12 * kStageRow) = r3;
#pragma unroll
            for (int d = 0; d < NG4; ++d) aq[rb][d] = *reinterpret_cast<const uint4 *>(st_r + 64 * d);
        };
        through_lds(std::integral_constant<int, 0>(), s00, s01, s02, s03);
        if constexpr (RB > 1) through_lds(std::integral_constant<int, 1>(), s10, s11, s12, s13);
        if constexpr (RB > 2) {
            through_lds(std::integral_constant<int, 2>(), s20, s21, s22, s23);
            through_lds(std::integral_constant<int, 3>(), s30, s31, s32, s33);
        }
        if (kc != 0) {                                    // k-slots 4 .. 15 of the scale MFMA stay empty
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) avs[rb] = make_uint2(0, 0);
        }
        // (what needs the weights stays behind what does not)
        __builtin_amdgcn_sched_barrier(0);
        if (kc != 0) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) wvs[cb] = make_uint2(0, 0);
        }

        auto int4_group = [&](auto dc) __attribute__((always_inline)) {
            constexpr int D = decltype(dc)::value;
            v4i b0[CB], b1[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) { b0[cb] = widen_lo(wq[cb][D]); b1[cb] = widen_hi(wq[cb][D]); }
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const v4i x0 = widen_lo(aq[rb][D]), x1 = widen_hi(aq[rb][D]);
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    v4i c = __builtin_amdgcn_mfma_i32_16x16x64_i8(x0, b0[cb], zi, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_i32_16x16x64_i8(x1, b1[cb], c, 0, 0, 0);
                    const v4f32 sc = __builtin_amdgcn_mfma_f32_16x16x16f16(scale_operand<D>(avs[rb]), scale_operand<D>(wvs[cb]), zf, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[cb][rb][e] = fmaf((float)c[e], sc[e], acc[cb][rb][e]);
                }
            }
        };
        int4_group(std::integral_constant<int, 0>());
        if constexpr (NG4 > 1) int4_group(std::integral_constant<int, 1>());
        if constexpr (NG4 > 2) int4_group(std::integral_constant<int, 2>());
        if constexpr (NG4 > 3) int4_group(std::integral_constant<int, 3>());
        if constexpr (HAS8) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) {
                    v4i c = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i, a8lo[rb]), __builtin_bit_cast(v4i, wq[cb][TAIL]), zi, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i, a8hi[rb]), __builtin_bit_cast(v4i, wx[cb]), c, 0, 0, 0);
                    const v4f32 sc = __builtin_amdgcn_mfma_f32_16x16x16f16(scale_operand<TAIL>(avs[rb]), scale_operand<TAIL>(wvs[cb]), zf, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[cb][rb][e] = fmaf((float)c[e], 256.0f * sc[e], acc[cb][rb][e]);
                }
        }
    };

    const int g_plain = wave == NW - 1 ? g_end - (TAIL + 1) : g_end;
    for (int gb = g_begin; gb < g_plain; gb += 4) batch(gb, std::false_type());
    if (wave == NW - 1) batch(G - (TAIL + 1), std::true_type());

    // the eight K-slices meet in LDS (each wavefront's region, its operand reads are complete) and
    // are added in slice order
    float *red = reinterpret_cast<float *>(mine);        // [channel block][row block][register][lane]
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[((cb * RB + rb) * 4 + e) * 64 + lane] = acc[cb][rb][e] * (1.0f / 256.0f);
    __syncthreads();
    for (int idx = tid; idx < CB * RB * 4 * 64; idx += NT) {
        const int l = idx & 63, e = (idx >> 6) & 3, rb = (idx >> 8) % RB, cb = (idx >> 8) / RB;
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < NW; ++w) s += reinterpret_cast<const float *>(stage + w * WREG)[idx];
        const int m = 16 * rb + 4 * (l >> 4) + e;
        const int64_t n = n0 + TN * cb + (l & 15);
        if (m < M && n < p.N) p.y[(int64_t)(row0 + m) * p.ldy + n] = __half_as_ushort(__float2half_rn(s));
    }
}

constexpr int kLeastSet = 32;               // rows of the smallest set of workgroups of the next kernel, which its rules also count work in

// Many blocks of channels per compute unit, 17 to 256 rows, K from 3840 to 12288 (30 to 96 groups): a workgroup takes 16 RB rows and a
// run of channel blocks, and every wavefront keeps the activation operand of its K-slice (NBK blocks of four groups, or one less) in
// registers for all of them.  w4a4_gemm_decode16_kernel reads the activations again for each block or two, more bytes from the L2 than
// the weights are, and every workgroup pays its own start and its own meeting of slices; here only weights stream, those of
// the next two blocks in flight while one is multiplied.  Same sums in the same order: the same bits.
// With one block of groups per wavefront (K up to 4096) the operand is kept widened to bytes: the widening is 24 of the 60 vector
// instructions of a group and 32 rows, and paid for each block of channels it kept 64 rows from one pass over the weights.  Canonical weights
// from memory, K = 4096, us, widened for every block (two sets of 32 rows beyond 32) and kept: N = 22016: M = 17 15.2 / 14.3, 32 15.8 / 15.0,
// 40 20.4 / 16.6, 64 21.0 / 19.0; N = 28672: M = 40 25.0 / 19.2, 64 25.6 / 21.3; N = 11008: M = 33 12.2 / 10.5.  K = 3840 (TAIL = 1) with 32 rows
// is as fast either way with few rows and 3 % slower with all 32 (N = 28672 18.1 / 18.6): not kept there.
// With two blocks of groups (K up to 8192) and TAIL = 3 the weights of one block of channels are in registers instead of two, every piece requested for
// the next where it has been used, and all activations are kept widened (254 registers); TAIL = 1, whose last block has fewer of them in flight, is 1 to 2 %
// slower so and has two sets of weights and the first block of groups kept.  None kept, the first, and all: K = 8192: N = 22016: M = 32 30.2 / 29.0 / 28.5, 64
// 40.8 / 38.3 / 37.5; N = 11008, M = 64 25.9 / 24.3 / 22.8; K = 5120, N = 13824, M = 40 19.2 / 18.3 / 16.9.  Three blocks (K up to 12288): widened every time,
// one set of weights (two spill 28 registers with TAIL = 3, and without spills K = 11008, N = 11008, M = 64 takes 35.1, 31.6 so).
// What bounds it now: the weights (9.0 us for 22016 x 4096 when only read; 4.4 TB/s by the slope over N) behind a start of 5 us with 32 rows
// and 7 with 64 in which the activations arrive.  The first block's weights requested ahead of the activations: 1 us slower.  Weights
// three blocks ahead: no faster.
// A wavefront with one block where others have two (K from 4352 to 7680) is code of its own and requests only what it uses.  (With a
// second request of its first block in the missing one's place six of eight wavefronts read their weights twice at K = 5120:
// M = 33, N = 13824 22.8 us, 20.3 so, w4a4_gemm_decode16_kernel 22.6; M = 32, N = 16400 19.5, 17.7, 18.3; K = 4352, M = 33, N = 13824
// 22.1, 16.6, 19.3.)
template <int RB, int NBK, int TAIL>
__global__ __launch_bounds__(NT, 2)
void w4a4_gemm_decode_resident_kernel(const GemmParams p)
{
    // one set of weights in registers (three blocks, two with TAIL = 3 or 48 rows), refilled piece by piece for the next block of channels where they have been used
    constexpr bool SINGLE = NBK == 3 || (NBK == 2 && (TAIL == 3 || RB > 2));
    // whether the widened activations of block j stay
    constexpr auto keep = [](int j) constexpr { return NBK == 1 ? RB > 2 || TAIL == 3 : NBK == 2 && RB == 2 ? TAIL == 3 || j == 0 : false; };
    // [parity of the pair of channel blocks][which of the pair][K-slice][row block, lane, register]
    constexpr int RED = RB * 256;
    __shared__ __align__(16) float red[4 * NW * RED];

    const int tid  = threadIdx.x;
    const int lane = tid & 63;
    const int col = lane & 15, kc = lane >> 4;
    const int K4 = p.K - 128, G = p.K >> 7;
    const int row0 = (int)blockIdx.y * (16 * RB);
    const int M = min((int)p.M - row0, 16 * RB);          // rows of this workgroup
    constexpr bool A8 = TAIL == 3;
    const int nblk    = (G + 3) >> 2;
    const int wave    = slice_of_wave(__builtin_amdgcn_readfirstlane(tid >> 6), p.swap_slices);
    const int g_begin = 4 * (int)((int64_t)wave * nblk / NW);
    const int g_end   = min(G, 4 * (int)((int64_t)(wave + 1) * nblk / NW));
    const uint8_t *w8b = reinterpret_cast<const uint8_t *>(p.w_q8), *a8b = reinterpret_cast<const uint8_t *>(p.a_q8);
    // this workgroup's blocks of 16 channels
    const int nb16  = (int)((p.N + TN - 1) / TN);
    const int first = (int)((int64_t)blockIdx.x * nb16 / gridDim.x), last = (int)((int64_t)(blockIdx.x + 1) * nb16 / gridDim.x);

    const v4i   zi = {0, 0, 0, 0};
    const v4f32 zf = {0.0f, 0.0f, 0.0f, 0.0f};

    // NB: this wavefront's blocks of groups (NBK, or one less where eight K-slices do not share them evenly); the last wavefront
    // has NBK, and its last block holds the INT8 group
    auto run = [&](auto has8_c, auto blocks_c) __attribute__((always_inline)) {
        constexpr bool HAS8 = decltype(has8_c)::value;
        constexpr int  NB   = decltype(blocks_c)::value;
        int gb[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) gb[j] = g_begin + 4 * j;
        auto ng4 = [](int j) constexpr { return HAS8 && j == NB - 1 ? TAIL : 4; };       // INT4 groups of block j

        struct Weights { uint4 q[NB][4], x; uint2 s[NB]; };
        struct Place { uint32_t w4o, w8o, so; };                // of a block of channels' weights
        auto place = [&](int blk) __attribute__((always_inline)) -> Place {
            blk = blk < last ? blk : last - 1;            // past the end: the last block once more, not used
            int64_t wr = (int64_t)blk * TN + col;         // clamped: columns >= N are computed and never stored
            wr = wr < p.N ? wr : p.N - 1;
            return {(uint32_t)(wr * (K4 >> 1)) + kc * 16, (uint32_t)(wr * 128) + kc * 16, (uint32_t)wr * (uint32_t)G};
        };
        auto fetch_piece = [&](Weights &w, const Place &at, int j, int d) __attribute__((always_inline)) {
            if (HAS8 && j == NB - 1 && d == TAIL) {
                w.q[j][d] = *reinterpret_cast<const uint4 *>(w8b + at.w8o);
                w.x       = *reinterpret_cast<const uint4 *>(w8b + (at.w8o + 64u));
            } else if (d < ng4(j)) {
                w.q[j][d] = *reinterpret_cast<const uint4 *>(p.w_q4 + (at.w4o + (uint32_t)(gb[j] + d) * 64u));
            }
        };
        auto fetch = [&](Weights &w, int blk) __attribute__((always_inline)) {
            const Place at = place(blk);
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                w.s[j] = load_scales<A8>(p.w_scale, at.so, gb[j], G);
#pragma unroll
                for (int d = 0; d < 4; ++d) fetch_piece(w, at, j, d);
            }
        };
        Weights wa, wb;

        // the activation operand of the wavefront's groups (row 16 rb + col of this lane; rows >= M read row 0 and are never
        // stored), ahead of the weights in the order of the requests
        uint4 aq[NB][RB][4], ax[RB];
        uint2 avs[NB][RB];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const uint32_t ar = row0 + (16 * rb + col < M ? 16 * rb + col : 0);
            const uint32_t a4o = ar * (uint32_t)(K4 >> 1) + kc * 16, a8o = ar * 128u + kc * 16;
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                avs[j][rb] = load_scales<A8>(p.a_scale, ar * (uint32_t)G, gb[j], G);
#pragma unroll
                for (int d = 0; d < ng4(j); ++d) aq[j][rb][d] = *reinterpret_cast<const uint4 *>(p.a_q4 + (a4o + (uint32_t)(gb[j] + d) * 64u));
            }
            if constexpr (HAS8) {
                aq[NB - 1][rb][TAIL] = *reinterpret_cast<const uint4 *>(a8b + a8o);
                ax[rb]               = *reinterpret_cast<const uint4 *>(a8b + (a8o + 64u));
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // (every wavefront's activations, hits in the L2, before any weights: loads return in order)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        fetch(wa, first);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!SINGLE) fetch(wb, first + 1);
        __builtin_amdgcn_sched_barrier(0);
        // (KEEP: widened once, for all channel blocks)
        v4i xa[NB][RB][4][2];
        auto widened = [&](int j, int rb, int d, int half) __attribute__((always_inline)) -> v4i {
            if (HAS8 && j == NB - 1 && d == TAIL) return __builtin_bit_cast(v4i, half ? ax[rb] : aq[j][rb][d]);
            return half ? widen_hi(aq[j][rb][d]) : widen_lo(aq[j][rb][d]);
        };
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                if (kc != 0) avs[j][rb] = make_uint2(0, 0);       // k-slots 4 .. 15 of the scale MFMA stay empty
                if (keep(j))
#pragma unroll
                    for (int d = 0; d < ng4(j) + (HAS8 && j == NB - 1 ? 1 : 0); ++d)
#pragma unroll
                        for (int half = 0; half < 2; ++half) xa[j][rb][d][half] = widened(j, rb, d, half);
            }

        auto step = [&](Weights &w, int blk, int slot_of) __attribute__((always_inline)) {
            const Place next = place(SINGLE ? blk + 1 : blk);
            float acc[RB][4];
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[rb][e] = 0.0f;
            // (hoisted out of the loop the widened codes would take twice the registers)
#pragma unroll
            for (int j = 0; j < NB; ++j)
                if (!keep(j))
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
                        for (int d = 0; d < ng4(j); ++d)
                            asm volatile("" : "+v"(aq[j][rb][d].x), "+v"(aq[j][rb][d].y), "+v"(aq[j][rb][d].z), "+v"(aq[j][rb][d].w));
                        asm volatile("" : "+v"(avs[j][rb].x), "+v"(avs[j][rb].y));
                    }
            auto group = [&](auto jc, auto dc) __attribute__((always_inline)) {
                constexpr int J = decltype(jc)::value, D = decltype(dc)::value;
                constexpr bool INT8 = HAS8 && J == NB - 1 && D == TAIL;
                const v4i b0 = INT8 ? __builtin_bit_cast(v4i, w.q[J][D]) : widen_lo(w.q[J][D]);
                const v4i b1 = INT8 ? __builtin_bit_cast(v4i, w.x) : widen_hi(w.q[J][D]);
                const uint2 ws = kc != 0 ? make_uint2(0, 0) : w.s[J];
                if constexpr (SINGLE) {
                    fetch_piece(w, next, J, D);
                    if constexpr (D == 3 || (HAS8 && J == NB - 1 && D == TAIL)) w.s[J] = load_scales<A8>(p.w_scale, next.so, gb[J], G);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int rb = 0; rb < RB; ++rb) {
                    const v4i x0 = keep(J) ? xa[J][rb][D][0] : widened(J, rb, D, 0), x1 = keep(J) ? xa[J][rb][D][1] : widened(J, rb, D, 1);
                    v4i c = __builtin_amdgcn_mfma_i32_16x16x64_i8(x0, b0, zi, 0, 0, 0);
                    c = __builtin_amdgcn_mfma_i32_16x16x64_i8(x1, b1, c, 0, 0, 0);
                    const v4f32 sc = __builtin_amdgcn_mfma_f32_16x16x16f16(scale_operand<D>(avs[J][rb]), scale_operand<D>(ws), zf, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[rb][e] = fmaf((float)c[e], INT8 ? 256.0f * sc[e] : sc[e], acc[rb][e]);
                }
            };
            auto slot = [&](auto jc) __attribute__((always_inline)) {
                constexpr int J = decltype(jc)::value;
                group(jc, std::integral_constant<int, 0>());
                group(jc, std::integral_constant<int, 1>());
                if constexpr (!(HAS8 && J == NB - 1 && TAIL == 1)) {
                    group(jc, std::integral_constant<int, 2>());
                    group(jc, std::integral_constant<int, 3>());
                }
            };
            slot(std::integral_constant<int, 0>());
            if constexpr (NB > 1) slot(std::integral_constant<int, 1>());
            if constexpr (NB > 2) slot(std::integral_constant<int, 2>());
            // the requests for the block after the next, as soon as these registers are free
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (!SINGLE) fetch(w, blk + 2);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
                *reinterpret_cast<float4 *>(&red[(slot_of * NW + wave) * RED + (rb * 64 + lane) * 4]) =
                    make_float4(acc[rb][0] * (1.0f / 256.0f), acc[rb][1] * (1.0f / 256.0f), acc[rb][2] * (1.0f / 256.0f), acc[rb][3] * (1.0f / 256.0f));
        };
        // The eight K-slices meet in LDS and are added in slice order, two blocks of channels at a time: one barrier for a pair
        // (its part of LDS was last read two pairs ago, before the barrier in between).
        int parity = 0;
        for (int blk = first; blk < last; blk += 2, parity ^= 2) {
            step(wa, blk, parity);
            if (blk + 1 < last) step(SINGLE ? wa : wb, blk + 1, parity + 1);
            __syncthreads();
            for (int idx = tid; idx < RB * 256; idx += NT) {      // two outputs each: rows m and m + 1 of a column
                const int one = idx >= RB * 128 ? 1 : 0, t = idx - one * RB * 128;
                if (blk + one >= last) break;
                float s0 = 0.0f, s1 = 0.0f;
#pragma unroll
                for (int v = 0; v < NW; ++v) {
                    const float2 f = *reinterpret_cast<const float2 *>(&red[((parity + one) * NW + v) * RED + 2 * t]);
                    s0 += f.x;
                    s1 += f.y;
                }
                const int l = (t >> 1) & 63, rb = t >> 7, m = 16 * rb + 4 * (l >> 4) + 2 * (t & 1);
                const int64_t n = (int64_t)(blk + one) * TN + (l & 15);
                uint16_t *y = p.y + (int64_t)(row0 + m) * p.ldy + n;
                if (n < p.N) {
                    if (m < M) y[0] = __half_as_ushort(__float2half_rn(s0));
                    if (m + 1 < M) y[p.ldy] = __half_as_ushort(__float2half_rn(s1));
                }
            }
        }
    };
    if (wave == NW - 1) {
        run(std::true_type(), std::integral_constant<int, NBK>());
    } else {
        if constexpr (NBK > 1)
            if (g_end - g_begin < 4 * NBK) return run(std::false_type(), std::integral_constant<int, NBK - 1>());
        run(std::false_type(), std::integral_constant<int, NBK>());
    }
}

// One block of activation rows (M <= 16): decode_staged_body of atom_gemm_decode_staged.h.
template <int SI, bool TILED, int TAIL>
__global__ __launch_bounds__(NT, 6)
void w4a4_gemm_decode_staged_kernel(const GemmParams p)
{
    __shared__ __align__(16) unsigned char stage[kStageBytes];
    decode_staged_body<SI, TILED, TAIL, false>(p, (int)blockIdx.x, stage, NoWait());
}

// Canonical weights, 17 to 64 rows and K such that every wavefront has one or two blocks of four groups (registers for the
// activations): the kernel that keeps the activations, with one block where a compute unit has more than four blocks of 16 channels and 32
// rows to do.  Up to there the other kernels' workgroups are resident together or nearly so, and the start counts: K = 4096, that
// kernel and the others, M = 32: N = 8192 8.5 / 7.8 us, 11008 9.7 / 10.0, 22016 15.0 / 17.2; M = 64: N = 8192 10.2 / 9.0, 9999 11.7 / 14.9.
// With two, as soon as a compute unit has more than one block of channels, up to 24 rows two (K = 7680, M = 17, N = 8000, with the front end and weights from the last-level
// cache 12.8 / 12.4): K = 8192: N = 4300: M = 32 12.0 / 13.5, 64 13.5 / 16.0, N = 13824, M = 32 20.5 / 25.6;
// K = 4864: N = 6000: M = 32 9.2 / 9.6, 64 10.3 / 11.1; N = 16384, M = 32 14.4 / 18.0; with fewer blocks: N = 3000: M = 32 6.3 / 6.2.
// Re-tiled weights stay with w4a4_gemm_decode16_kernel.  Canonical and re-tiled, us: K = 4096, N = 22016: M = 32 14.6 / 17.1, M = 64 19.7 /
// 23.9; K = 5120, N = 28672, M = 64 31.0 / 38.8; K = 8192: M = 32, N = 28672 32.2 / 40.1, M = 64, N = 13824 25.3 / 26.5, but M = 33, N = 8192 15.6 / 14.4.
bool resident(int64_t M, int64_t N, int K, int64_t cus)
{
    const int     nblk = ((K >> 7) + 3) >> 2;
    const int64_t blocks = (N + TN - 1) / TN, sets = (M + kLeastSet - 1) / kLeastSet;
    return M > 16 && M <= 64 && nblk >= NW && nblk <= 2 * NW && (nblk > NW ? blocks > (M > 24 ? 1 : 2) * cus : blocks * sets > 4 * cus);
}

// The same with K from 8448 to 12288, three blocks of groups to a wavefront.  This kernel and w4a4_gemm_decode16_kernel, us: K = 11008: N = 22016: M = 20 36.7 / 44.5,
// 64 51.5 / 60.0; N = 8400, M = 64 27.5 / 38.8; K = 12288, N = 16384, M = 20 30.0 / 35.5.  On the other side, with the front end and weights from the last-level cache,
// K = 9216, M = 20: N = 9000 21.0 / 19.4, 13824 23.3 / 21.7; K = 12288, M = 40, N = 4300 21.5 / 20.2.
bool resident_three(int64_t M, int64_t N, int K, int64_t cus)
{
    const int     nblk = ((K >> 7) + 3) >> 2;
    const int64_t blocks = (N + TN - 1) / TN;
    return M > 16 && M <= 64 && nblk > 2 * NW && nblk <= 3 * NW && blocks > (M > 32 ? 2 : K > 10240 ? 3 : 4) * cus;
}

// Rounds of workgroups over the compute units of w4a4_gemm_decode16_kernel on more than 64 rows, as launch_common picks them.
int64_t decode_rounds(int64_t M, int64_t N, int64_t cus)
{
    const int64_t blocks = (N + TN - 1) / TN, yb = (M + 63) / 64;
    const int64_t wgs = blocks * yb <= cus ? blocks * yb : (blocks + 1) / 2 * yb;
    return (wgs + cus - 1) / cus;
}

// Workgroups of a set: a multiple of eight, where that leaves nine tenths of them, so that those with the same channels run on the same XCD and read the weights
// through one L2.  As many as there are room for and a multiple of eight: three sets (85, 80), M = 96, K = 8192, N = 11008 33.4 / 29.3 us, five (51, 48), M =
// 160, K = 5120, N = 8192 24.9 / 22.5, six (42, 40), M = 192, K = 8192, N = 22016 85.3 / 86.2, N = 8192 38.0 / 37.0; but seven (36, 32), M = 224, K = 5120, N = 8192 28.9 / 29.8.
int64_t set_width(int64_t cus, int64_t sets)
{
    const int64_t w = cus / sets, even = w & ~(int64_t)7;
    return 10 * even >= 9 * w ? even : w;
}

// Rows of a set of workgroups beyond 64 rows: K up to 4096 64, or 48 where these are as many sets; beyond 32, or 48 where these are two sets instead of three or
// three instead of five and every wavefront has two blocks of groups, K over 7680 (sets of 32 and 48, us: K = 8192: M = 96, N = 22016 51.1 / 45.1, M = 140, N =
// 13824 46.9 / 42.4; but K = 7168: M = 80, N = 11008 24.4 / 26.1, M = 136, N = 8192 27.0 / 28.8; K = 5120: M = 96, N = 11008 19.9 / 21.2).
int64_t set_rows(int64_t M, int K)
{
    if (K > 960 * NW && K <= 1024 * NW && (M <= 96 || (M > 128 && M <= 144))) return 48;
    return K > 512 * NW ? 32 : (M + 47) / 48 <= (M + 63) / 64 ? 48 : 64;
}

// 65 to 256 rows, the same K: sets of workgroups share the compute units, and a compute unit has n blocks of 16 channels.  With K up to 8192 it is ahead of
// w4a4_gemm_decode16_kernel (up to three rounds of its workgroups) wherever it may run; against the tiled kernels, and with three blocks of groups
// against both, it is by the estimates of both: fitted, us, 5.0 + 1.75 n with sets of 48 rows, 5.5 + 2.1 n of 64; with K beyond 4096 4 + 0.0006 K + (0.3 +
// 0.000244 K) n (1.4 times that by n with sets of 48), beyond 8192 9.5 + (0.95 + 0.000217 K) n; a round of w4a4_gemm_decode16_kernel 0.00145 K, and 3; the tiled kernels' is a tenth low with one
// round of tiles and weights from HBM, beyond 8192 channels only with tiles of 64 x 64.  Tiled or w4a4_gemm_decode16_kernel, and this: K = 4096: N = 8192: M = 96
// 15.9, 12.0, 256 26.5, 21.3; N = 13824: M = 65 25.7, 16.4, 128 27.9, 20.5, but 256 31.1, 32.3; N = 22016: M = 128 32.5, 28.9, 192 52.6, 40.5; K = 5120, N =
// 13824: M = 128 34.3, 27.6, but 192 35.4, 40.9; K = 8192: N = 13824: M = 128 61.2, 40.6, but 192 53.9, 58.9; N = 22016: M = 192 96.8, 86.3; K = 11008: N =
// 11008: M = 96 52.9, 40.5, but 192 66.2, 68.2; N = 4096: M = 160 33.3, 29.2, but 96 19.3, 23.1; N = 13824, M = 128 79.7, 57.2.
bool resident_sets(int64_t M, int64_t N, int K, int64_t cus)
{
    const int     nblk = ((K >> 7) + 3) >> 2;
    const int64_t blocks = (N + TN - 1) / TN, rows = set_rows(M, K), sets = (M + rows - 1) / rows;
    if (M <= 64 || M > 256 || nblk < NW || nblk > 3 * NW || blocks * ((M + kLeastSet - 1) / kLeastSet) <= 4 * cus || sets > cus) return false;
    const int64_t rounds = decode_rounds(M, N, cus);
    const float n = (float)((blocks + set_width(cus, sets) - 1) / set_width(cus, sets)), k = (float)K;
    if (nblk > 2 * NW) {
        const float us = 9.5f + (0.95f + 0.000217f * k) * n;
        return us < (rounds <= 3 ? 3.0f + 0.00145f * k * (float)rounds : (((M + 63) / 64) * ((N + 63) / 64) <= 2 * cus ? 1.1f : 1.0f) * tiles_us(M, N, K, cus));
    }
    if (rounds <= 3) return true;
    const float us = nblk > NW  ? 4.0f + 0.0006f * k + (rows == 48 ? 1.4f : 1.0f) * (0.3f + 0.000244f * k) * n
                   : rows == 48 ? 5.0f + 1.75f * n : 5.5f + 2.1f * n;
    return us < (((M + 127) / 128) * ((N + 127) / 128) <= cus ? 1.1f : 1.0f) * tiles_us(M, N, K, cus);
}

// Rows of a set of workgroups of the kernel that keeps the activations; 0: another kernel runs.
// Beyond 32 rows a workgroup takes all of them (K up to 4096), or there are two sets of workgroups of 32 rows each.  A lone set reads the
// weights once but starts later (three or four blocks of rows to fetch and widen), and the blocks of channels of a compute unit
// are whole numbers, one and two of them to the same N: fitted, K = 4096, us, 4.2 + 2.2 n for 33 to 48 rows and 4.5 + 2.45 n
// beyond, n the most blocks that a workgroup has, and 1.6 + 1.78 n for two sets.  Measured at M = 64, one set and two: N = 8208 11.4 / 10.1,
// 10000 12.2 / 10.9, 12288 12.3 / 11.9, 14000 14.2 / 13.5, 16384 14.4 / 15.9; at M = 33: 10.1 / 9.7, 10.5 / 10.2, 10.7 / 11.2, 12.0 / 12.6, 12.9 / 15.2.
// With K from 4352 to 8192 33 to 48 rows are one set as soon as a workgroup of two has six blocks; two sets and one, M = 40: K = 8192: N = 8192 16.2 / 16.2, 11008
// 22.0 / 20.0, 22016 35.6 / 31.8; K = 5120: N = 8192 11.3 / 11.8, 11008 15.0 / 14.7, 28672 31.2 / 27.3.  (64 rows in one: K = 8192, N = 22016 37.6 / 38.7.)
int64_t resident_rows(int64_t M, int64_t N, int K, int64_t cus)
{
    if (!resident(M, N, K, cus) && !resident_three(M, N, K, cus) && !resident_sets(M, N, K, cus)) return 0;
    if (M <= 32) return kLeastSet;
    if (M > 64) return set_rows(M, K);
    const int64_t blocks = (N + TN - 1) / TN, one = (blocks + cus - 1) / cus, two = (blocks + cus / 2 - 1) / (cus / 2);
    if (K > 512 * NW) return M > 48 || K > 1024 * NW || two < 6 ? kLeastSet : 48;
    if (M <= 48) return 160 + 178 * two < 420 + 220 * one ? kLeastSet : 48;
    return 160 + 178 * two < 450 + 245 * one ? kLeastSet : 64;
}

template <int TAIL>
void launch_resident(const GemmParams &p, int64_t rows, hipStream_t stream)
{
    const unsigned sets = (unsigned)((p.M + rows - 1) / rows);
    auto kern = p.K > 1024 * NW ? &w4a4_gemm_decode_resident_kernel<2, 3, TAIL>
              : p.K > 512 * NW ? (rows == 48 ? &w4a4_gemm_decode_resident_kernel<3, 2, TAIL> : &w4a4_gemm_decode_resident_kernel<2, 2, TAIL>)
              : rows == 32     ? &w4a4_gemm_decode_resident_kernel<2, 1, TAIL>
              : rows == 48     ? &w4a4_gemm_decode_resident_kernel<3, 1, TAIL>
                               : &w4a4_gemm_decode_resident_kernel<4, 1, TAIL>;
    hipLaunchKernelGGL(kern, dim3((unsigned)set_width(atom_launch::compute_units(), sets), sets), dim3(NT), 0, stream, p);   // (fewer workgroups than blocks: every one has some)
}

// Workgroups along the channels of w4a4_gemm_decode16_kernel in `sets` sets of rows: a multiple of eight, the last ones without channels of their own, where
// all of them keep a compute unit or are in rounds anyway: those with the same channels then run on the same XCD and read the weights through one L2.  As
// they come and so: K = 8192, N = 1000: M = 64 5.9 / 5.2 us, 128 7.6 / 6.6; K = 11008, M = 33: N = 1000 7.2 / 6.5, N = 2000 9.7 / 9.2.
unsigned channel_groups(int64_t groups, int64_t sets, int64_t cus)
{
    const int64_t even = (groups + 7) & ~(int64_t)7;
    return (unsigned)(sets > 1 && (even * sets <= cus || groups * sets > cus) ? even : groups);
}

// The kernels of the common case: M <= 16 staged, else blocks of 16 rows.
template <bool TILED, int TAIL>
void launch_common(const GemmParams &p, unsigned blocks, hipStream_t stream)
{
    if (p.M <= 4)       hipLaunchKernelGGL((w4a4_gemm_decode_staged_kernel<1, TILED, TAIL>), dim3(blocks), dim3(NT), 0, stream, p);
    else if (p.M <= 8)  hipLaunchKernelGGL((w4a4_gemm_decode_staged_kernel<2, TILED, TAIL>), dim3(blocks), dim3(NT), 0, stream, p);
    else if (p.M <= 16) hipLaunchKernelGGL((w4a4_gemm_decode_staged_kernel<4, TILED, TAIL>), dim3(blocks), dim3(NT), 0, stream, p);
    // As many sets of workgroups as give every one of them a compute unit of its own, of 16 or of 32 rows: fewer rows in the chain of a
    // wavefront.  Sets of 64 (up to 32 rows: 32), 32 and 16 rows, weights from HBM, us: M = 64: K = 4096, N = 1000 5.6, 4.2, 4.0, N = 2048 5.7, 4.3,
    // 4.7; K = 8192, N = 1000 8.6, 6.2, 5.8, N = 2048 11.5, 7.8, 8.4; M = 32: K = 4096, N = 2048 -, 4.2, 3.6, N = 4096 -, 5.3, 5.6; K = 11008, N =
    // 2048 -, 10.8, 8.5, N = 4096 -, 11.6, 13.0; M = 128: K = 8192, N = 500 8.5, 6.1, 4.9.  (At both N = 2048 with 64 rows and N = 4096 with
    // 32 sets of 16 are two to a compute unit.)
    else if ((int64_t)blocks * ((p.M + 15) / 16) <= atom_launch::compute_units())
        hipLaunchKernelGGL((w4a4_gemm_decode16_kernel<1, 1, TILED, TAIL>), dim3(channel_groups(blocks, (p.M + 15) / 16, atom_launch::compute_units()), (unsigned)((p.M + 15) / 16)), dim3(NT), 0, stream, p);
    else if (const int64_t rows = TILED ? 0 : resident_rows(p.M, p.N, p.K, atom_launch::compute_units())) launch_resident<TAIL>(p, rows, stream);
    else if (p.M <= 32) hipLaunchKernelGGL((w4a4_gemm_decode16_kernel<2, 1, TILED, TAIL>), dim3(blocks), dim3(NT), 0, stream, p);
    // Four row blocks (and with more than 64 rows further sets of workgroups for rows 64 and up: the
    // weights of a channel block are then read again, out of the caches): two channel
    // blocks per workgroup once there is more than one workgroup per CU otherwise.  M = 64, K = 4096,
    // weights from HBM: N = 4096 6.6 us with one, 8.2 us with two; N = 5120 10.9 / 8.3; N = 8192 11.5 /
    // 9.1; N = 11008 16.2 / 15.3; N = 22016 30.8 / 23.7.
    else {
        const unsigned yb = (unsigned)((p.M + 63) / 64), y32 = (unsigned)((p.M + 31) / 32);
        if ((int64_t)blocks * y32 <= atom_launch::compute_units())
            hipLaunchKernelGGL((w4a4_gemm_decode16_kernel<2, 1, TILED, TAIL>), dim3(channel_groups(blocks, y32, atom_launch::compute_units()), y32), dim3(NT), 0, stream, p);
        else if ((int64_t)blocks * yb <= atom_launch::compute_units())
            hipLaunchKernelGGL((w4a4_gemm_decode16_kernel<4, 1, TILED, TAIL>), dim3(channel_groups(blocks, yb, atom_launch::compute_units()), yb), dim3(NT), 0, stream, p);
        else
            hipLaunchKernelGGL((w4a4_gemm_decode16_kernel<4, 2, TILED, TAIL>), dim3(channel_groups((blocks + 1) / 2, yb, atom_launch::compute_units()), yb), dim3(NT), 0, stream, p);
    }
}

// Re-tiling of the canonical weight codes for the TILED variants: one workgroup per block of 16
// rows; rows past N are zeros.
__global__ __launch_bounds__(256)
void tile_weight_kernel(const uint8_t *__restrict__ q4, const int8_t *__restrict__ q8, int64_t N, int K4h, int O,
                        uint8_t *__restrict__ t4, uint8_t *__restrict__ t8)
{
    const int64_t blk = blockIdx.x;
    const int G4 = K4h >> 6, G8 = O >> 7;
    // INT4: piece p = (group, lane) -> row blk*16 + (lane & 15), bytes [64 g + 16 (lane >> 4), +16)
    for (int p = threadIdx.x; p < G4 * 64; p += 256) {
        const int g = p >> 6, l = p & 63;
        const int64_t row = blk * 16 + (l & 15);
        uint4 v = make_uint4(0, 0, 0, 0);
        if (row < N) v = *reinterpret_cast<const uint4 *>(q4 + row * K4h + g * 64 + (l >> 4) * 16);
        *reinterpret_cast<uint4 *>(t4 + (blk * G4 + g) * 1024 + l * 16) = v;
    }
    // INT8: piece (group, half, lane) -> row, bytes [128 g + 64 half + 16 (lane >> 4), +16)
    for (int p = threadIdx.x; p < G8 * 128; p += 256) {
        const int g = p >> 7, h = (p >> 6) & 1, l = p & 63;
        const int64_t row = blk * 16 + (l & 15);
        uint4 v = make_uint4(0, 0, 0, 0);
        if (row < N) v = *reinterpret_cast<const uint4 *>(q8 + row * O + g * 128 + h * 64 + (l >> 4) * 16);
        *reinterpret_cast<uint4 *>(t8 + ((blk * G8 + g) * 2 + h) * 1024 + l * 16) = v;
    }
}

}  // namespace

// Whether a decode GEMM of the common case on canonical weights takes the kernel that keeps the activations, and with how many rows to a set (0: another kernel), as
// its tests ask it.
extern "C" int atom_internal_decode_resident(int64_t M, int64_t N, int K, int64_t cus) { return resident(M, N, K, cus); }
extern "C" int atom_internal_decode_resident_sets(int64_t M, int64_t N, int K, int64_t cus) { return resident_sets(M, N, K, cus); }
extern "C" int atom_internal_decode_resident_rows(int64_t M, int64_t N, int K, int64_t cus) { return (int)resident_rows(M, N, K, cus); }

namespace atom_gemm {

hipError_t launch_tile_weight(const void *q4, const void *q8, int64_t N, int K, int O, void *t4, void *t8,
                              hipStream_t stream)
{
    hipLaunchKernelGGL(tile_weight_kernel, dim3((unsigned)((N + TN - 1) / TN)), dim3(256), 0, stream,
                       (const uint8_t *)q4, (const int8_t *)q8, N, (K - O) >> 1, O, (uint8_t *)t4, (uint8_t *)t8);
    return hipGetLastError();
}

// What the kernels that read tiled weights need: the common case (see common_tail).
bool decode_tiled_supported(const GemmParams &p) { return common_tail(p) != 0; }

bool decode_many_rows(const GemmParams &p)
{
    const int64_t cus = atom_launch::compute_units();
    return decode_rounds(p.M, p.N, cus) <= 3 || resident_sets(p.M, p.N, p.K, cus);
}

hipError_t launch_decode_tiled(const GemmParams &call, hipStream_t stream)
{
    GemmParams p = call;
    p.swap_slices = swapped_slices(p.K);
    const unsigned blocks = (unsigned)((p.N + TN - 1) / TN);
    if (common_tail(p) == 3) launch_common<true, 3>(p, blocks, stream);
    else                     launch_common<true, 1>(p, blocks, stream);
    return hipGetLastError();
}

hipError_t launch_decode(const GemmParams &call, hipStream_t stream)
{
    GemmParams p = call;
    p.swap_slices = swapped_slices(p.K);
    const unsigned blocks = (unsigned)((p.N + TN - 1) / TN);
    const int tail = common_tail(p);
    if (tail == 3) { launch_common<false, 3>(p, blocks, stream); return hipGetLastError(); }
    if (tail == 1) { launch_common<false, 1>(p, blocks, stream); return hipGetLastError(); }
    // The general kernel.  Vector scale loads: G even (a scale row then starts on a 4-byte boundary),
    // both scale arrays 4-byte aligned
    const int  G  = p.K >> 7;
    const bool vs = G % 2 == 0 && G >= 4 && ((reinterpret_cast<uintptr_t>(p.a_scale) | reinterpret_cast<uintptr_t>(p.w_scale)) & 3) == 0 &&
                    (uint64_t)p.N * (uint64_t)G < (1ull << 31);          // 32-bit scale offsets
    // exactly one INT8 group, and it is the last group of the last wavefront's run (G >= 8)
    const bool one8 = p.O == 128 && G >= NW && (uint64_t)p.N * (uint64_t)(p.K >> 1) < (1ull << 32);   // 32-bit byte offsets
    if (p.M <= 16 && vs && one8) {
        hipLaunchKernelGGL((w4a4_gemm_decode_kernel<1, true, true>), dim3(blocks), dim3(NT), 0, stream, p);
    } else if (p.M <= 32 && vs && one8) {
        hipLaunchKernelGGL((w4a4_gemm_decode_kernel<2, true, true>), dim3(blocks), dim3(NT), 0, stream, p);
    } else if (vs && one8) {
        hipLaunchKernelGGL((w4a4_gemm_decode_kernel<4, true, true>), dim3(blocks), dim3(NT), 0, stream, p);
    } else if (p.M <= 16) {
        if (vs) hipLaunchKernelGGL((w4a4_gemm_decode_kernel<1, true>), dim3(blocks), dim3(NT), 0, stream, p);
        else    hipLaunchKernelGGL((w4a4_gemm_decode_kernel<1, false>), dim3(blocks), dim3(NT), 0, stream, p);
    } else if (p.M <= 32) {
        if (vs) hipLaunchKernelGGL((w4a4_gemm_decode_kernel<2, true>), dim3(blocks), dim3(NT), 0, stream, p);
        else    hipLaunchKernelGGL((w4a4_gemm_decode_kernel<2, false>), dim3(blocks), dim3(NT), 0, stream, p);
    } else {
        hipLaunchKernelGGL((w4a4_gemm_decode_kernel<4, false>), dim3(blocks), dim3(NT), 0, stream, p);
    }
    return hipGetLastError();
}

}  // namespace atom_gemm
