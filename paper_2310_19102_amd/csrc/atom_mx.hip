// GEMM of the MX variant for gfx950: both operands hold FP4 E2M1 codes (normal channels) and
// FP8 E4M3 codes (outlier channels, last) with one E8M0 scale byte per block of 32 channels.
// The paper (Section 5.2, FP4 paragraph) expects hardware group scaling to take the
// dequantisation out of the kernel; on gfx950 that is v_mfma_scale_f32_32x32x64_f8f6f4, which
// multiplies each lane's 32 elements by 2^(scale byte - 127) inside the matrix core.  The
// K loop below is therefore nothing but operand movement and MFMAs.
//
// Operand layout of the instruction (checked on the hardware against a CPU sum):
//   A 32 x 64: lane l holds row l % 32; FP4: its 16 bytes are elements 32g .. 32g+31 of the
//     K = 64 step, g = l / 32, even element in the low nibble; FP8: its 32 bytes are elements
//     16g .. 16g+15 and 32+16g .. 32+16g+15.  B likewise with columns for rows.
//   scale: byte `op_sel` of the scale register of lane (row, g) is the scale of elements
//     32g .. 32g+31 of the row: for FP4 the lane's own 16 bytes, for FP8 the low (g = 0) or
//     high (g = 1) 16 bytes of both lanes of the row.  Either way an MX block of 32
//     consecutive channels has one scale.
//   C 32 x 32: lane l holds column l % 32, rows 8 (v / 4) + 4 (l / 32) + v % 4, v = 0..15.

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include <type_traits>

#include "atom_gemm_f6.h"
#include "atom_internal.h"
#include "atom_launch.h"

namespace {

using namespace atom_gemm_f6;             // vector types, LDS-DMA requests, order control, wait_imm

constexpr int ROWB = 64;                  // bytes per tile row and K step: 128 FP4 or 64 FP8 channels

struct MxParams {
    const uint8_t *a_q4, *a_q8, *a_e8;
    const uint8_t *w_q4, *w_q8, *w_e8;
    uint16_t *y;
    int64_t M, N, ldy;
    int K, O;
};

// 16-byte chunk `chunk` (0..3) of tile row `row`: rows r, r+4, r+8, r+12 would share a bank
// group (4 rows of 64 bytes span the 64 banks once), so the chunk index is rotated by row / 4;
// a fragment read (16 consecutive rows, one chunk index) and the loader's writes (4 rows x 4
// chunks per 16 lanes) then touch 16 different bank groups.
__device__ __forceinline__ int mx_lds_off(int row, int chunk)
{
    return row * ROWB + (((chunk + (row >> 2)) & 3) << 4);
}

template <int FMT, int OPSEL>
__device__ __forceinline__ v16f mfma_mx(v8i a, v8i b, v16f c, int sa, int sb)
{
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, FMT, FMT, OPSEL, sa, OPSEL, sb);
}

__device__ __forceinline__ v8i widen(v4i lo)
{
    return __builtin_shufflevector(lo, lo, 0, 1, 2, 3, -1, -1, -1, -1);
}
__device__ __forceinline__ v8i join(v4i lo, v4i hi)
{
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

__device__ __forceinline__ void dma4(uint32_t lds, uint32_t voff, const uint8_t *sbase)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                 :: "s"(lds), "v"(voff), "s"(sbase) : "memory", "m0");
}

// WM x WN wavefronts (four or eight), each TM x TN MFMA tiles: a workgroup tile of 32 WM TM x 32 WN TN; ST stages in LDS.
template <int WM, int WN, int TM, int TN, int ST>
struct MxTile {
    static constexpr int NW    = WM * WN, NT = 64 * NW;
    static constexpr int BM    = 32 * WM * TM, BN = 32 * WN * TN;
    static constexpr int CODES = (BM + BN) * ROWB;         // bytes of codes per stage, the A rows first
    static constexpr int NSC   = (BM + BN + 63) / 64;      // requests of 64 scale dwords per stage
    static constexpr int STAGE = CODES + NSC * 256;        // + one scale dword per row
    static constexpr int NST   = ST;                       // LDS stages
    static constexpr int NBLK  = (BM + BN) / 16;           // requests of a kilobyte (16 rows) per stage
    static constexpr int J     = (NBLK + NW - 1) / NW;     // ... per wavefront
    static constexpr int JS    = (NSC + NW - 1) / NW;      // ... per wavefront
    static constexpr int LOADS = J + JS;
    static constexpr int SPARE = NST * STAGE;              // 16 bytes that are written and never read
    static constexpr int LDS   = SPARE + 64;
    static constexpr int PITCH = 64 * TN + 16;             // output staging: bytes per row of a wavefront's block
    static constexpr int EPIW  = 32 * TM * PITCH;
    static_assert(BM % 64 == 0 && BN % 32 == 0, "whole requests of codes, and of the activations' scales");
    static_assert(NW * EPIW <= NST * STAGE && LDS <= 160 * 1024, "LDS");
    static constexpr int PER_CU = 2 * LDS <= 160 * 1024 ? 2 : 1;
};

// One K step per iteration: 64 bytes of every tile row, i.e. 64 FP8 channels (one MFMA per tile
// pair; these outlier steps come first) or 128 FP4 channels (two MFMA sub-steps).  The operands go
// from global memory straight into LDS (global_load_lds_dwordx4), so no wavefront spends issue slots
// on staging registers and ds_write.  With four stages: while step u is multiplied, tile u+1 has
// landed or is landing, tile u+2 is on its way and tile u+3 is requested.  A request fills one
// kilobyte = 16 tile rows; lane l supplies the chunk that the rotated layout wants at its position:
// row l / 4 of the 16, chunk ((l % 4) - (l / 16)) % 4.  The requests are inline assembly, the compiler does
// not count them: the waits on vmcnt before the barriers are written by hand.
//
// What bounds it.  Many tiles: the power the matrix cores may take (M = 4096, N = K = 8192: the MFMAs alone, operands in
// registers, 107 us, this kernel 126, the LDS reads and barriers alone 19, the requests alone 61).  Few tiles: the chain barrier,
// fragment reads, MFMAs of one workgroup, so they run as small tiles, several workgroups of four wavefronts to a compute unit, whose barriers are
// not each other's.  Either way
//   * an in-order wavefront that issues its requests in one go waits until the memory path has taken them (16 cycles
//     each, all wavefronts of the CU in turn) and its MFMAs wait behind: every SIMD has two wavefronts or more, and
//     a wavefront's requests stand one at a time behind MFMAs (M = 1024, K = 4096, N = 22016 with 256 x 256 tiles: 70 us
//     with one wavefront per SIMD and all requests at the step's start, 58 so);
//   * the weights are the row operand of the MFMA, so that a lane holds four consecutive columns of a
//     row of Y and the output staging is a quarter of the LDS writes.
template <int WM, int WN, int TM, int TN, int ST>
__global__ __launch_bounds__(64 * WM * WN, (WM * WN * MxTile<WM, WN, TM, TN, ST>::PER_CU + 3) / 4)
void mx_gemm_dma_kernel(MxParams p)
{
    using Gm = MxTile<WM, WN, TM, TN, ST>;
    constexpr int BM = Gm::BM, BN = Gm::BN, NW = Gm::NW, J = Gm::J, JS = Gm::JS, LOADS = Gm::LOADS, STAGE = Gm::STAGE, NST = Gm::NST;
    extern __shared__ __align__(16) uint8_t smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int lr = lane & 31, g = lane >> 5;

    const int tiles_m = (int)((p.M + BM - 1) / BM);
    const int bid = atom_gemm::xcd_contiguous_block_id();
    const int64_t m0 = (int64_t)(bid % tiles_m) * BM, n0 = (int64_t)(bid / tiles_m) * BN;

    const int K4 = p.K - p.O;
    const int S4 = K4 >> 7, S8 = p.O >> 6, S = S4 + S8;

    // ---- loader: kilobyte block b = NW j + wave of a stage are its rows 16 b .. 16 b + 15; ragged tiles repeat the last
    // row.  Request b of the scales are the dwords of rows 64 b .. 64 b + 63.
    uint32_t goff[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int b = NW * j + wave, trow = 16 * b + (lane >> 2);
        const bool act = b < BM / 16;
        int64_t r = act ? m0 + trow : n0 + (trow - BM);
        const int64_t last = (act ? p.M : p.N) - 1;
        r = r < last ? r : last;
        goff[j] = (uint32_t)r * ROWB + 16u * (((lane & 3) - (lane >> 4)) & 3);
    }
    uint32_t soff[JS];
#pragma unroll
    for (int j = 0; j < JS; ++j) {
        const int b = NW * j + wave;
        const bool act = b < BM / 64;
        int64_t r = act ? m0 + 64 * b + lane : n0 + (64 * b - BM) + lane;
        const int64_t last = (act ? p.M : p.N) - 1;
        soff[j] = (uint32_t)(r < last ? r : last) * 4u;
    }
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(smem), spare = lds0 + Gm::SPARE;
    // where tile u's codes and scales start; steps 0 .. S8-1 are the FP8 (outlier) steps, the FP4 steps follow
    struct Src { const uint8_t *a, *w, *ae, *we; };
    auto src_of = [&](int u) __attribute__((always_inline)) -> Src {
        const bool    f8 = u < S8;
        const int64_t sl = f8 ? u : u - S8;                        // slab index inside q8 or q4
        const int64_t d  = f8 ? S4 + (u >> 1) : u - S8;            // slab index inside e8
        return {(f8 ? p.a_q8 : p.a_q4) + sl * p.M * ROWB, (f8 ? p.w_q8 : p.w_q4) + sl * p.N * ROWB,
                p.a_e8 + d * p.M * 4, p.w_e8 + d * p.N * 4};
    };
    // request k of a tile into stage `buf` (the same number per wavefront: the waits count them)
    auto request = [&](int k, const Src &s, int buf) __attribute__((always_inline)) {
        const uint32_t st = lds0 + buf * STAGE;
        if (k < J) {
            const int b = NW * k + wave;
            const uint8_t *base = NW * (k + 1) <= BM / 16 ? s.a : NW * k >= BM / 16 ? s.w : b < BM / 16 ? s.a : s.w;
            if (NW * (k + 1) <= Gm::NBLK) dma16(st + 1024 * b, goff[k], base);
            else dma16_masked(b < Gm::NBLK ? st + 1024 * b : spare, goff[k], base, b < Gm::NBLK ? ~0ull : 1ull);
        } else {
            const int b = NW * (k - J) + wave;
            const uint8_t *base = NW * (k - J + 1) <= BM / 64 ? s.ae : NW * (k - J) >= BM / 64 ? s.we : b < BM / 64 ? s.ae : s.we;
            if (NW * (k - J + 1) <= Gm::NSC || b < Gm::NSC) dma4(st + Gm::CODES + 256 * b, soff[k < J ? 0 : k - J], base);
            else dma16_masked(spare, 0u, s.a, 1ull);
        }
    };
    auto request_all = [&](int u, int buf) __attribute__((always_inline)) {
        const Src s = src_of(u);
#pragma unroll
        for (int k = 0; k < LOADS; ++k) request(k, s, buf);
    };
    // all but the two newest tiles' loads of this wavefront have landed, and its own LDS reads are done
    auto landed = [&]() __attribute__((always_inline)) { __builtin_amdgcn_s_waitcnt(wait_imm((NST - 2) * LOADS)); };

    v16f acc[TM][TN];
#pragma unroll
    for (int s = 0; s < TM; ++s)
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[s][t][v] = 0.0f;

    const int a_base = mx_lds_off(32 * TM * wm + lr, g);
    const int b_base = mx_lds_off(BM + 32 * TN * wn + lr, g);
    const int sa_off = Gm::CODES + 4 * (32 * TM * wm + lr), sb_off = Gm::CODES + 4 * (BM + 32 * TN * wn + lr);
    int sa[TM], sb[TN];
    auto read_scales = [&](const uint8_t *buf) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < TM; ++s) sa[s] = (int)(*reinterpret_cast<const uint32_t *>(buf + sa_off + 128 * s) >> (8 * g));
#pragma unroll
        for (int t = 0; t < TN; ++t) sb[t] = (int)(*reinterpret_cast<const uint32_t *>(buf + sb_off + 128 * t) >> (8 * g));
    };
    using fp4 = std::integral_constant<int, 4>;
    using fp8 = std::integral_constant<int, 0>;
    using b0  = std::integral_constant<int, 0>;
    using b2  = std::integral_constant<int, 2>;
    // the MFMAs of a sub-step; `after(i)` runs behind the i-th
    auto mma = [&](auto fmt, auto opsel, const v8i (&af)[TM], const v8i (&bf)[TN], const int (&sa_)[TM],
                   const int (&sb_)[TN], auto after) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < TM; ++s)
#pragma unroll
            for (int t = 0; t < TN; ++t) {
                acc[s][t] = mfma_mx<decltype(fmt)::value, decltype(opsel)::value>(bf[t], af[s], acc[s][t], sb_[t], sa_[s]);
                ATOM_F6_PIN(acc[s][t]);
                after(s * TN + t);
            }
    };
    auto nothing = [](int) {};

    int cur = 0;                                           // stage of tile u
#pragma unroll
    for (int v = 0; v < NST - 1; ++v) request_all(min(v, S - 1), v);
    landed();
    __syncthreads();

    // ---- FP8 steps first, in pairs
    int u = 0;
    auto fp8_step = [&](auto opsel) __attribute__((always_inline)) {
        request_all(min(u + NST - 1, S - 1), cur == 0 ? NST - 1 : cur - 1);
        const uint8_t *buf = smem + cur * STAGE;
        v8i af8[TM], bf8[TN];
#pragma unroll
        for (int s = 0; s < TM; ++s)
            af8[s] = join(*reinterpret_cast<const v4i *>(buf + (a_base + 2048 * s)),
                          *reinterpret_cast<const v4i *>(buf + ((a_base ^ 32) + 2048 * s)));
#pragma unroll
        for (int t = 0; t < TN; ++t)
            bf8[t] = join(*reinterpret_cast<const v4i *>(buf + (b_base + 2048 * t)),
                          *reinterpret_cast<const v4i *>(buf + ((b_base ^ 32) + 2048 * t)));
        read_scales(buf);
        mma(fp8{}, opsel, af8, bf8, sa, sb, nothing);
        landed();
        __syncthreads();
        cur = cur + 1 == NST ? 0 : cur + 1;
        ++u;
    };
    while (u < S8) {
        fp8_step(b0{});
        fp8_step(b2{});
    }

    // ---- FP4 steps, software-pipelined: the second sub-step's fragments are read under the first
    // sub-step's MFMAs, the next step's first fragments and scales under the second's
    v8i af[TM], bf[TN];
    auto read_half = [&](v8i (&x)[TM], v8i (&y)[TN], const uint8_t *buf, int half) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < TM; ++s) x[s] = widen(*reinterpret_cast<const v4i *>(buf + ((a_base ^ half) + 2048 * s)));
#pragma unroll
        for (int t = 0; t < TN; ++t) y[t] = widen(*reinterpret_cast<const v4i *>(buf + ((b_base ^ half) + 2048 * t)));
    };
    read_half(af, bf, smem + cur * STAGE, 0);
    read_scales(smem + cur * STAGE);
    Src ahead = src_of(min(u + NST - 1, S - 1));
    for (; u < S; ++u) {
        const uint8_t *buf = smem + cur * STAGE;
        const int into = cur == 0 ? NST - 1 : cur - 1;
        cur = cur + 1 == NST ? 0 : cur + 1;
        const uint8_t *nbuf = smem + cur * STAGE;
        v8i ag[TM], bg[TN];
        read_half(ag, bg, buf, 32);
        mma(fp4{}, b0{}, af, bf, sa, sb, [&](int i) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < LOADS; ++k)
                if (k * (TM * TN) / LOADS == i) request(k, ahead, into);
        });
        if (u + NST < S) { ahead.a += p.M * ROWB; ahead.w += p.N * ROWB; ahead.ae += p.M * 4; ahead.we += p.N * 4; }
        landed();                         // tile u+1 is in its stage ...
        __syncthreads();                  // ... for every wavefront; stage u has been read
        __builtin_amdgcn_sched_barrier(0);
        int sc[TM], sd[TN];
#pragma unroll
        for (int s = 0; s < TM; ++s) sc[s] = sa[s];
#pragma unroll
        for (int t = 0; t < TN; ++t) sd[t] = sb[t];
        read_half(af, bf, nbuf, 0);
        read_scales(nbuf);
        mma(fp4{}, b2{}, ag, bg, sc, sd, nothing);
        __builtin_amdgcn_sched_barrier(0);
    }

    // ---- store: a lane holds four consecutive columns of one row of Y at a time; through LDS, so that global memory sees
    // 16-byte row pieces.  The last (repeated) requests must have landed before the stages are reused.
    __builtin_amdgcn_s_waitcnt(wait_imm(0));
    __syncthreads();
    const int64_t wrow = m0 + 32 * TM * wm, wcol = n0 + 32 * TN * wn;
    uint8_t *reg = smem + wave * Gm::EPIW;
#pragma unroll
    for (int s = 0; s < TM; ++s)
#pragma unroll
        for (int t = 0; t < TN; ++t)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v2h lo = __builtin_convertvector((v2f{acc[s][t][4 * q], acc[s][t][4 * q + 1]}), v2h);
                const v2h hi = __builtin_convertvector((v2f{acc[s][t][4 * q + 2], acc[s][t][4 * q + 3]}), v2h);
                *reinterpret_cast<v2u *>(reg + (32 * s + lr) * Gm::PITCH + (32 * t + 8 * q + 4 * g) * 2) =
                    v2u{__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi)};
            }
    // (LDS only, and the wavefront reads what it wrote itself)
    atom_gemm::store_block<32 * TM, 32 * TN>(reg, Gm::PITCH, p.y, p.ldy, wrow, wcol, p.M, p.N, lane);
}

template <int WM, int WN, int TM, int TN, int ST>
hipError_t launch_tile(const MxParams &p, hipStream_t stream)
{
    using Gm = MxTile<WM, WN, TM, TN, ST>;
    auto kern = &mx_gemm_dma_kernel<WM, WN, TM, TN, ST>;
    static atom_launch::LdsOptIn opt_in;   // one attribute call per kernel variant and device
    hipError_t err = atom_launch::ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(kern), Gm::LDS);
    if (err != hipSuccess) return err;
    const int64_t tiles = ((p.M + Gm::BM - 1) / Gm::BM) * ((p.N + Gm::BN - 1) / Gm::BN);
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(Gm::NT), Gm::LDS, stream, p);
    return hipGetLastError();
}

// The same on wide tiles, 256 x 32 TN: eight wavefronts of 64 rows x 16 TN columns, three stages.
//
// The tiles above load 41 to 45 GB/s per compute unit, which has about 256 lines of 128 bytes in flight at most (alone 54 GB/s out of the memory, 96 to 110 out of the
// last-level cache, 115 to 148 out of the L2, with all of them at it 25, 29 and 115: profiles/loads_per_compute_unit.txt); loads return in order across its wavefronts, so a
// request out of the L2 waits behind one from farther away.  So this kernel loads fewer bytes per multiply-add: 28 GB/s at M = 1024, K = 4096, N = 22016, which
// no longer bounds it.  A step of 256 x 384 takes 1.27 us, its MFMAs alone 0.74 at their full rate (clocks fall to about 1.6 GHz with all compute units at it), and a round 8.5 us for
// prologue and store, which nothing overlaps (fitted to 185 sizes).  Only the accumulators stay (16 TN registers); the fragments of the
// weights are read from LDS four MFMAs ahead, in one run over both halves of a step, and the barrier of a step stands before its last MFMAs, behind
// which the first fragments of the next step are read.  (With 32 rows x 32 TN columns per wavefront LDS gives 1.6 times as much and the kernel is 3 to 9 %
// slower; TN = 9 and 11 were within 3 % of 10 and 12.)
// In turn on one card, us, the best of the tiles above and this kernel, weights from memory: M = 1024, K = 4096, N = 22016 64.5, 52.1 (TN = 12);
// M = 1300, N = 13824 52.4, 47.4; M = 2048, N = 10000 58.0, 48.0 (TN = 10); M = 1700, K = 14336, N = 11264 158.7, 134.1; M = 4096, N = 12288 110.6, 104.8.
// (16 x 16 x 128 MFMAs instead take a tenth less power and turn as fast, operands in registers; here, 0.97 to 1.03 of the time: half as long, they leave half
// the room for what stands between them.)
template <int TN>
struct MxWide {
    static constexpr int TM    = 2, CN = TN / 2, WM = 4;   // blocks of rows and of columns of a wavefront, wavefronts side by side in M
    static constexpr int NW    = 8, NT = 512, NST = 3;
    static constexpr int BM    = 256, BN = 32 * TN;
    static constexpr int CODES = (BM + BN) * ROWB;
    static constexpr int NSC   = (BM + BN) / 64;          // requests of 64 scale dwords per stage
    static constexpr int STAGE = CODES + 256 * NSC;
    static constexpr int NBLK  = (BM + BN) / 16;           // requests of a kilobyte (16 rows) per stage
    static constexpr int J     = (NBLK + NW - 1) / NW, JS = (NSC + NW - 1) / NW, LOADS = J + JS;
    static constexpr int SPARE = NST * STAGE;              // 16 bytes that are written and never read
    static constexpr int LDS   = SPARE + 64;
    static constexpr int PITCH = 144;                      // output staging: 32 rows of 64 columns per wavefront
    static constexpr int AHEAD = 2;                        // fragments read ahead of their MFMAs
    static_assert(NW * 32 * PITCH <= NST * STAGE && LDS <= 160 * 1024 && 2 * LOADS <= 63, "LDS, vmcnt");
    static_assert(TN % 2 == 0, "two wavefronts side by side in N, whole requests of scales");
};

template <int TN>
__global__ __launch_bounds__(512, 2)
void mx_gemm_wide_kernel(MxParams p)
{
    using Gm = MxWide<TN>;
    constexpr int TM = Gm::TM, CN = Gm::CN, WM = Gm::WM;
    constexpr int BM = Gm::BM, BN = Gm::BN, NW = Gm::NW, J = Gm::J, JS = Gm::JS, LOADS = Gm::LOADS, STAGE = Gm::STAGE, NST = Gm::NST, AHEAD = Gm::AHEAD;
    extern __shared__ __align__(16) uint8_t smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lr = lane & 31, g = lane >> 5;

    const int tiles_m = (int)((p.M + BM - 1) / BM);
    const int bid = atom_gemm::xcd_contiguous_block_id();
    const int64_t m0 = (int64_t)(bid % tiles_m) * BM, n0 = (int64_t)(bid / tiles_m) * BN;

    const int K4 = p.K - p.O;
    const int S4 = K4 >> 7, S8 = p.O >> 6, S = S4 + S8;

    // ---- loader, as above
    uint32_t goff[J], soff[JS];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int b = NW * j + wave, trow = 16 * b + (lane >> 2);
        const bool act = b < BM / 16;
        int64_t r = act ? m0 + trow : n0 + (trow - BM);
        const int64_t last = (act ? p.M : p.N) - 1;
        r = r < last ? r : last;
        goff[j] = (uint32_t)r * ROWB + 16u * (((lane & 3) - (lane >> 4)) & 3);
    }
#pragma unroll
    for (int j = 0; j < JS; ++j) {
        const int b = NW * j + wave;
        const bool act = b < BM / 64;
        int64_t r = act ? m0 + 64 * b + lane : n0 + (64 * b - BM) + lane;
        const int64_t last = (act ? p.M : p.N) - 1;
        soff[j] = (uint32_t)(r < last ? r : last) * 4u;
    }
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(smem), spare = lds0 + Gm::SPARE;
    struct Src { const uint8_t *a, *w, *ae, *we; };
    auto src_of = [&](int u) __attribute__((always_inline)) -> Src {
        const bool    f8 = u < S8;
        const int64_t sl = f8 ? u : u - S8;
        const int64_t d  = f8 ? S4 + (u >> 1) : u - S8;
        return {(f8 ? p.a_q8 : p.a_q4) + sl * p.M * ROWB, (f8 ? p.w_q8 : p.w_q4) + sl * p.N * ROWB,
                p.a_e8 + d * p.M * 4, p.w_e8 + d * p.N * 4};
    };
    auto request = [&](int k, const Src &s, int buf) __attribute__((always_inline)) {
        const uint32_t st = lds0 + buf * STAGE;
        if (k < J) {
            const int b = NW * k + wave;
            const uint8_t *base = NW * (k + 1) <= BM / 16 ? s.a : s.w;                 // (BM / 16 is whole rounds of the wavefronts)
            if (NW * (k + 1) <= Gm::NBLK) dma16(st + 1024 * b, goff[k], base);
            else dma16_masked(b < Gm::NBLK ? st + 1024 * b : spare, goff[k], base, b < Gm::NBLK ? ~0ull : 1ull);
        } else {
            const int b = NW * (k - J) + wave;
            const uint8_t *base = NW * (k - J) >= BM / 64 ? s.we : b < BM / 64 ? s.ae : s.we;
            if (NW * (k - J + 1) <= Gm::NSC || b < Gm::NSC) dma4(st + Gm::CODES + 256 * b, soff[k < J ? 0 : k - J], base);
            else dma16_masked(spare, 0u, s.a, 1ull);
        }
    };
    static_assert(BM / 16 % NW == 0, "a request's operand is known at compile time");
    auto request_all = [&](int u, int buf) __attribute__((always_inline)) {
        const Src s = src_of(u);
#pragma unroll
        for (int k = 0; k < LOADS; ++k) request(k, s, buf);
    };

    v16f acc[TM][CN];
#pragma unroll
    for (int r = 0; r < TM; ++r)
#pragma unroll
        for (int t = 0; t < CN; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[r][t][v] = 0.0f;

    const int wm = wave % WM, wn = wave / WM;
    const int a_base = mx_lds_off(32 * TM * wm + lr, g), b_base = mx_lds_off(BM + 32 * CN * wn + lr, g);
    // A scale is read as a byte alone, the block's of its half: shifted out of its dword it would be waited for behind every fragment's
    // read, not where its MFMA stands (M = 1024, K = 4096, N = 22016
    // 52.2 us, so 50.8; M = 3000 147.8, 141.9; M = 1700, K = 14336, N = 11264 134.2, 132.3)
    const int sa_off = Gm::CODES + 4 * (32 * TM * wm + lr) + g, sb_off = Gm::CODES + 4 * (BM + 32 * CN * wn + lr) + g;
    struct Frag { v4i b; int s; };
    auto read_frag = [&](const uint8_t *buf, int i) __attribute__((always_inline)) -> Frag {       // i = CN * half + block of columns
        const int half = i / CN, t = i % CN;
        return {*reinterpret_cast<const v4i *>(buf + ((half ? b_base ^ 32 : b_base) + 2048 * t)),
                (int)buf[sb_off + 128 * t + 2 * half]};
    };
    struct Rows { v4i a[TM]; int s[TM]; };
    auto read_rows = [&](const uint8_t *buf, int half) __attribute__((always_inline)) -> Rows {
        Rows x;
#pragma unroll
        for (int r = 0; r < TM; ++r) {
            x.a[r] = *reinterpret_cast<const v4i *>(buf + ((half ? a_base ^ 32 : a_base) + 2048 * r));
            x.s[r] = (int)buf[sa_off + 128 * r + 2 * half];
        }
        return x;
    };
    // Step u: tile u is in stage u % 3.  At its start stage (u - 1) % 3 has been read by everyone and is refilled with tile u + 2; before its
    // end tile u + 1 has landed.
    int cur = 0;
#pragma unroll
    for (int v = 0; v < NST; ++v) request_all(min(v, S - 1), v);
    __builtin_amdgcn_s_waitcnt(wait_imm(2 * LOADS));
    __syncthreads();
    int u = 0;
    auto next_stage = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_waitcnt(wait_imm(LOADS));
        __syncthreads();
        __builtin_amdgcn_sched_barrier(0);
        cur = cur + 1 == NST ? 0 : cur + 1;
        ++u;
    };
    auto refill = [&](int k, const Src &s) __attribute__((always_inline)) { request(k, s, cur == 0 ? NST - 1 : cur - 1); };
    bool started = false;                                  // (the first step has nothing to refill)

    // ---- FP8 steps, in pairs that share their scales
    auto fp8_step = [&](auto second) __attribute__((always_inline)) {            // (of a pair: its scales are the second half of the dword)
        constexpr int HALF = decltype(second)::value;
        if (started) {
            const Src s = src_of(min(u + 2, S - 1));
#pragma unroll
            for (int k = 0; k < LOADS; ++k) refill(k, s);
        }
        started = true;
        const uint8_t *buf = smem + cur * STAGE;
        const Rows lo = read_rows(buf, 0), hi = read_rows(buf, 1);
#pragma unroll
        for (int t = 0; t < CN; ++t) {
            const Frag x = read_frag(buf, t), y = read_frag(buf, CN + t);
            const v8i b = join(x.b, y.b);
#pragma unroll
            for (int r = 0; r < TM; ++r) {
                acc[r][t] = mfma_mx<0, 0>(b, join(lo.a[r], hi.a[r]), acc[r][t], HALF ? y.s : x.s, HALF ? hi.s[r] : lo.s[r]);
                ATOM_F6_PIN(acc[r][t]);
            }
            if (t % 2 == 1) ATOM_F6_SLOT_END();            // (not all fragments of the step in registers at once)
        }
        next_stage();
    };
    while (u < S8) {
        fp8_step(std::integral_constant<int, 0>{});
        fp8_step(std::integral_constant<int, 1>{});
    }

    // ---- FP4 steps
    constexpr int NF = 2 * CN, RING = AHEAD + 1, LASTREAD = NF - AHEAD - 1;      // MFMAs behind which the step's last fragment is read
    constexpr int SLOTS = TM * (LASTREAD + 1);                                   // the requests stand behind these MFMAs
    Frag f[RING];
    Rows a0, a1;
    {
        const uint8_t *buf = smem + cur * STAGE;
        a0 = read_rows(buf, 0);
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) f[i] = read_frag(buf, i);
    }
    Src ahead = src_of(min(u + 2, S - 1));
    // (the ring of fragments turns by NF per step: its start is a template argument, and RING steps bring it back)
    auto fp4_step = [&](auto start) __attribute__((always_inline)) {
        constexpr int ST = decltype(start)::value;
        const uint8_t *buf = smem + cur * STAGE;
        a1 = read_rows(buf, 1);
#pragma unroll
        for (int i = 0; i < NF; ++i) {
            const Frag &x = f[(ST + i) % RING];
#pragma unroll
            for (int r = 0; r < TM; ++r) {
                if (i < CN) acc[r][i % CN] = mfma_mx<4, 0>(widen(x.b), widen(a0.a[r]), acc[r][i % CN], x.s, a0.s[r]);
                else        acc[r][i % CN] = mfma_mx<4, 0>(widen(x.b), widen(a1.a[r]), acc[r][i % CN], x.s, a1.s[r]);
                ATOM_F6_PIN(acc[r][i % CN]);
                if (r == 0 && i + AHEAD < NF) f[(ST + i + AHEAD) % RING] = read_frag(buf, i + AHEAD);
#pragma unroll
                for (int k = 0; k < LOADS; ++k)
                    if (k * SLOTS / LOADS == TM * i + r) refill(k, ahead);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (i == LASTREAD + 1) {
                next_stage();
                a0 = read_rows(smem + cur * STAGE, 0);
            }
            if (i > LASTREAD) f[(ST + NF + i - LASTREAD - 1) % RING] = read_frag(smem + cur * STAGE, i - LASTREAD - 1);    // of the next step
            __builtin_amdgcn_sched_barrier(0);
        }
        if (u + 2 < S) { ahead.a += p.M * ROWB; ahead.w += p.N * ROWB; ahead.ae += p.M * 4; ahead.we += p.N * 4; }
    };
    auto steps = [&](auto self, auto k) __attribute__((always_inline)) -> bool {       // RING steps, or to the end
        constexpr int KK = decltype(k)::value;
        if constexpr (KK < RING) {
            if (u >= S) return false;
            fp4_step(std::integral_constant<int, KK * NF % RING>{});
            return self(self, std::integral_constant<int, KK + 1>{});
        }
        return true;
    };
    while (steps(steps, std::integral_constant<int, 0>{})) {}

    // ---- store, 64 columns at a time through LDS.  The last (repeated) requests must have landed before the stages are reused.
    __builtin_amdgcn_s_waitcnt(wait_imm(0));
    __syncthreads();
    uint8_t *reg = smem + wave * (32 * Gm::PITCH);
#pragma unroll
    for (int r = 0; r < TM; ++r)
#pragma unroll
        for (int t0 = 0; t0 < CN; t0 += 2) {
#pragma unroll
            for (int t = t0; t < t0 + 2 && t < CN; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v2h lo = __builtin_convertvector((v2f{acc[r][t][4 * q], acc[r][t][4 * q + 1]}), v2h);
                    const v2h hi = __builtin_convertvector((v2f{acc[r][t][4 * q + 2], acc[r][t][4 * q + 3]}), v2h);
                    *reinterpret_cast<v2u *>(reg + lr * Gm::PITCH + (32 * (t - t0) + 8 * q + 4 * g) * 2) =
                        v2u{__builtin_bit_cast(unsigned, lo), __builtin_bit_cast(unsigned, hi)};
                }
            // (LDS only, and the wavefront reads what it wrote itself)
            const int64_t row = m0 + 32 * (TM * wm + r), col = n0 + 32 * (CN * wn + t0);
            if (t0 + 2 <= CN) atom_gemm::store_block<32, 64>(reg, Gm::PITCH, p.y, p.ldy, row, col, p.M, p.N, lane);
            else              atom_gemm::store_block<32, 32>(reg, Gm::PITCH, p.y, p.ldy, row, col, p.M, p.N, lane);
        }
}

template <int TN>
hipError_t launch_wide(const MxParams &p, hipStream_t stream)
{
    using Gm = MxWide<TN>;
    auto kern = &mx_gemm_wide_kernel<TN>;
    static atom_launch::LdsOptIn opt_in;
    hipError_t err = atom_launch::ensure_dynamic_lds(opt_in, reinterpret_cast<const void *>(kern), Gm::LDS);
    if (err != hipSuccess) return err;
    const int64_t tiles = ((p.M + Gm::BM - 1) / Gm::BM) * ((p.N + Gm::BN - 1) / Gm::BN);
    hipLaunchKernelGGL(kern, dim3((unsigned)tiles), dim3(Gm::NT), Gm::LDS, stream, p);
    return hipGetLastError();
}

// Which tile.  The cost of a launch, in microseconds per K step, with f tiles per compute unit: `full` for each whole tile
// every compute unit has, and for a last part r of them what they add when few compute units have one (`alone` where it is
// all there is, `more` beside other workgroups), growing to `full` as the chip fills and the power limit sets in.  Measured
// at 43 sizes, K = 1024 to 14336 (profiles/mx_gemm_tiles.txt has all of them; us, weights from memory; the choice among these five is within 5 % of the
// best tile but at M = 256, N = 22016 and M = 2048, N = 12288, K = 4096, where 128 x 256 would be 8 and 10 % faster):
//   M = 65,   N = 4096,  K = 4096:   64 x 64 9.2, 64 x 128 10.7, 128 x 128 11.3, 128 x 256 16.9, 256 x 256 23.7
//   M = 256,  N = 12288, K = 4096:   64 x 64 18.2, 64 x 128 18.0, 128 x 128 14.2, 128 x 256 20.7, 256 x 256 25.5
//   M = 512,  N = 4096,  K = 4096:   64 x 64 12.4, 64 x 128 11.5, 128 x 128 12.2, 128 x 256 17.7, 256 x 256 24.1
//   M = 777,  N = 13824, K = 5120:   64 x 64 64.3, 64 x 128 54.7, 128 x 128 38.5, 128 x 256 43.3, 256 x 256 40.2
//   M = 1024, N = 22016, K = 4096:   64 x 64 103.4, 64 x 128 85.5, 128 x 128 62.4, 128 x 256 55.9, 256 x 256 61.1
//   M = 4096, N = 22016, K = 4096:   64 x 64 436.6, 64 x 128 331.6, 128 x 128 251.2, 128 x 256 207.0, 256 x 256 203.1
// The wide tiles come out of it too well, since nothing stands for their prologue and store, one workgroup to a compute unit: they also have to be ahead
// in microseconds (kOther, kWide: with K / 128 + 1 steps, fitted to 361 sizes of K = 2048 to 14336 where the cost takes them, within 3 to 5 %:
// profiles/mx_gemm_wide_tiles.txt).  Without that 32 of the 361 were slower than the tile they replaced, by up to 6 % (K = 2048, M = 3000, N = 12288 128 x 256 50.7,
// 256 x 320 53.1; K = 5120, M = 1300, N = 28672 128 x 256 112.3, 256 x 384 116.4), with it 10, by up to 5 %.  256 x 256, 256 x 320, 256 x 384 on another card:
//   M = 1024, N = 22016, K = 4096:   64.6, 72.7, 52.1          M = 2048, N = 10000, K = 4096:    63.0, 48.0, 50.3
//   M = 1200, N = 12288, K = 11008:  81.9, 95.4, 92.5          M = 1300, N = 16000, K = 5120:    73.2, 85.3, 61.9
//   M = 4096, N = 22016, K = 4096:   206.0, -, 199.4           M = 1500, N = 8192,  K = 8192:    60.8, -, 68.4
// (The kernel before, 256 x 256 and 128 x 128 with four wavefronts: 15.0, 16.4, 15.7, 49.1, 73.5 and 242.3.)
enum Tile { k64x64, k64x128, k128x128, k128x256, k256x256, k256x320, k256x384, kTiles };
struct TileCost { int bm, bn; float alone, more, full; };
constexpr TileCost kCost[kTiles] = {{64, 64, 0.150f, 0.080f, 0.125f}, {64, 128, 0.190f, 0.110f, 0.205f}, {128, 128, 0.235f, 0.110f, 0.300f},
                                    {128, 256, 0.380f, 0.280f, 0.590f}, {256, 256, 0.600f, 0.600f, 1.050f},
                                    {256, 320, 0.900f, 0.900f, 1.200f}, {256, 384, 0.950f, 0.950f, 1.380f}};

int64_t tiles_of(const TileCost &t, int64_t M, int64_t N) { return ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn); }

struct OtherTime { float launch, round, cost, mb; };        // us: once, per round of tiles, per K step and unit of cost, per MB of operands
constexpr OtherTime kOther[k256x256 + 1] = {{5.0f, 0.0f, 1.0f, 0.0f}, {5.0f, 0.0f, 1.0f, 0.0f}, {1.8f, 0.91f, 0.945f, 0.082f}, {7.4f, 0.18f, 0.89f, 0.090f},
                                            {4.3f, 4.4f, 0.89f, 0.028f}};
struct WideTime { float round, step, last; };               // us: per round of tiles, per K step of a round, what the last round's fill adds to a step
constexpr WideTime kWide[2] = {{7.1f, 1.117f, 0.124f}, {8.45f, 1.27f, 0.083f}};

Tile pick_tile(int64_t M, int64_t N, int K, int cus)
{
    Tile other = k256x256, best = k256x256;
    float least = 0.0f, least_other = 0.0f;
    for (int i = 0; i < kTiles; ++i) {
        const int64_t tiles = tiles_of(kCost[i], M, N);
        if (tiles > 0x7fffff) continue;                    // (the grid's limit in threads; the 256 x 256 tile takes what is left)
        if (i > k256x256 && K < 2048) continue;            // (the wide kernel: steps enough for its prologue and store)
        const TileCost &t = kCost[i];
        const float r = (float)(tiles % cus) / (float)cus, few = tiles < cus ? t.alone : t.more;
        const float cost = t.full * (float)(tiles / cus) + (r > 0.0f ? few + (t.full - few) * r * r * r : 0.0f);
        if (i <= k256x256 && (least_other == 0.0f || cost <= least_other)) { least_other = cost; other = (Tile)i; }
        if (least == 0.0f || cost <= least) { least = cost; best = (Tile)i; }
    }
    if (best <= k256x256) return best;
    const float     steps = (float)(K / 128 + 1);
    const int64_t   tiles = tiles_of(kCost[best], M, N), tiles_other = tiles_of(kCost[other], M, N);
    const WideTime  &w = kWide[best - k256x320];
    const OtherTime &o = kOther[other];
    const float r    = (float)(tiles % cus) / (float)cus;
    const float wide = (float)((tiles + cus - 1) / cus) * (w.round + w.step * steps) + w.last * r * r * r * steps;
    const float us   = o.launch + o.round * (float)((tiles_other + cus - 1) / cus) + o.cost * least_other * steps +
                       o.mb * (float)(M + N) * (float)K * 0.56e-6f;
    return wide < 1.02f * us ? best : other;
}

// Tiles of 64 x 32, with six stages or eight, where there are compute units for twice the tiles of 64 x 64: what a compute unit has in flight bounds its loads, and
// a step of them fetches a quarter less.  64 x 64 and so, M = 128, N = 4096, weights from HBM, us: K = 8192 17.5 / 12.6, 2048 6.9 / 5.8, 1024 5.1 / 4.5 (with eight stages
// 4.7).  (64 x 64 with more stages than four: from HBM M = 256, K = 11008 22.4 / 20.2, but from the last-level cache K = 5120 3.5 % slower; 64 x 96 on
// six wavefronts for 64 x 128: 1.2 times as slow.)
// (The stages; 0: 64 x 64 as it is.)
int narrow_stages(int64_t M, int64_t N, int K, int cus)
{
    return 2 * tiles_of(kCost[k64x64], M, N) > cus ? 0 : K > 4096 ? 8 : 6;
}

}  // namespace

// Which tile a launch takes, as the test of the tiles asks it (rows and columns of the tile in one number).
extern "C" int atom_internal_mx_tile(int64_t M, int64_t N, int64_t cus)
{
    const TileCost &t = kCost[pick_tile(M, N, 0, (int)cus)];
    return 1000 * t.bm + t.bn;
}

// The same for a call of K channels (above: of few).
extern "C" int atom_internal_mx_tile_k(int64_t M, int64_t N, int32_t K, int64_t cus)
{
    const TileCost &t = kCost[pick_tile(M, N, K, (int)cus)];
    return 1000 * t.bm + t.bn;
}

// Stages of the 64 x 32 tiles that a call with tiles of 64 x 64 takes in their place; 0: it does not.
extern "C" int atom_internal_mx_narrow_stages(int64_t M, int64_t N, int32_t K, int64_t cus)
{
    return pick_tile(M, N, K, (int)cus) == k64x64 ? narrow_stages(M, N, K, (int)cus) : 0;
}

namespace atom_internal {

hipError_t launch_mx_gemm(const void *a_q4, const void *a_q8, const void *a_e8, int64_t M,
                          const void *w_q4, const void *w_q8, const void *w_e8, int64_t N, int K,
                          int O, void *y, int64_t ldy, hipStream_t stream)
{
    MxParams p;
    p.a_q4 = (const uint8_t *)a_q4; p.a_q8 = (const uint8_t *)a_q8; p.a_e8 = (const uint8_t *)a_e8;
    p.w_q4 = (const uint8_t *)w_q4; p.w_q8 = (const uint8_t *)w_q8; p.w_e8 = (const uint8_t *)w_e8;
    p.y = (uint16_t *)y; p.M = M; p.N = N; p.ldy = ldy; p.K = K; p.O = O;
    const int cus = atom_launch::compute_units();
    switch (pick_tile(M, N, K, cus)) {
    case k64x64:
        switch (narrow_stages(M, N, K, cus)) {
        case 6:  return launch_tile<2, 1, 1, 1, 6>(p, stream);
        case 8:  return launch_tile<2, 1, 1, 1, 8>(p, stream);
        default: return launch_tile<2, 2, 1, 1, 4>(p, stream);
        }
    case k64x128:  return launch_tile<2, 2, 1, 2, 6>(p, stream);
    case k128x128:                                         // up to one per compute unit with four stages, else three workgroups per compute unit
        return tiles_of(kCost[k128x128], M, N) <= cus ? launch_tile<2, 2, 2, 2, 4>(p, stream) : launch_tile<2, 2, 2, 2, 3>(p, stream);
    case k128x256: return launch_tile<2, 4, 2, 2, 3>(p, stream);
    case k256x320: return launch_wide<10>(p, stream);
    case k256x384: return launch_wide<12>(p, stream);
    default:       return launch_tile<4, 2, 2, 4, 4>(p, stream);
    }
}

}  // namespace atom_internal
