// Shared definitions of the group-GEMM kernels.
#ifndef ATOM_GEMM_COMMON_H
#define ATOM_GEMM_COMMON_H

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include <type_traits>

namespace atom_gemm {

typedef int v4i  __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

struct GemmParams {
    const uint8_t *a_q4; const int8_t *a_q8; const uint16_t *a_scale;
    const uint8_t *w_q4; const int8_t *w_q8; const uint16_t *w_scale;
    uint16_t *y; int32_t *partials;
    int64_t M, N, ldy;
    int K, O;
    int swap_slices = 0;                  // decode kernels (slice_of_wave)
};

__device__ __forceinline__ float half_bits_to_float(uint16_t h)
{
    return __half2float(__ushort_as_half(h));
}

// Byte offset of 16-byte chunk `chunk` (0..7) of tile row `row` (128 bytes per row).
// Measured on gfx950: a 128-bit LDS read is served 16 lanes per pass out of 64 banks of
// 4 bytes, so two consecutive rows span the banks once, and a fragment read (16
// consecutive rows, one chunk index) is conflict-free only if those rows land on 16
// different 16-byte bank groups.  Xor-ing the chunk with the low three row bits alone
// repeats after eight rows (2-way conflicts, half the read rate); folding row bit 3 in
// separates rows r and r+8.  The loader's 128-bit writes (4 rows x 4 chunks per 16
// lanes) run at their full rate with it as well.  The pattern has period 16 rows.
__device__ __forceinline__ int lds_off(int row, int chunk)
{
    return row * 128 + (((chunk ^ row ^ ((row >> 3) & 1)) & 7) << 4);
}


// Logical tile index of this workgroup.  Hardware deals consecutive workgroup
// ids round-robin to the 8 XCDs; give every XCD a contiguous run of logical
// tiles so neighbouring tiles (which share operand rows) meet in one L2.
__device__ __forceinline__ int xcd_contiguous_block_id()
{
    const int nb = gridDim.x, b = blockIdx.x;
    const int per = nb >> 3, rem = nb & 7, xcd = b & 7;
    return xcd * per + (xcd < rem ? xcd : rem) + (b >> 3);
}

// Eight fp16 elements from element h (0 .. 7) of the sixteen in (lo, hi).
__device__ __forceinline__ v4i from_element(const v4i &lo, const v4i &hi, unsigned h)
{
    unsigned w[8] = {(unsigned)lo[0], (unsigned)lo[1], (unsigned)lo[2], (unsigned)lo[3],
                     (unsigned)hi[0], (unsigned)hi[1], (unsigned)hi[2], (unsigned)hi[3]};
#pragma unroll
    for (int j = 0; j < 6; ++j) { const unsigned stay = w[j], move = w[j + 2]; w[j] = h & 4 ? move : stay; }
#pragma unroll
    for (int j = 0; j < 5; ++j) { const unsigned stay = w[j], move = w[j + 1]; w[j] = h & 2 ? move : stay; }
    v4i d;
#pragma unroll
    for (int j = 0; j < 4; ++j) d[j] = (int)__builtin_amdgcn_alignbit(w[j + 1], w[j], 16 * (h & 1));
    return d;
}

// Elements of a row in front of its first 16-byte aligned one.
__device__ __forceinline__ unsigned to_aligned(const uint16_t *row)
{
    return (0u - ((unsigned)reinterpret_cast<uintptr_t>(row) >> 1)) & 7u;
}

// A finished block of Y (ROWS x COLS fp16; its rows `pitch` >= 2 COLS + 16 bytes apart in LDS, 16-byte aligned) to rows of Y
// that start on any element (an odd row length, a view): whole 16-byte pieces wherever 16-byte aligned addresses lie in
// the row, put together from two neighbouring pieces of the staged row, then what is left at its two ends, eight lanes per
// row.  `y` is the block's first element; rows and columns at and past rows_left and cols_left are not stored.  (Two
// bytes per lane, as the accumulators hold them, a block of 64 x 64 is 64 store instructions and more lines than bytes: the
// packed GEMM at M = 2048, K = 4096 took 132 us for N = 12289 and 88 us for N = 12288.)
template <int ROWS, int COLS>
__device__ __forceinline__ void store_block_any(const unsigned char *blk, int pitch, uint16_t *y, int64_t ldy, int rows_left,
                                                int cols_left, int lane)
{
    constexpr int LPR = COLS / 8;
    static_assert(ROWS * LPR % 64 == 0 && ROWS % 8 == 0, "whole wavefronts");
    const int nc = cols_left < COLS ? cols_left : COLS;
#pragma unroll 2
    for (int i = 0; i < ROWS * LPR / 64 && 64 * i < LPR * rows_left; ++i) {
        const int q = 64 * i + lane, r = q / LPR, k = q % LPR;
        uint16_t *row = y + (int64_t)r * ldy;
        const unsigned h = to_aligned(row);
        const v4i lo = *reinterpret_cast<const v4i *>(blk + r * pitch + 16 * k);
        const v4i hi = *reinterpret_cast<const v4i *>(blk + r * pitch + 16 * k + 16);
        const v4i d = from_element(lo, hi, h);
        if (r < rows_left && (int)h + 8 * k + 8 <= nc) *reinterpret_cast<v4i *>(row + h + 8 * k) = d;
    }
    // slot e of a row: its first h elements, then those behind the last whole piece (a block of all COLS columns has eight
    // or none of them, a cut one up to fourteen)
    if (((reinterpret_cast<uintptr_t>(y) | (uintptr_t)(ldy * 2)) & 15) == 0 && (nc & 7) == 0) return;
    for (int e0 = 0; e0 < (nc == COLS ? 8 : 16); e0 += 8)
#pragma unroll 2
        for (int i = 0; i < ROWS / 8 && 8 * i < rows_left; ++i) {
            const int r = 8 * i + (lane >> 3), e = e0 + (lane & 7);
            uint16_t *row = y + (int64_t)r * ldy;
            const int h = (int)to_aligned(row);
            const int n = e < h ? e : h + (nc > h ? (nc - h) & ~7 : 0) + (e - h);
            if (r < rows_left && n < nc) row[n] = *reinterpret_cast<const uint16_t *>(blk + r * pitch + 2 * n);
        }
}

// The same for the kernels of launches of few tiles.  What bounds it there is latency, one wavefront per SIMD: a chunk of rows reads
// everything from LDS before it stores anything, and eight rows or fewer are a chunk of their own.  (Packed GEMM, N = 100, Y off the grid,
// K = 512: M = 65 8.0 us with two bytes per lane, 9.0 step by step, 8.2 so; M = 777 8.4, 9.3, 8.3.  The kernels of many tiles keep the
// steps: the registers and the code of this form cost the walking one 1 to 2.5 % at every size, M = 4096, K = 8192, N = 57344 1626 us,
// 1663 so, and the canonical one 27.6 against 29.2 at M = 4096, K = 512, N = 4096 off the grid.)
template <int ROWS, int COLS>
__device__ __forceinline__ void store_block_few(const unsigned char *blk, int pitch, uint16_t *y, int64_t ldy, int rows_left,
                                                int cols_left, int lane)
{
    constexpr int LPR = COLS / 8, RPS = 64 / LPR;          // lanes per row, rows that a wavefront's 16-byte pieces cover
    static_assert(64 % LPR == 0 && RPS <= 16 && ROWS % 32 == 0, "whole wavefronts");
    const int nc = cols_left < COLS ? cols_left : COLS;
    const bool ends = ((reinterpret_cast<uintptr_t>(y) | (uintptr_t)(ldy * 2)) & 15) != 0 || (nc & 7) != 0;
    const int k = lane % LPR, e = lane & 7;
    auto chunk = [&](auto rows_c, int r0) __attribute__((always_inline)) {
        constexpr int C = decltype(rows_c)::value, P = C > RPS ? C / RPS : 1, E = C / 8;
        const int rp = r0 + lane / LPR, re = r0 + (lane >> 3);
        uint16_t *const yp = y + rp * ldy, *const ye = y + re * ldy;
        v4i d[P];
#pragma unroll
        for (int j = 0; j < P; ++j) {
            const unsigned char *src = blk + (rp + RPS * j) * pitch + 16 * k;
            d[j] = from_element(*reinterpret_cast<const v4i *>(src), *reinterpret_cast<const v4i *>(src + 16), to_aligned(yp + RPS * j * ldy));
        }
        // slot e of a row: its first h elements, then those behind the last whole piece (a block of all COLS columns has eight
        // or none of them, a cut one up to fourteen: slot e + 8)
        uint16_t one[E], two[E];
        int n[E], n2[E];
        if (ends) {
#pragma unroll
            for (int j = 0; j < E; ++j) {
                const uint16_t *src = reinterpret_cast<const uint16_t *>(blk + (re + 8 * j) * pitch);
                const int h = (int)to_aligned(ye + 8 * j * ldy), whole = nc > h ? (nc - h) & ~7 : 0;
                n[j]  = e < h ? e : whole + e;
                n2[j] = whole + e + 8;
                one[j] = src[n[j]];
                two[j] = nc < COLS ? src[n2[j]] : 0;
            }
        }
#pragma unroll
        for (int j = 0; j < P; ++j) {
            uint16_t *row = yp + RPS * j * ldy;
            const int h = (int)to_aligned(row);
            if (rp + RPS * j < rows_left && h + 8 * k + 8 <= nc) *reinterpret_cast<v4i *>(row + h + 8 * k) = d[j];
        }
        if (ends) {
#pragma unroll
            for (int j = 0; j < E; ++j) {
                uint16_t *row = ye + 8 * j * ldy;
                if (re + 8 * j < rows_left && n[j] < nc) row[n[j]] = one[j];
                if (re + 8 * j < rows_left && nc < COLS && n2[j] < nc) row[n2[j]] = two[j];
            }
        }
    };
    if (rows_left <= 8) return chunk(std::integral_constant<int, 8>(), 0);
    for (int r0 = 0; r0 < ROWS && r0 < rows_left; r0 += 32) chunk(std::integral_constant<int, 32>(), r0);
}

// The block of Y whose first element is (m, n), cut at M and N.  FEW: a kernel of launches of few tiles.
template <int ROWS, int COLS, bool FEW = false>
__device__ __forceinline__ void store_block(const unsigned char *blk, int pitch, uint16_t *y, int64_t ldy, int64_t m, int64_t n,
                                            int64_t M, int64_t N, int lane)
{
    constexpr int LPR = COLS / 8;
    static_assert(64 % LPR == 0, "a step of the loop is whole rows");
    if (m >= M || n >= N) return;
    const int rows = (int)(M - m < ROWS ? M - m : ROWS);
    uint16_t *first = y + m * ldy + n;
    if (((reinterpret_cast<uintptr_t>(y) | (uintptr_t)(ldy * 2)) & 15) == 0 && n + COLS <= N) {
        const int r = lane / LPR, k = lane % LPR;
        uint16_t *const mine = first + r * ldy + 8 * k;
#pragma unroll
        for (int i = 0; i < ROWS * LPR / 64; ++i)
            if (i * (64 / LPR) + r < rows)
                *reinterpret_cast<v4i *>(mine + i * (64 / LPR) * ldy) = *reinterpret_cast<const v4i *>(blk + (i * (64 / LPR) + r) * pitch + 16 * k);
    } else {
        if constexpr (FEW) store_block_few<ROWS, COLS>(blk, pitch, first, ldy, rows, (int)(N - n < COLS ? N - n : COLS), lane);
        else               store_block_any<ROWS, COLS>(blk, pitch, first, ldy, rows, (int)(N - n < COLS ? N - n : COLS), lane);
    }
}

// Big-tile kernel for compute-bound sizes, M > 64 (atom_gemm_big.hip).
hipError_t launch_big(const GemmParams &p, hipStream_t stream);

// Weight-streaming kernel for decode-sized M <= 64 (atom_gemm_decode.hip).
hipError_t launch_decode(const GemmParams &p, hipStream_t stream);
// The same on weight codes re-tiled by launch_tile_weight (w_q4, w_q8 of p are the tiled arrays).
hipError_t launch_tile_weight(const void *q4, const void *q8, int64_t N, int K, int O, void *t4, void *t8,
                              hipStream_t stream);
bool decode_tiled_supported(const GemmParams &p);
// whether a problem of the common case with 65 to 256 rows goes to the streaming kernels
bool decode_many_rows(const GemmParams &p);
// estimated time of the tiled kernels in us (atom_gemm.hip)
float tiles_us(int64_t M, int64_t N, int K, int64_t cus);
hipError_t launch_decode_tiled(const GemmParams &p, hipStream_t stream);

}  // namespace atom_gemm
#endif
