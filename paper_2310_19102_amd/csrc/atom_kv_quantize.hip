// INT4 KV cache for gfx950: asymmetric per-head quantisation (Section 2 of the paper,
// asymmetric equations; Section 4.4: granularity of one attention head).

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "atom_internal.h"

namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));

// Maxima of two pairs of fp16 values.  (As an instruction: the compiler puts one that quiets signalling NaNs in front of
// every loaded or moved operand of its own maxima.  The instruction itself ignores NaNs.)
__device__ __forceinline__ h2 pair_max(h2 a, h2 b)
{
    h2 r;
    asm("v_pk_max_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ h2 pair_min(h2 a, h2 b)
{
    h2 r;
    asm("v_pk_min_f16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// The maximum of both halves over the LPR (8 or 16) lanes that share a row; LPR lanes are consecutive and
// aligned, so rotations inside the 16-lane DPP row stay inside the row for LPR = 16, and an
// xor butterfly is used for LPR = 8
template <int LPR>
__device__ __forceinline__ h2 row_max(h2 v)
{
    if constexpr (LPR == 16) {            // DPP rotations of the 16-lane row: vector-ALU speed, no LDS crossbar
#define ATOM_ROW_ROR(n) \
        v = pair_max(v, __builtin_bit_cast(h2, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), 0x120 | (n), 0xF, 0xF, true)))
        ATOM_ROW_ROR(8);
        ATOM_ROW_ROR(4);
        ATOM_ROW_ROR(2);
        ATOM_ROW_ROR(1);
#undef ATOM_ROW_ROR
    } else {
#pragma unroll
        for (int d = 1; d < LPR; d <<= 1)
            v = pair_max(v, __builtin_bit_cast(h2, __shfl_xor(__builtin_bit_cast(int, v), d, 64)));
    }
    return v;
}

// One row of D = 8 * LPR values on LPR lanes (this lane's eight are `raw`):
//   s = fp16(((max - min) * clip) / 15), z = clamp(rne(-min / s)), code = clamp(rne(x/s) + z, 0, 15)
// with correctly rounded fp32 quotients by the stored scale; a zero scale gives zero codes and z = 0.
//   * max and min of the fp16 values two at a time, as fp16;
//   * the nine quotients share the reciprocal r = RN(1/s), exact for every fp16 s after one Newton step (every
//     scale is tested); q = y r, then q + (y - q s) r rounded once is the quotient: q is within two units of it,
//     the residual is exact, and y/s lies at least 2^-12 units from the middle of two floats (s has 11 bits); the
//     quotient by 15 likewise (a quotient so small that its residual would be inexact is a zero scale);
//   * clamp(rne(v) + z, 0, 15) = rne(clamp(v, -z, 15 - z)) + z; adding 1.5 * 2^23 rounds to the nearest even integer and
//     leaves it in the low bits, and a chain of shift-and-add of those bits packs the eight codes: what z and the
//     exponent bits add to the sum is one term of the row.
// About 10 vector instructions per value (20 with five per quotient and integer codes).
struct KvRow { uint32_t w, sz; };                            // codes; scale in the low half, zero point in the high half
template <int LPR>
__device__ __forceinline__ KvRow kv_quantize_row(const uint4 &raw, float clip)
{
    const h2 *hp = reinterpret_cast<const h2 *>(&raw);
    const h2 hx = pair_max(pair_max(hp[0], hp[1]), pair_max(hp[2], hp[3]));
    const h2 hn = pair_min(pair_min(hp[0], hp[1]), pair_min(hp[2], hp[3]));
    const h2 m = row_max<LPR>(pair_max(h2{hx[0], -hn[0]}, h2{hx[1], -hn[1]}));
    const float  mx = (float)m[0], mn = -(float)m[1];
    // Within 15 * 65504 (the largest scale is the largest fp16) and what gives minus infinity; a NaN stays one (these two hand it on).
    const float  span = __builtin_elementwise_maximum(__builtin_elementwise_minimum((mx - mn) * clip, 982560.0f), -1000000.0f);
    const float  q15 = span * (1.0f / 15.0f);
    float        s32 = fmaf(fmaf(15.0f, q15, -span), -1.0f / 15.0f, q15);      // (in these signs a zero quotient keeps its sign)
    asm("" : "+v"(s32));                                   // (a fused form would round to fp16 once, not to fp32 first)
    const _Float16 sh = (_Float16)s32;
    const float  s  = (float)sh;
    const float  r0 = __builtin_amdgcn_rcpf(s);
    const float  r  = s != 0.0f ? fmaf(fmaf(-s, r0, 1.0f), r0, r0) : 0.0f;
    auto quotient = [&](float y) {
        const float q = fmaf(y, r, 0.0f);                    // (a fused form takes fp16 operands as they are)
        return fmaf(fmaf(-s, q, y), r, q);
    };
    const float    zf = __builtin_amdgcn_fmed3f(rintf(quotient(-mn)), -32768.0f, 32767.0f), lo = -zf, hi = 15.0f - zf;
    const int32_t  z = (int32_t)zf;
    constexpr float kRound = 12582912.0f;                    // 1.5 * 2^23
    KvRow o;
    o.w = ((uint32_t)z - 0x4b400000u) * 0x11111111u;
    uint32_t sum = 0;
#pragma unroll
    for (int i = 7; i >= 0; --i) {
        const float v = __builtin_amdgcn_fmed3f(quotient((float)hp[i >> 1][i & 1]), lo, hi);
        sum = (sum << 4) + __builtin_bit_cast(uint32_t, v + kRound);
    }
    o.w += sum;
    o.sz = (uint32_t)__builtin_bit_cast(uint16_t, sh) | ((uint32_t)z << 16);
    return o;
}

// Rows into a whole cache (prefill): 64 / LPR rows per wavefront and load, kLoads of them in flight, all
// consecutive, so that a wavefront's scales (and zero points) leave in one store of a contiguous piece.  Bound by HBM
// (the loads and stores alone: 15.5 us for 8192 tokens of 32 heads of 128 values, 85 MB) with the vector ALU close behind:
// 19 us there (28 us with one load per wavefront and twice the instructions), 46 us instead of 66 for 655360 rows.
template <int LPR, int kLoads>
__global__ __launch_bounds__(256)
void kv_quantize_bulk_kernel(const __half *__restrict__ x, int64_t R, int64_t ldx, float clip, uint8_t *__restrict__ q,
                             uint16_t *__restrict__ scale, uint16_t *__restrict__ zero)
{
    constexpr int D = 8 * LPR, RPL = 64 / LPR;               // rows per load
    static_assert(kLoads <= LPR, "a lane of the row for each load's scale");
    const int     lane = threadIdx.x & 63, j = lane % LPR, g = lane / LPR;
    const int64_t first = ((int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * (RPL * kLoads);
    if (first >= R) return;
    const int left = (int)(R - first < RPL * kLoads ? R - first : RPL * kLoads);
    x += first * ldx;
    q += first * (D / 2);
    const int64_t mine = g * ldx;
    uint4 raws[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
        const bool in = left == RPL * kLoads || g + RPL * u < left;                  // a row past the end: the first one again
        raws[u] = *reinterpret_cast<const uint4 *>(x + (in ? mine + RPL * u * ldx : 0) + 8 * j);
    }
    uint32_t sz = 0;
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
        const KvRow o = kv_quantize_row<LPR>(raws[u], clip);
        if (left == RPL * kLoads || g + RPL * u < left)
            *reinterpret_cast<uint32_t *>(q + u * (RPL * D / 2) + (g * (D / 2) + 4 * j)) = o.w;
        sz = j == u ? o.sz : sz;                             // lane u of a row's lanes keeps what load u gave
    }
    if (j < kLoads && g + RPL * j < left) {
        scale[first + g + RPL * j] = (uint16_t)sz;
        zero[first + g + RPL * j] = (uint16_t)(sz >> 16);
    }
}

// Rows of a step: row r goes to row r (pos == nullptr), or to r * Tmax + pos[r / rows_per_seq] (append one token per
// sequence: row r = (sequence, head)); rows whose position is outside [0, Tmax) write nothing.  grid.y = 2: the same rows
// of a second tensor into a second cache (K and V of one append).
template <int LPR>
__global__ __launch_bounds__(256)
void kv_quantize_kernel(const __half *__restrict__ x0, int64_t R, int64_t ldx, float clip,
                        const int32_t *__restrict__ pos, int32_t rows_per_seq, int64_t Tmax,
                        uint8_t *__restrict__ q0, uint16_t *__restrict__ scale0,
                        uint16_t *__restrict__ zero0, const __half *__restrict__ x1,
                        uint8_t *__restrict__ q1, uint16_t *__restrict__ scale1,
                        uint16_t *__restrict__ zero1)
{
    constexpr int D = 8 * LPR;
    const bool second = blockIdx.y != 0;
    const int64_t r = ((int64_t)blockIdx.x * 256 + threadIdx.x) / LPR;
    const int     j = threadIdx.x % LPR;
    if (r >= R) return;                                      // (whole rows of lanes)
    const uint4 raw = *reinterpret_cast<const uint4 *>((second ? x1 : x0) + r * ldx + 8 * j);
    int64_t orow = r;
    bool    keep = true;
    if (pos) {                                               // a position outside the cache is dropped
        const int64_t p = pos[r / rows_per_seq];
        keep = p >= 0 && p < Tmax;
        orow = r * Tmax + p;
    }
    const KvRow o = kv_quantize_row<LPR>(raw, clip);
    if (keep) {
        *reinterpret_cast<uint32_t *>((second ? q1 : q0) + orow * (D / 2) + 4 * j) = o.w;
        if (j == 0) {
            (second ? scale1 : scale0)[orow] = (uint16_t)o.sz;
            (second ? zero1 : zero0)[orow] = (uint16_t)(o.sz >> 16);
        }
    }
}

}  // namespace

namespace atom_internal {

hipError_t launch_kv_quantize(const void *x, int64_t R, int64_t ldx, int D, float clip,
                              const int32_t *pos, int32_t rows_per_seq, int64_t Tmax, void *q,
                              void *scale, void *zero, hipStream_t stream, const void *x2, void *q2,
                              void *scale2, void *zero2)
{
    const int lpr = D / 8;
    if (R >= 16384 && !pos && !x2) {                      // 1024 wavefronts of four loads; fewer rows: one load per wavefront, more of them
        constexpr int kLoads = 4;
        const int64_t per = (int64_t)kLoads * (256 / lpr), grid = (R + per - 1) / per;      // rows per workgroup
        if (D == 128)
            hipLaunchKernelGGL((kv_quantize_bulk_kernel<16, kLoads>), dim3((unsigned)grid), dim3(256), 0, stream, (const __half *)x,
                               R, ldx, clip, (uint8_t *)q, (uint16_t *)scale, (uint16_t *)zero);
        else
            hipLaunchKernelGGL((kv_quantize_bulk_kernel<8, kLoads>), dim3((unsigned)grid), dim3(256), 0, stream, (const __half *)x,
                               R, ldx, clip, (uint8_t *)q, (uint16_t *)scale, (uint16_t *)zero);
        return hipGetLastError();
    }
    const int64_t grid = (R + 256 / lpr - 1) / (256 / lpr);
#define ATOM_KVQ_LAUNCH(LPR)                                                                          \
    hipLaunchKernelGGL((kv_quantize_kernel<LPR>), dim3((unsigned)grid, x2 ? 2 : 1), dim3(256),        \
                       0, stream, (const __half *)x, R, ldx, clip, pos, rows_per_seq, Tmax,           \
                       (uint8_t *)q, (uint16_t *)scale, (uint16_t *)zero, (const __half *)x2,            \
                       (uint8_t *)q2, (uint16_t *)scale2, (uint16_t *)zero2)
    if (D == 128) ATOM_KVQ_LAUNCH(16);
    else          ATOM_KVQ_LAUNCH(8);
#undef ATOM_KVQ_LAUNCH
    return hipGetLastError();
}

}  // namespace atom_internal
