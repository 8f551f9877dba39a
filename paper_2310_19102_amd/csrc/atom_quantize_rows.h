// Row routine of the activation front end, shared by the stand-alone front-end kernels and
// by the decode kernel that runs the front end in its prologue: RMSNorm, reorder (Section 4.1
// of the paper), dynamic group quantisation (Section 4.2, Section 2 symmetric equations).
//
// Compile WITHOUT fast-math: the fp32 division, sqrt and the absence of fused multiply-adds
// are part of the bit-exact contract with the CPU oracle.
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

namespace atom_quantize_rows {

__device__ __forceinline__ void halves_to_floats(const uint4 &raw, float *f)
{
    const __half2 *h = reinterpret_cast<const __half2 *>(&raw);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float2 t = __half22float2(h[i]);
        f[2 * i]     = t.x;
        f[2 * i + 1] = t.y;
    }
}

// h = fp16(a + b) per element: the sum of two fp16 values formed in fp32 and rounded once
// (where the fp32 sum is inexact the addends are more than 2^13 apart, nowhere near an
// fp16 rounding tie, so this is the correctly rounded fp16 sum)
__device__ __forceinline__ uint4 add_halves(const uint4 &a, const uint4 &b)
{
    float fa[8], fb[8];
    halves_to_floats(a, fa);
    halves_to_floats(b, fb);
    uint4 out;
    uint32_t *o = reinterpret_cast<uint32_t *>(&out);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t lo = __half_as_ushort(__float2half_rn(fa[2 * i] + fb[2 * i]));
        const uint32_t hi = __half_as_ushort(__float2half_rn(fa[2 * i + 1] + fb[2 * i + 1]));
        o[i] = lo | (hi << 16);
    }
    return out;
}

// exp(x) on [-87, 87] from IEEE operations only (one value on every machine, the CPU
// oracle's included): n = round(x*log2(e)); r = x - n*ln2 with ln2 split in two, the first
// part short enough for n*ln2_hi to be exact; e^r by its Taylor polynomial of degree 7 in
// Horner form; 2^n through the exponent field.  The rounding is one fused multiply-add onto 1.5 * 2^23, which leaves n in
// the low bits as well: a shift and an add put it into the exponent of e^r (between 0.7 and 1.5, and |n| <= 126).  Both are
// exact, and for every fp16 x the fused product rounds to the same n as a rounded one.
__device__ __forceinline__ float exp_ieee(float x)
{
    x = __builtin_amdgcn_fmed3f(x, -87.0f, 87.0f);
    const float biased = fmaf(x, 1.44269502162933349609375f, 12582912.0f);
    const float n = biased - 12582912.0f;
    float r = fmaf(n, -0.693145751953125f, x);
    r = fmaf(n, -1.428606765330187045037746429443359375e-06f, r);
    float p = 1.0f / 5040.0f;
    p = fmaf(p, r, 1.0f / 720.0f);
    p = fmaf(p, r, 1.0f / 120.0f);
    p = fmaf(p, r, 1.0f / 24.0f);
    p = fmaf(p, r, 1.0f / 6.0f);
    p = fmaf(p, r, 0.5f);
    p = fmaf(p, r, 1.0f);
    p = fmaf(p, r, 1.0f);
    return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, p) + (__builtin_bit_cast(uint32_t, biased) << 23));
}

// silu(g) * u in fp32: sigma = the correctly rounded 1/(1 + exp(-g)), then (g*sigma)*u.  g is an fp16 number, so
// there are 65536 cases: the hardware's reciprocal with one Newton step (three instructions, a general division
// takes eleven) is the correctly rounded value in every one of them (all of them are tested).
__device__ __forceinline__ float silu_mul(float g, float u)
{
    const float d  = 1.0f + exp_ieee(-g);
    const float r0 = __builtin_amdgcn_rcpf(d);
    const float sigma = fmaf(fmaf(-d, r0, 1.0f), r0, r0);
    return (g * sigma) * u;
}

// Sum over the 64 lanes, the value in every lane: the butterfly L + shfl_xor(L, d) with d = 1, 2, 4, .. 32, addition for
// addition.  After the strides 1 and 2 all lanes of a quad agree, so mirroring a half row reaches the same value
// as stride 4, mirroring a row the same as stride 8; the last two are the lane-half swaps of gfx950.  (Through
// LDS, as ds_bpermute, the six steps were a quarter of the time of a single row.)
__device__ __forceinline__ float wave_butterfly_sum(float L)
{
#define ATOM_DPP_ADD(ctrl)                                                                       \
    L = L + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(                               \
                0, __builtin_bit_cast(int, L), ctrl, 0xF, 0xF, false))
    ATOM_DPP_ADD(0xB1);      // quad_perm [1,0,3,2]
    ATOM_DPP_ADD(0x4E);      // quad_perm [2,3,0,1]
    ATOM_DPP_ADD(0x141);     // row_half_mirror
    ATOM_DPP_ADD(0x140);     // row_mirror
#undef ATOM_DPP_ADD
    typedef unsigned v2ui __attribute__((ext_vector_type(2)));
    unsigned u = __builtin_bit_cast(unsigned, L), w = u;
    asm volatile("" : "+v"(w));          // (two registers: the swap exchanges halves between them)
    v2ui x = __builtin_amdgcn_permlane16_swap(u, w, false, false);
    unsigned second = x[1];
    asm volatile("" : "+v"(second));
    L = __builtin_bit_cast(float, x[0]) + __builtin_bit_cast(float, second);
    u = w = __builtin_bit_cast(unsigned, L);
    asm volatile("" : "+v"(w));
    x = __builtin_amdgcn_permlane32_swap(u, w, false, false);
    second = x[1];
    asm volatile("" : "+v"(second));
    return __builtin_bit_cast(float, x[0]) + __builtin_bit_cast(float, second);
}

// what happens to a row before it is normalised and quantised
constexpr int kPlain = 0;    // nothing
constexpr int kAdd = 1;      // x + res, rounded to fp16 and written to sum_out
constexpr int kSwiglu = 2;   // silu(x) * res in fp32 (x = gate row, res = up row), not stored

// max over the 16 lanes of a DPP row (xor butterfly; max is exact in any order)
__device__ __forceinline__ float row16_max(float v)
{
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) v = fmaxf(v, __shfl_xor(v, d, 64));
    return v;
}

// max over the 16 lanes of a DPP row by rotations (max is exact in any order), no LDS crossbar traffic.  Of values that are
// not negative and not NaN, whose bits are in the order of the numbers: one v_max_u32 with a DPP operand per step (as floats a move,
// a canonicalising maximum and the maximum itself).
__device__ __forceinline__ float row16_max_dpp(float f)
{
    uint32_t v = __builtin_bit_cast(uint32_t, f);
#define ATOM_ROW_ROR(n)                                                                          \
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x120 | (n), 0xF, 0xF, false))
    ATOM_ROW_ROR(8);
    ATOM_ROW_ROR(4);
    ATOM_ROW_ROR(2);
    ATOM_ROW_ROR(1);
#undef ATOM_ROW_ROR
    return __builtin_bit_cast(float, v);
}

// Scale of a group from its maximum (Section 2 symmetric equations, fp32, stored as fp16).  The division by 15 (7, 255) is a
// product with the rounded reciprocal and one correction, a = amax * 2 clip cut to the finite numbers: the same fp16 for
// every fp32 a >= 0 and each of the three (all of them were compared).
__device__ __forceinline__ __half group_scale(float amax, bool is4, int nbits, float clip)
{
    const float denom = is4 ? (nbits == 3 ? 7.0f : 15.0f) : 255.0f;
    const float recip = is4 ? (nbits == 3 ? 1.0f / 7.0f : 1.0f / 15.0f) : 1.0f / 255.0f;
    const float a     = fminf((2.0f * amax) * clip, 3.40282346638528859812e38f);
    const float q     = a * recip;
    float s32         = fmaf(fmaf(-q, denom, a), recip, q);
    asm volatile("" : "+v"(s32));      // (rounded to fp32 and then to fp16: left to itself the compiler makes one rounding of the two)
    return (s32 > 65504.0f) ? __ushort_as_half((unsigned short)0x7bffu) : __float2half_rn(s32);
}

// The scale of a group from its maximum and the
// codes of this lane's eight values: the IEEE quotient by the stored scale, round-half-to-even, clamp.
// The quotient takes three instructions per element.  s is an fp16 number, and r = rcp(s) with one Newton step is
// the correctly rounded 1/s for every one of them (every scale is tested, at its ties and beside them).  q = y r is within two
// units of y/s, e = y - q s is exact, and q + e r, rounded once, is the quotient unless y/s lies within 2^-23 units of the
// middle between two floats; with an 11-bit s it is at least 2^-12 units away from every such middle.  Returns the stored scale,
// s = its fp32 value.  The codes stay floats (whole numbers): what packs them needs no integers
// (pack_nibbles8 below, the conversion to FP6).
__device__ __forceinline__ __half quantise_lane8(const float (&y)[8], float amax, bool is4, int nbits, float clip,
                                                 float (&q)[8], float &s)
{
    // normal channels: n = nbits (4, or 3 with the codes still in nibbles), outliers n = 8
    const float qmin  = is4 ? (nbits == 3 ? -4.0f : -8.0f) : -128.0f;
    const float qmax  = is4 ? (nbits == 3 ? 3.0f : 7.0f) : 127.0f;
    const __half sh   = group_scale(amax, is4, nbits, clip);
    s = __half2float(sh);
    const float r0    = __builtin_amdgcn_rcpf(s);
    const float e0    = fmaf(-s, r0, 1.0f);
    const float r1    = fmaf(e0, r0, r0);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float qf = y[e] * r1;
        qf = fmaf(fmaf(-s, qf, y[e]), r1, qf);
        qf = rintf(qf);
        q[e] = __builtin_amdgcn_fmed3f(qf, qmin, qmax);      // (finite: the same as min(max(qf, qmin), qmax))
    }
    return sh;
}

// Eight codes in [-8, 7], given as floats, to eight two's-complement nibbles, code 0 lowest.
// c0 + 16 c1 + 256 c2 + 4096 c3 is a whole number below 2^16 in magnitude, exact in fp32; with 8
// added to every code (0x8888 to the sum) the digits are the offset-binary nibbles and no digit
// borrows from the next; flipping the top bit of each nibble turns offset binary into two's
// complement.  Eleven instructions instead of a conversion, a mask, a shift and an or per code.
__device__ __forceinline__ uint32_t pack_nibbles8(const float (&c)[8])
{
    const float lo = fmaf(c[3], 4096.0f, fmaf(c[2], 256.0f, fmaf(c[1], 16.0f, c[0])));
    const float hi = fmaf(c[7], 4096.0f, fmaf(c[6], 256.0f, fmaf(c[5], 16.0f, c[4])));
    const uint32_t a = (uint32_t)((int)lo + 0x8888);                       // in [0, 0xffff]
    const uint32_t b = ((uint32_t)(int)hi << 16) + 0x88880000u;
    return (a | b) ^ 0x88888888u;
}

// Same result as the plain front-end kernel (compiler-generated IEEE division), bit for bit, for
// K <= 8 * NT * NS and clip >= 2^-20
// (NT threads per row),
// with the per-element work cut down:
//   * a workgroup walks several rows; the gather offsets of the reorder (they are the same
//     for every row) and gamma stay in registers, and the next row's global loads are in
//     flight while this row is quantised;
//   * the IEEE division by the group's scale shares the reciprocal across the group (quantise_lane8).  Nothing
//     overflows: a scale that is not zero is at least 2^-24, and |y| < 2^33 for finite inputs (a normalised value is at most
//     sqrt(K), gamma below 2^16; silu(g) u below 2^32).  How far beyond the codes y / s lies is not bounded by the clip factor
//     alone: a subnormal scale can be two thirds of its quotient, one that saturates at 65504 any small part of it.  The
//     clamp takes those; quotients below 2^-100 round to code 0 either way.  A zero scale yields zero codes;
//   * the group maximum is a DPP rotation reduction.
// The rows row_first, row_first + row_step, ... < rows are handled by the calling workgroup
// (NT threads, all of them call); lds holds K + (NORM ? K / 8 : 0) floats.  q4, q8 and scale
// are the canonical arrays (row strides (K - O) / 2, O and K / 128) and may live in LDS.
// IDENT: the row already is in reordered channel order (the producer emitted it so, Section 4.1
// of the paper: the reorder fused into the prior operator): thread t's vector t + NT*i is its own
// share of group (t + NT*i) / 16, nothing is staged or gathered, idx is not read and lds holds
// the K / 8 sums of squares only (NORM) or nothing.
struct NoHook { __device__ __forceinline__ void operator()() const {} };

// after_first_fetch is called once, right after the global loads of the first row are issued (a
// caller with loads of its own that may take longer to return issues them there).
// ONE: the row row_first only, without a loop.  In a loop the wait for a row's values is the same
// instruction for every row, and behind the fetch of a next row it is a wait for all loads: a
// caller's own, too, which are meant to fly while the row is quantised.
// PACKED: the codes and scales do not go to the canonical arrays but straight into the unit images
// the packed GEMM reads (units of 64 rows; per unit one image per group: INT4 codes as FP6 E3M2 in
// three 16-byte chunks per row and half at 2048 c + 1024 h + 16 r, scales as 8-byte entries at
// 6144 + 8 r; INT8: chunk c of row r at 128 r + 16 ((c ^ r ^ (r/8 % 2)) % 8), scales at 8192 + 8 r).
// A row's packed bytes are first collected in LDS (pk_lds: 3 K4 / 4 + O bytes, in the order group,
// half, chunk), then copied out as whole 16-byte chunks.
typedef _Float16 pk_v32h __attribute__((ext_vector_type(32)));
typedef unsigned pk_v6u  __attribute__((ext_vector_type(6)));
// Wavefronts per SIMD that a kernel's registers have to leave room for, where the compiler would take a few more than that without being
// told: two workgroups of 512 threads per CU instead of one, five of 256 or four of 320 instead of four and three.  Two kernels with the loop over rows
// spill for it and are the faster ones: RMSNorm of three sweeps (2 registers; 1100 rows of 11008 16.8 us, without the bound 21.8; 4096 43.1, 55.4) and its
// tiled form of two sweeps of 256 (1 register; 2500 rows of 4096 12.0, 13.0; 4096 19.8, 19.6; 8192 35.5, 33.1).  Not the residual add with RMSNorm in order,
// tiled, three sweeps (6 registers: 1100 rows of 9216 24.2, 25.0, but 3000 of 10240 52.3, 48.5, and 4096 of 9216 75.5, 61.0).
constexpr int min_waves(bool norm, int ns, int nt, int pre, bool ident, bool packed, bool mx)
{
    if (nt == 512 && ns == 4) return norm ? 1 : 4;
    if (nt == 512 && ns == 3) return norm && (ident ? packed && pre == kAdd : pre == kAdd || packed || mx) ? 1 : 4;
    return nt <= 320 && ns == 2 && pre != kAdd ? 5 : 1;
}
// Where a workgroup has one row, a kernel without the loop over rows (ONE) has 20 to 40 registers less, room for another workgroup on the CU,
// and begins the norm while the index is on its way: 1024 rows of 5120, RMSNorm: 8.3 -> 7.2 us, with the residual add, tiled, 15.2 ->
// 10.1; of 8192: 11.0 -> 10.1; of 14336 in order 19.4 -> 13.0.  Elsewhere it is the same or up to 9 % slower.
constexpr bool one_row_pays(bool norm, int ns, int nt, bool ident)
{
    return norm && nt < 1024 && (ident ? ns >= 3 : ns == 2);
}

// A lane's place behind a pointer that is the same for the workgroup, as 32 bits beside it in the memory instruction.  (The offset is
// made opaque where it is used: as 64-bit addresses in front of the loop over rows they took up to 20 registers.)
template <class T>
__device__ __forceinline__ char *at(T *base, unsigned offset)
{
    asm volatile("" : "+v"(offset));
    return const_cast<char *>(reinterpret_cast<const char *>(base)) + offset;
}

constexpr int kImg4 = 6656, kImg8 = 8704, kSc4 = 6144, kSc8 = 8192;

// MX: codes and scale bytes of the MX variant (FP4 E2M1 / FP8 E4M3, one E8M0 byte per 32 channels = 4 lanes) in their
// step-major arrays instead: q4 [K4/128][rows][64], q8 [O/64][rows][64], scale as bytes [K/128][rows][4].  The hardware
// converts two values at a time, divided by the block's power of two, to the nearest, ties to even (13 vector
// instructions per lane and group, where comparing with every boundary took 120: 4096 x 8192 with RMSNorm 48 -> 26.5 us).
template <bool NORM, int NS, int NT, int PRE, bool IDENT = false, bool PACKED = false, class Hook = NoHook, bool MX = false,
          bool ONE = false>
__device__ __forceinline__
void quantize_rows_fast_body(float *lds, int64_t row_first, int64_t row_step,
                             const __half *x, int64_t rows, int64_t ld,
                             const __half *res, int64_t ldr, __half *sum_out, int64_t ldo,
                             const __half *__restrict__ gamma, float eps,
                             const int32_t *__restrict__ idx, int K, int O, int nbits, float clip,
                             uint8_t *q4, int8_t *q8, __half *scale, Hook after_first_fetch = Hook(),
                             uint8_t *pk_out = nullptr, uint8_t *pk_lds = nullptr)
{
    float *ybuf = lds;                        // [K]   staged row, original channel order (not IDENT)
    float *qbuf = lds + (IDENT ? 0 : K);      // [K/8] per-vector sums of squares (NORM only)

    const int tid  = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // the same in every lane: group decisions become scalar
    const int V    = K >> 3;
    const int K4   = K - O;
    const int G    = K >> 7;
    const int G4   = K4 >> 7;

    uint4 raw[NS];
    uint4 rres[PRE != kPlain ? NS : 1];
    // Threads past the end of the row load its last vector again (and use nothing of it): with a branch around each load the
    // compiler waits for every one of them inside its branch, one memory latency after the other.
    auto load_vector = [&](const __half *p, int i) -> uint4 {
        return *reinterpret_cast<const uint4 *>(at(p, 16u * (unsigned)min(tid + NT * i, V - 1)));
    };
    auto fetch_row = [&](int64_t row) {
        const __half *xr = x + row * ld, *rr = PRE != kPlain ? res + row * ldr : nullptr;
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            raw[i] = load_vector(xr, i);
            if (PRE != kPlain) rres[i] = load_vector(rr, i);
        }
    };
    int64_t row = row_first;
    if (row < rows) fetch_row(row);       // (first: the longest way of all the loads before the loop)
    // gather offsets (bytes into ybuf) of this lane's 8 channels in each of its groups
    // (with 1024 threads or four sweeps two of them share a register: as 16-bit offsets up to 16384 channels, as channel numbers beyond.
    // Not in the MX form, which has registers for them: 2048 rows of 13824 16.6 us, packed 17.8; 4096 of 12416 30.0 and 32.7, with RMSNorm 52.9 and 55.4)
    constexpr bool OPACK = NT >= 1024 || (NS >= 4 && !MX);
    constexpr int OSHIFT = !OPACK || NS * NT <= 2048 ? 2 : 0;
    uint32_t off[IDENT ? 1 : NS][OPACK ? 4 : 8];
#pragma unroll
    for (int j = 0; j < (IDENT ? 0 : NS); ++j) {
        const int g  = 4 * wave + (lane >> 4) + (NT / 16) * j;
        const int gg = g < G ? g : G - 1;
        const int j0 = gg * 128 + (lane & 15) * 8;
        const int4 i0 = *reinterpret_cast<const int4 *>(idx + j0);
        const int4 i1 = *reinterpret_cast<const int4 *>(idx + j0 + 4);
        const int id[8] = {i0.x, i0.y, i0.z, i0.w, i1.x, i1.y, i1.z, i1.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t c = min((unsigned)id[e], (unsigned)(K - 1));
            if (!OPACK)          off[j][e] = c << OSHIFT;
            else if (e % 2 == 0) off[j][e / 2] = c << OSHIFT;
            else                 off[j][e / 2] |= c << (16 + OSHIFT);
        }
    }
    // gamma stays in registers too, except with 1024 threads (128 registers per lane):
    // there each row re-reads it through the cache
    constexpr bool GREG = NT < 1024;
    uint4 graw[NORM && GREG ? NS : 1];
    if (NORM && GREG) {
#pragma unroll
        for (int i = 0; i < NS; ++i) graw[i] = load_vector(gamma, i);
    }

    after_first_fetch();

    for (; row < rows; row += row_step) {
        float yv[IDENT ? NS : 1][8];          // IDENT: the row, normalised, stays in registers
        // ---- 0. residual add; the sum is the new residual stream and the row quantised below
        if (PRE == kAdd) {
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const int v = tid + NT * i;
                if (v < V) {
                    raw[i] = add_halves(raw[i], rres[i]);
                    *reinterpret_cast<uint4 *>(at(sum_out + row * ldo, 16u * (unsigned)v)) = raw[i];
                }
            }
        }
        // ---- 1./2. stage the row (after RMSNorm, if any) in LDS, original channel order
        float r = 1.0f;
        if (NORM) {
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                const int v = tid + NT * i;
                if (v < V) {
                    float f[8];
                    halves_to_floats(raw[i], f);
                    float s0 = f[0] * f[0], s1 = f[1] * f[1], s2 = f[2] * f[2], s3 = f[3] * f[3];
                    float s4 = f[4] * f[4], s5 = f[5] * f[5], s6 = f[6] * f[6], s7 = f[7] * f[7];
                    qbuf[v] = ((s0 + s1) + (s2 + s3)) + ((s4 + s5) + (s6 + s7));
                }
            }
            __syncthreads();
            // (reads past the last vector add +0; eight at a time are in flight)
            float L = 0.0f;
            constexpr int NV = NS * NT / 64, CH = NV < 8 ? NV : 8;
#pragma unroll NV <= 16 ? NV / CH : 1
            for (int i0 = 0; i0 < NV; i0 += CH) {
                float part[CH];
#pragma unroll
                for (int i = 0; i < CH; ++i) part[i] = lane + 64 * (i0 + i) < V ? qbuf[lane + 64 * (i0 + i)] : 0.0f;
#pragma unroll
                for (int i = 0; i < CH; ++i) L = L + part[i];
            }
            L = wave_butterfly_sum(L);
            const float mean = L / (float)K;
            r = 1.0f / sqrtf(mean + eps);
        }
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int v = tid + NT * i;
            if (v < V) {
                float f[8];
                halves_to_floats(raw[i], f);
                if (PRE == kSwiglu) {
                    float u[8];
                    halves_to_floats(rres[i], u);
#pragma unroll
                    for (int e = 0; e < 8; ++e) f[e] = silu_mul(f[e], u[e]);
                }
                if (NORM) {
                    float g[8];
                    halves_to_floats(GREG ? graw[i] : *reinterpret_cast<const uint4 *>(gamma + 8 * v), g);
#pragma unroll
                    for (int e = 0; e < 8; ++e) f[e] = (f[e] * r) * g[e];
                }
                if constexpr (IDENT) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) yv[i][e] = f[e];
                } else {
                    *reinterpret_cast<float4 *>(ybuf + 8 * v)     = make_float4(f[0], f[1], f[2], f[3]);
                    *reinterpret_cast<float4 *>(ybuf + 8 * v + 4) = make_float4(f[4], f[5], f[6], f[7]);
                }
            } else if constexpr (IDENT) {
#pragma unroll
                for (int e = 0; e < 8; ++e) yv[i][e] = 0.0f;
            }
        }
        // the next row's loads fly while this one is quantised
        if (!ONE && row + row_step < rows) fetch_row(row + row_step);
        if (!IDENT) __syncthreads();

        // ---- 3./4. reorder, group amax, scale, quantise, pack ----------------
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const int  g    = 4 * wave + (lane >> 4) + (NT / 16) * j;
            const bool live = g < G;          // ragged last sweep: whole 16-lane rows idle
            const int  gg   = live ? g : G - 1;
            const int  j0   = gg * 128 + (lane & 15) * 8;
            float y[8];
            float amax = 0.0f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if constexpr (IDENT) {
                    y[e] = yv[j][e];
                } else {
                    uint32_t o = off[j][OPACK ? e / 2 : e];
                    if (OPACK) {
                        // unpacked here, per row: hoisted out of the row loop the unpacked
                        // offsets would take the registers the packing saves
                        asm volatile("" : "+v"(o));
                        o = (e % 2 ? o >> 16 : o & 0xffffu) << (2 - OSHIFT);
                    }
                    y[e] = *reinterpret_cast<const float *>(reinterpret_cast<const unsigned char *>(ybuf) + o);
                }
                if constexpr (MX) amax = __builtin_elementwise_maximum(amax, fabsf(y[e]));    // (a NaN if any value is one)
                else              amax = fmaxf(amax, fabsf(y[e]));
            }
            const bool  is4   = gg < G4;
            if constexpr (MX) {
                // The block's scale is that of its numbers.  A NaN among them (an infinite channel times the zero factor of its
                // own norm) becomes a zero in FP4 and the largest value in FP8, with its sign.
                if (__builtin_expect(amax != amax, 0)) {
                    amax = 0.0f;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        amax = fmaxf(amax, fabsf(y[e]));
                        y[e] = y[e] == y[e] ? y[e] : copysignf(is4 ? 0.0f : __builtin_inff(), y[e]);
                    }
                }
#define ATOM_QUAD_MAX(ctrl)                                                                      \
    amax = fmaxf(amax, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(                    \
                     0, __builtin_bit_cast(int, amax), ctrl, 0xF, 0xF, false)))
                ATOM_QUAD_MAX(0xB1);
                ATOM_QUAD_MAX(0x4E);
#undef ATOM_QUAD_MAX
                const float a = amax * clip;
                int byte = 0;
                if (a > 0.0f) {
                    int E = (__builtin_amdgcn_frexp_expf(a) - 1) - (is4 ? 2 : 8);      // floor(log2 a) - emax
                    E = E < -127 ? -127 : (E > 127 ? 127 : E);
                    byte = E + 127;
                }
                const float sc = __int_as_float(byte << 23);                           // (the exponent field is what the conversion takes)
                if (live) {
                    if (is4) {
                        unsigned w = 0;
                        w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, y[0], y[1], sc, 0);
                        w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, y[2], y[3], sc, 1);
                        w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, y[4], y[5], sc, 2);
                        w = __builtin_amdgcn_cvt_scalef32_pk_fp4_f32(w, y[6], y[7], sc, 3);
                        *reinterpret_cast<uint32_t *>(q4 + ((int64_t)gg * rows + row) * 64 + ((j0 & 127) >> 1)) = w;
                    } else {
                        typedef short v2s __attribute__((ext_vector_type(2)));
                        const float top = __builtin_amdgcn_ldexpf(448.0f, byte - 127); // larger magnitudes saturate
                        float c[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) c[e] = __builtin_amdgcn_fmed3f(y[e], -top, top);
                        v2s w0 = {0, 0}, w1 = {0, 0};
                        w0 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w0, c[0], c[1], sc, false);
                        w0 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w0, c[2], c[3], sc, true);
                        w1 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w1, c[4], c[5], sc, false);
                        w1 = __builtin_amdgcn_cvt_scalef32_pk_fp8_f32(w1, c[6], c[7], sc, true);
                        *reinterpret_cast<uint2 *>(q8 + ((int64_t)((j0 - K4) >> 6) * rows + row) * 64 + ((j0 - K4) & 63)) =
                            make_uint2(__builtin_bit_cast(unsigned, w0), __builtin_bit_cast(unsigned, w1));
                    }
                    if ((lane & 3) == 0)
                        reinterpret_cast<uint8_t *>(scale)[((int64_t)gg * rows + row) * 4 + ((j0 >> 5) & 3)] = (uint8_t)byte;
                }
                continue;
            }
            amax = row16_max_dpp(amax);

            float q[8];
            float s;
            const __half sh = quantise_lane8(y, amax, is4, nbits, clip, q, s);
            const bool nz = s != 0.0f;
            if constexpr (PACKED) {
                if (__builtin_expect(__ballot(!nz) != 0, 0)) {      // (a group of zeros: rare, and one branch for the wavefront)
#pragma unroll
                    for (int e = 0; e < 8; ++e) q[e] = nz ? q[e] : 0.0f;
                }
                if (live) {
                    const int pos = lane & 15;                      // 8 channels at 8 * pos of the group
                    const int64_t unit = row >> 6;
                    const int     r    = (int)(row & 63);
                    uint8_t *ubase = pk_out + unit * ((int64_t)G4 * kImg4 + (int64_t)(G - G4) * kImg8);
                    if (is4) {
                        // the E3M2 number of each code (a plain conversion: every code is representable);
                        // eight codes = 48 bits, at byte 6 (pos % 4) of the 24 bytes of their 32-channel block.
                        // (+ 0: a code that was rounded up to zero is -0, and FP6 has a sign bit.  The other 24 numbers are
                        // converted too and not used: whatever the registers hold.)
                        typedef _Float16 v2h __attribute__((ext_vector_type(2)));
                        pk_v32h h;
                        asm volatile("" : "=v"(h));
#pragma unroll
                        for (int e = 0; e < 8; e += 2) {
                            const v2h two = __builtin_bit_cast(v2h, __builtin_amdgcn_cvt_pkrtz(q[e], q[e + 1])) + (v2h)(_Float16)0.0f;
                            h[e] = two[0];
                            h[e + 1] = two[1];
                        }
                        const pk_v6u f6 = __builtin_amdgcn_cvt_scalef32_pk32_bf6_f16(h, 1.0f);
                        const int blk = pos >> 2;                   // block b: half b % 2, first or second MFMA b / 2
                        uint16_t *dst = reinterpret_cast<uint16_t *>(pk_lds + 96 * gg + 48 * (blk & 1) + 24 * (blk >> 1) + 6 * (pos & 3));
                        dst[0] = (uint16_t)f6[0];
                        dst[1] = (uint16_t)(f6[0] >> 16);
                        dst[2] = (uint16_t)f6[1];
                        if (pos == 0)
                            *reinterpret_cast<uint2 *>(at(ubase + kSc4 + 8 * r, (unsigned)gg * kImg4)) = make_uint2(__half_as_ushort(sh), 0u);
                    } else {
                        uint32_t w0 = 0, w1 = 0;
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            w0 |= (uint32_t)((int)q[e] & 0xFF) << (8 * e);
                            w1 |= (uint32_t)((int)q[e + 4] & 0xFF) << (8 * e);
                        }
                        *reinterpret_cast<uint2 *>(pk_lds + 3 * (K4 >> 2) + (j0 - K4)) = make_uint2(w0, w1);
                        if (pos == 0)
                            *reinterpret_cast<uint2 *>(at(ubase + (int64_t)G4 * kImg4 + kSc8 + 8 * r, (unsigned)(gg - G4) * kImg8)) =
                                make_uint2(__half_as_ushort(sh), 0u);
                    }
                }
            } else if (live) {
                if (is4) {
                    const uint32_t w = pack_nibbles8(q);
                    *reinterpret_cast<uint32_t *>(at(q4 + row * (int64_t)(K4 >> 1), (unsigned)j0 >> 1)) = nz ? w : 0u;
                } else {
                    uint32_t w0 = 0, w1 = 0;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        w0 |= (uint32_t)((int)q[e] & 0xFF) << (8 * e);
                        w1 |= (uint32_t)((int)q[e + 4] & 0xFF) << (8 * e);
                    }
                    *reinterpret_cast<uint2 *>(at(q8 + row * (int64_t)O, (unsigned)(j0 - K4))) =
                        make_uint2(nz ? w0 : 0u, nz ? w1 : 0u);
                }
                if ((lane & 15) == 0) *reinterpret_cast<__half *>(at(scale + row * (int64_t)G, 2u * (unsigned)gg)) = sh;
            }
        }
        if (!IDENT || NORM || PACKED) __syncthreads();   // ybuf and qbuf are rewritten by the next row
        if constexpr (PACKED) {
            // the row's packed bytes, 16 at a time: chunk j of the INT4 part is (group j / 6, half
            // (j % 6) / 3, chunk j % 3); chunk j of the INT8 part is (group j / 8, source chunk j % 8)
            const int64_t unit = row >> 6;
            const int     r    = (int)(row & 63);
            uint8_t *ubase = pk_out + unit * ((int64_t)G4 * kImg4 + (int64_t)(G - G4) * kImg8);
            const int n4 = 6 * G4, n8 = O >> 4;
            for (int j = tid; j < n4 + n8; j += NT) {
                const uint4 v = *reinterpret_cast<const uint4 *>(pk_lds + 16 * j);
                unsigned dst;
                if (j < n4) {
                    const unsigned gq = (unsigned)j / 6, hc = j - 6 * gq, hh = hc >= 3 ? 1 : 0, c = hc - 3 * hh;
                    dst = gq * kImg4 + 2048 * c + 1024 * hh + 16 * r;
                } else {
                    const unsigned j8 = j - n4, g8 = j8 >> 3, c = j8 & 7;
                    dst = G4 * kImg4 + g8 * kImg8 + 128 * r + 16 * ((c ^ r ^ ((r >> 3) & 1)) & 7);
                }
                *reinterpret_cast<uint4 *>(at(ubase, dst)) = v;
            }
            if (IDENT && !NORM) __syncthreads();     // (no other barrier stands before the next row's writes to pk_lds)
        }
        if constexpr (ONE) break;
    }
}

}  // namespace atom_quantize_rows
