// Decode-stage attention over the INT4 KV cache for gfx950: reads the cache in 4 bits and dequantises
// inside the operator (Sections 4.4 and 4.5 of the paper); atom_kv_quantize.hip fills it.
//
// Cache layout (one K cache and one V cache, same shape):
//   codes [B, Hkv, Tmax, D/2] bytes, two codes per byte, even d in the low nibble
//   scale [B, Hkv, Tmax] fp16,  zero [B, Hkv, Tmax] int16
// i.e. 64 + 4 bytes per token and head at D = 128: 4.25 bits per element.

#include <hip/hip_runtime.h>
#include <type_traits>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include <atomic>

#include "atom_internal.h"

namespace {

typedef _Float16 h2 __attribute__((ext_vector_type(2)));

// ---------------------------------------------------------------- decode attention

// sum / max over the 16 lanes of a DPP row by rotations
__device__ __forceinline__ float row16_sum(float v)
{
#define ATOM_ROW_ROR(n)                                                                          \
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),   \
                                                               0x120 | (n), 0xF, 0xF, false))
    ATOM_ROW_ROR(8);
    ATOM_ROW_ROR(4);
    ATOM_ROW_ROR(2);
    ATOM_ROW_ROR(1);
#undef ATOM_ROW_ROR
    return v;
}
__device__ __forceinline__ float row16_max(float v)
{
#define ATOM_ROW_ROR(n)                                                                          \
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(                          \
                     0, __builtin_bit_cast(int, v), 0x120 | (n), 0xF, 0xF, false)))
    ATOM_ROW_ROR(8);
    ATOM_ROW_ROR(4);
    ATOM_ROW_ROR(2);
    ATOM_ROW_ROR(1);
#undef ATOM_ROW_ROR
    return v;
}

// The eight codes of a dword (code n in bits 4n..4n+3) as four fp16 pairs with two shifts:
// a code placed in mantissa bits 6..9 under the exponent of 16 reads as 16 + c, one placed
// in bits 2..5 under the exponent of 256 reads as 256 + c, both exactly.
//   pr[0] = (16 + n1, 16 + n5)   pr[1] = (256 + n0, 256 + n4)      from w << 2
//   pr[2] = (16 + n3, 16 + n7)   pr[3] = (256 + n2, 256 + n6)      from w >> 6
// The offsets are subtracted once per sum by the caller.
constexpr int   kNib[4] = {1, 0, 3, 2};                  // low-half code of pair k
constexpr float kOff[4] = {16.0f, 256.0f, 16.0f, 256.0f};

__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t mask, uint32_t magic)
{
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(mask), "v"(magic));
    return r;
}

// All eight as 16 + c, pr[k] = (16 + n_k, 16 + n_(k+4)), with four shifts: for sums whose
// result may be small against the offsets' total (the value side of attention).
__device__ __forceinline__ void unpack8_16(uint32_t w, uint32_t (&pr)[4])
{
    pr[0] = and_or(w << 6, 0x03C003C0u, 0x4C004C00u);
    pr[1] = and_or(w << 2, 0x03C003C0u, 0x4C004C00u);
    pr[2] = and_or(w >> 2, 0x03C003C0u, 0x4C004C00u);
    pr[3] = and_or(w >> 6, 0x03C003C0u, 0x4C004C00u);
}

__device__ __forceinline__ void unpack8(uint32_t w, uint32_t (&pr)[4])
{
    const uint32_t a = w << 2, b = w >> 6;
    pr[0] = and_or(a, 0x03C003C0u, 0x4C004C00u);
    pr[1] = and_or(a, 0x003C003Cu, 0x5C005C00u);
    pr[2] = and_or(b, 0x03C003C0u, 0x4C004C00u);
    pr[3] = and_or(b, 0x003C003Cu, 0x5C005C00u);
}

// max over the lanes l, l ^ 16, l ^ 32, l ^ 48 with the lane-half swaps of gfx950 (vector ALU
// speed; a ds_bpermute pair per exchange would sit on the critical path of every step).  A swap
// exchanges the upper half (32) or the odd rows (16) of its first register with the lower half
// or the even rows of its second; fed two copies of v, the two results hold, lane by lane, v of
// the lane itself and of its partner.  This compiler folds max(first result, second result)
// into the first result, so the second one passes through an empty asm statement (no
// instruction; it only hides where the value came from), and `zero`, a 0 the compiler cannot
// see, keeps the two inputs distinct values.
__device__ __forceinline__ float max_across_chunks(float v, unsigned zero)
{
    typedef unsigned v2ui __attribute__((ext_vector_type(2)));
    unsigned u = __builtin_bit_cast(unsigned, v);
    v2ui r = __builtin_amdgcn_permlane32_swap(u, u | zero, false, false);
    unsigned other = r[1];
    asm volatile("" : "+v"(other));
    u = __builtin_bit_cast(unsigned, fmaxf(__builtin_bit_cast(float, r[0]), __builtin_bit_cast(float, other)));
    r = __builtin_amdgcn_permlane16_swap(u, u | zero, false, false);
    other = r[1];
    asm volatile("" : "+v"(other));
    return fmaxf(__builtin_bit_cast(float, r[0]), __builtin_bit_cast(float, other));
}

// One step of a reduction of four values over the lanes l, l ^ 16, l ^ 32, l ^ 48, each result in one chunk of lanes: a's own and
// its partner row's (half's) value in the rows (the half) that keep a, likewise b's in the others, to be added or compared.
struct Two { float mine, other; };
template <int WIDTH>
__device__ __forceinline__ Two swap_two(float a, float b)
{
    typedef unsigned v2ui __attribute__((ext_vector_type(2)));
    const unsigned ua = __builtin_bit_cast(unsigned, a), ub = __builtin_bit_cast(unsigned, b);
    v2ui r;
    if constexpr (WIDTH == 16) r = __builtin_bit_cast(v2ui, __builtin_amdgcn_permlane16_swap(ua, ub, false, false));
    else                       r = __builtin_bit_cast(v2ui, __builtin_amdgcn_permlane32_swap(ua, ub, false, false));
    unsigned second = r[1];
    asm volatile("" : "+v"(second));      // (as in max_across_chunks)
    return {__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, second)};
}
template <int WIDTH>
__device__ __forceinline__ float swap_max(float a, float b) { const Two t = swap_two<WIDTH>(a, b); return fmaxf(t.mine, t.other); }
template <int WIDTH>
__device__ __forceinline__ float swap_add(float a, float b) { const Two t = swap_two<WIDTH>(a, b); return t.mine + t.other; }

// The way back: o[i] = the value of lane 16 i + (l & 15) in every lane l.
__device__ __forceinline__ void spread(float v, float (&o)[4])
{
    typedef unsigned v2ui __attribute__((ext_vector_type(2)));
    unsigned u = __builtin_bit_cast(unsigned, v), w = u;
    asm volatile("" : "+v"(w));           // (two registers: a swap exchanges parts of them)
    const v2ui r = __builtin_bit_cast(v2ui, __builtin_amdgcn_permlane32_swap(u, w, false, false));
    unsigned a = r[0], b = r[1];
    asm volatile("" : "+v"(b));           // (as in max_across_chunks)
    unsigned a2 = a, b2 = b;
    asm volatile("" : "+v"(a2), "+v"(b2));
    const v2ui x = __builtin_bit_cast(v2ui, __builtin_amdgcn_permlane16_swap(a, a2, false, false));
    const v2ui y = __builtin_bit_cast(v2ui, __builtin_amdgcn_permlane16_swap(b, b2, false, false));
    unsigned x1 = x[1], y1 = y[1];
    asm volatile("" : "+v"(x1), "+v"(y1));
    o[0] = __builtin_bit_cast(float, (unsigned)x[0]);
    o[1] = __builtin_bit_cast(float, x1);
    o[2] = __builtin_bit_cast(float, (unsigned)y[0]);
    o[3] = __builtin_bit_cast(float, y1);
}

// value i (0..31) of the 32 fp16 numbers held by four 16-byte registers (i known at compile time)
__device__ __forceinline__ float half_of(const uint4 (&raw)[4], int i)
{
    const uint4 &v = raw[i >> 3];
    const uint32_t w = ((i >> 1) & 3) == 0 ? v.x : ((i >> 1) & 3) == 1 ? v.y : ((i >> 1) & 3) == 2 ? v.z : v.w;
    return __half2float(__ushort_as_half((unsigned short)((i & 1) ? w >> 16 : w & 0xFFFFu)));
}

// 16 bytes of the cache.  ONCE: with the hint that nothing reads them again (see attention_reads_once).
template <bool ONCE>
__device__ __forceinline__ uint4 load_row(const uint8_t *p)
{
    typedef unsigned v4u_ __attribute__((ext_vector_type(4)));
    if constexpr (ONCE) {
        const v4u_ v = __builtin_nontemporal_load(reinterpret_cast<const v4u_ *>(p));
        return make_uint4(v[0], v[1], v[2], v[3]);
    } else {
        return *reinterpret_cast<const uint4 *>(p);
    }
}

constexpr int kTile  = 16;                // tokens per wavefront step
constexpr int kTokens = 64;                // tokens per wavefront group: four steps, one per ring slot

// One workgroup per (sequence, query head) and split of the token range, head dimension 128.
// A wavefront owns every kWaves-th group of 64 tokens and walks it in four steps of 16 tokens:
// lane l holds token (l & 15) and the 32 head dimensions of chunk (l >> 4), i.e. 16 bytes of
// that token's K row and 16 bytes of its V row (a wavefront load is 1 KB of contiguous cache).
//   scores  : the codes become fp16 offset + c, two at a time (unpack8), and meet the
//             matching pairs of q in v_dot2_f32_f16 (fp32 accumulate); the offsets and the
//             zero point leave as sum(offset * q) + z * sum(q) per chunk (offsets of 16 and
//             256 keep the cancellation in fp32 harmless); all four steps first, then the four chunks of a
//             token are added across lanes such that lane l ends with token l of the group, where its scales are;
//             then * scale * sm_scale.
//   softmax : online, per wavefront (running max m and sum l), in the order of the steps, but the maxima, weights and sums of the
//             four steps are found together and spread to the lanes afterwards; the accumulators are rescaled
//             only when the maximum moves.
//   values  : acc[d] += w * (16 + code[d]) with w = p * v_scale (unpack8_16), the fp16 codes
//             read by mixed-precision fmas; the 16 and the zero points leave once per group
//             of 64 tokens through the sums of w and w * z; the 16 tokens of the lanes meet
//             once, at the end, each half of them keeping half of the values; the wavefronts merge through LDS.
//   What bounds it besides the memory: the vector instructions of a group, at four cycles each (two for fp32 additions and fused
//             multiply-adds): of 2200 cycles 640 for the scores' codes and products and 1024 for the values'.  Against one step after the
//             other with its own cross-lane work (32 heads, lengths from T / 4 to T, us): 64 x 1024 40.9 -> 39.8, 64 x 200 17.0 -> 16.2,
//             128 x 512 42.8 -> 41.6, 64 x 2048 67.0 -> 66.3, 16 x 1024 19.5 -> 18.9, 8 x 1024 12.2 either way.  Same sums in the same
//             order, the same bits.  (Codes as subnormal numbers, one shift and four ands for eight of them, and no offsets to take out:
//             12 to 19 % faster and no less exact, but other roundings, which a decoder's next quantisation turns into other codes.)
//   loads   : the codes of the next group (four steps ahead) are in flight while a step is
//             computed.  Scales and zero points are read once per group, lane l taking
//             token l of the 64, one full cache line per array: 2-byte loads per step would have several
//             wavefronts wait on the same line, which stalls the vector cache.
//             q is asked for before everything else: loads return in order, and a conversion of q that waits for the first
//             rows as well delays every wavefront's first scores.  Lengths from T / 4 to T, us, q behind the rows and in
//             front of them: 256 heads, T = 1024 12.8 -> 12.0; 512 heads, T = 700 16.1 -> 15.3; 4096 heads, T = 200 28.9 ->
//             27.4; 1200 heads, T = 3000 67.2 -> 64.9; 2048 heads, T = 2048 (5.1 TB/s of cache bytes) 74.2 -> 73.6.
template <int kWaves, bool ONCE>          // wavefronts per workgroup: 4, or 16 when B * H alone is a thin grid
__global__ __launch_bounds__(kWaves * 64)
void decode_attention_kv4_kernel(const __half *__restrict__ q, int H, int Hkv, int64_t Tmax,
                                 const int32_t *__restrict__ seq_len,
                                 const uint8_t *__restrict__ kq, const __half *__restrict__ ks,
                                 const int16_t *__restrict__ kz, const uint8_t *__restrict__ vq,
                                 const __half *__restrict__ vs, const int16_t *__restrict__ vz,
                                 float sm_scale, __half *__restrict__ out, int groups_per_split,
                                 float *__restrict__ part)
{
    constexpr int D = 128;
    __shared__ float s_acc[kWaves][D];
    __shared__ float s_m[kWaves], s_l[kWaves];

    const int b = blockIdx.x / H, h = blockIdx.x % H;
    const int kvh = h / (H / Hkv);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tl = lane & 15, c = lane >> 4;
    uint4 qraw[4];                        // this lane's 32 query values (32 two-byte loads cost a microsecond of prologue)
#pragma unroll
    for (int j = 0; j < 4; ++j) qraw[j] = *reinterpret_cast<const uint4 *>(q + ((int64_t)b * H + h) * D + 32 * c + 8 * j);
    int T = seq_len[b];
    T = T < 0 ? 0 : (T > Tmax ? (int)Tmax : T);          // never read past the cache
    const int64_t base = ((int64_t)b * Hkv + kvh) * Tmax;
    const uint8_t *kb = kq + base * (D / 2), *vb = vq + base * (D / 2);
    const __half  *ksb = ks + base, *vsb = vs + base;
    const int16_t *kzb = kz + base, *vzb = vz + base;

    // this workgroup's share of the groups (all of them when the grid has one split)
    const int g_first = blockIdx.y * groups_per_split;
    const int g_end   = min((T + kTokens - 1) / kTokens, g_first + groups_per_split);
    int  G     = g_first + wave;
    const bool alive = G < g_end;                        // then T >= 1: clamped addresses are valid
    const int  t_last = min(T, g_end * kTokens) - 1;     // loads never leave this split's tokens

    uint4 kst[4], vst[4];
    uint32_t kmeta = 0, vmeta = 0;        // scale bits | zero << 16 of token `lane` of the group
    auto row_of = [&](int tile) -> uint32_t {
        int t = tile * kTile + tl;
        t = t <= t_last ? t : t_last;     // masked tokens and steps past the end repeat the last token
        return (uint32_t)t * (D / 2) + 16u * c;
    };
    auto fetch_meta = [&](int g, uint32_t &km, uint32_t &vm) {
        int t = g * kTokens + lane;
        t = t <= t_last ? t : t_last;
        km = (uint32_t)__half_as_ushort(ksb[(uint32_t)t]) | ((uint32_t)(uint16_t)kzb[(uint32_t)t] << 16);
        vm = (uint32_t)__half_as_ushort(vsb[(uint32_t)t]) | ((uint32_t)(uint16_t)vzb[(uint32_t)t] << 16);
    };
    float m_run = -INFINITY, l_run = 0.0f;
    if (alive) {                          // every first load leaves before any is waited for, q first: loads return in order
        fetch_meta(G, kmeta, vmeta);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t off = row_of(4 * G + i);
            kst[i] = load_row<ONCE>(kb + off);
            vst[i] = load_row<ONCE>(vb + off);
        }
        __builtin_amdgcn_sched_barrier(0);
        // this lane's 32 query values as 16 pairs in the order unpack8 delivers the codes of a
        // dword (dword j holds d = 32c + 8j + 0..7), and the sums that take the offsets back out
        h2 qp[16];
        float qsum = 0.0f, qoff = 0.0f;       // sum(q), sum(offset(d) * q)
        {
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float lo = half_of(qraw, 8 * j + kNib[k]), hi = half_of(qraw, 8 * j + kNib[k] + 4);
                    qp[4 * j + k] = h2{(_Float16)lo, (_Float16)hi};
                    qsum += lo + hi;
                    qoff += kOff[k] * (lo + hi);
                }
        }
        float acc[32];                    // acc[8j + 2k + half] <-> d = 32c + 8j + k + 4 half
#pragma unroll
        for (int i = 0; i < 32; ++i) acc[i] = 0.0f;

        while (G < g_end) {
            const int Gn = G + kWaves;                    // past the end: clamped, unused loads
            uint32_t nk, nv;
            fetch_meta(Gn, nk, nv);
            const int steps = (T - G * kTokens + kTile - 1) / kTile;      // those that hold tokens: four and more but for a sequence's last group
            // ---- scores: every lane its chunk of head dimensions of token tl of each step ...
            float dot[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            auto product = [&](int i) __attribute__((always_inline)) {
                const uint32_t kw[4] = {kst[i].x, kst[i].y, kst[i].z, kst[i].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    uint32_t pr[4];
                    unpack8(kw[j], pr);
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        dot[i] = __builtin_amdgcn_fdot2(__builtin_bit_cast(h2, pr[k]), qp[4 * j + k], dot[i], false);
                }
            };
            product(0);
            if (steps > 1) {
                product(1);
                product(2);
                product(3);
            }
            uint32_t row[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {                 // the slot's next use is a group away (on every path: the compiler counts the loads in flight)
                row[i] = row_of(4 * Gn + i);
                kst[i] = load_row<ONCE>(kb + row[i]);
            }
            float kz[4];
            spread((float)(int16_t)(kmeta >> 16), kz);
#pragma unroll
            for (int i = 0; i < 4; ++i) dot[i] -= fmaf(kz[i], qsum, qoff);
            // ... and the four chunks meet in lane 16 i + tl: lane l has token l of the group, as it has its scales
            const float sum = swap_add<32>(swap_add<16>(dot[0], dot[1]), swap_add<16>(dot[2], dot[3]));
            const float k_s = __half2float(__ushort_as_half((unsigned short)(kmeta & 0xFFFFu)));
            const float score = G * kTokens + lane < T ? sum * (k_s * sm_scale) : -INFINITY;

            // ---- online softmax, step by step (every lane of the wavefront has the same m and l)
            float mx[4], m[5];
            spread(row16_max(score), mx);
            m[0] = m_run;
#pragma unroll
            for (int i = 0; i < 4; ++i) m[i + 1] = fmaxf(m[i], mx[i]);
            const bool  moved = m[4] > m_run;             // rare after the first groups; the same decision in every lane
            const float m_lo = c & 1 ? m[2] : m[1], m_hi = c & 1 ? m[4] : m[3];
            const float p = __expf(score - (c & 2 ? m_hi : m_lo));
            float ps[4], alpha[4];
            spread(row16_sum(p), ps);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                alpha[i] = 1.0f;
                if (moved) alpha[i] = m[i + 1] > m[i] ? __expf(m[i] - m[i + 1]) : 1.0f;   // 0 on the first step
                l_run = l_run * alpha[i] + ps[i];
            }
            m_run = m[4];

            // ---- values: the fp16 halves go straight into mixed-precision fmas
            float w[4], vz[4];
            spread(p * __half2float(__ushort_as_half((unsigned short)(vmeta & 0xFFFFu))), w);
            spread((float)(int16_t)(vmeta >> 16), vz);
            float wsum = 0.0f, zacc = 0.0f;               // sums of w = p * v_scale and of w * v_zero of this group
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (i == 0 || i < steps) {
                    if (moved) {
                        wsum *= alpha[i];
                        zacc *= alpha[i];
#pragma unroll
                        for (int e = 0; e < 32; ++e) acc[e] *= alpha[i];
                    }
                    wsum += w[i];
                    zacc = fmaf(w[i], vz[i], zacc);
                    const uint32_t vw[4] = {vst[i].x, vst[i].y, vst[i].z, vst[i].w};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        uint32_t pr[4];
                        unpack8_16(vw[j], pr);
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const h2 cv = __builtin_bit_cast(h2, pr[k]);
                            acc[8 * j + 2 * k]     = fmaf(w[i], (float)cv[0], acc[8 * j + 2 * k]);
                            acc[8 * j + 2 * k + 1] = fmaf(w[i], (float)cv[1], acc[8 * j + 2 * k + 1]);
                        }
                    }
                }
                vst[i] = load_row<ONCE>(vb + row[i]);
            }
            // the offsets of this group's four steps leave the accumulators now, not at the end:
            // left in, their sum grows with the sequence and its rounding would show in
            // outputs that are small against it
            const float off = fmaf(16.0f, wsum, zacc);
#pragma unroll
            for (int i = 0; i < 32; ++i) acc[i] -= off;
            kmeta = nk;
            vmeta = nv;
            G = Gn;
        }

        // ---- the 16 tokens of the lanes meet, half of the values at a time in each half of them: lanes that differ in bits 3, 2, 1, 0
        // keep the upper or the lower half of what both have; lane l ends with acc[2 (l & 15)] and the next
        auto meet = [&](auto n_c, auto from_other) __attribute__((always_inline)) {
            constexpr int n = decltype(n_c)::value;                 // values kept; the lanes differ in bit n / 2
            const bool up = (lane & (n / 2)) != 0;
#pragma unroll
            for (int i = 0; i < n; ++i) {
                const float keep = up ? acc[i + n] : acc[i], give = up ? acc[i] : acc[i + n];
                acc[i] = keep + __builtin_bit_cast(float, from_other(__builtin_bit_cast(int, give)));
            }
        };
        meet(std::integral_constant<int, 16>(), [](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, false); });   // row_ror:8
        meet(std::integral_constant<int, 8>(), [](int v) {          // from four lanes on and from four lanes back
            return __builtin_amdgcn_update_dpp(__builtin_amdgcn_update_dpp(0, v, 0x12C, 0xF, 0xF, false), v, 0x124, 0xF, 0xA, false);
        });
        meet(std::integral_constant<int, 4>(), [](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false); });     // quad_perm
        meet(std::integral_constant<int, 2>(), [](int v) { return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false); });
        float *dst = &s_acc[wave][32 * c + 8 * (tl >> 2) + (tl & 3)];
        dst[0] = acc[0];
        dst[4] = acc[1];
    }
    if (lane == 0) {
        s_m[wave] = m_run;
        s_l[wave] = l_run;
    }
    __syncthreads();

    // ---- merge the wavefronts: out = sum_w e^(m_w - M) acc_w / sum_w e^(m_w - M) l_w (a wavefront without tokens has left no acc_w)
    if (tid < D) {
        float M = s_m[0];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) M = fmaxf(M, s_m[w]);
        float num = 0.0f, den = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const bool  none = s_m[w] == -INFINITY;
            const float e = none ? 0.0f : __expf(s_m[w] - M);
            num += none ? 0.0f : e * s_acc[w][tid];
            den += e * s_l[w];
        }
        if (part == nullptr) {
            out[((int64_t)b * H + h) * D + tid] = __float2half_rn(den > 0.0f ? num / den : 0.0f);
        } else {                                          // one partial (M, den, num[D]) per split
            float *dst = part + ((int64_t)blockIdx.x * gridDim.y + blockIdx.y) * (D + 2);
            dst[2 + tid] = num;
            if (tid == 0) {
                dst[0] = M;
                dst[1] = den;
            }
        }
    }
}

// ---------------------------------------------------------------- grouped-query variant

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef float    v4f __attribute__((ext_vector_type(4)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));

__device__ __forceinline__ v8h quad_operand(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    const v4u t = {a, b, c, d};
    return __builtin_bit_cast(v8h, t);
}

// unpack8_16 in plain C: these values feed MFMAs, and the wait states an MFMA needs after the
// instruction that wrote its operand are only inserted for instructions the compiler can see
// (mask and magic arrive in registers whose contents the compiler cannot see: with literal
// constants it emits an and and an or, with register operands the fused v_and_or_b32)
__device__ __forceinline__ void unpack8_16_mfma(uint32_t w, uint32_t mask, uint32_t magic, uint32_t (&pr)[4])
{
    pr[0] = ((w << 6) & mask) | magic;
    pr[1] = ((w << 2) & mask) | magic;
    pr[2] = ((w >> 2) & mask) | magic;
    pr[3] = ((w >> 6) & mask) | magic;
}

constexpr int kGqaWaves    = 4;
constexpr int kGqaMaxHeads = 16;          // query heads per cache head served by one MFMA column block
constexpr int kGqaHeadPitch = 4 * 33 + 1; // floats per head in the merge area (32 + 1 per chunk, + 1)

// One workgroup per (sequence, CACHE head) and split of the token range: the Gq = H / Hkv
// query heads that share a cache head (2 <= Gq <= 16) share every load and every unpacked
// code, and both contractions run on the fp16 MFMA 16x16x32 (lane l supplies row or column
// l & 15 and the eight k of chunk l >> 4; the result has column l & 15 in lane l and rows
// 4 (l >> 4) + e in register e).  A wavefront owns every fourth group of 64 tokens, four steps of 16 tokens.
//   scores  : S[t, h] = sum_d (16 + code[t, d]) q[h, d]: the row operand is the K codes as
//             fp16 16 + c (lane = token l & 15, 32 head dimensions of chunk l >> 4, four
//             MFMAs), the column operand q in the same order of d (registers, loaded once);
//             the result leaves head h = l & 15 and tokens 4 (l >> 4) + e in lane l, and
//             score = k_scale sm_scale (S - (16 + k_zero) sum_d q).  All four steps first: their
//             chains of MFMAs and the exchanges of the maximum are independent of each other.  The last group of a sequence does
//             the MFMAs of the steps that hold tokens only (1 to 10 tokens, 64 heads on 8: 6.2 us, 5.3 so; 1 to 60 7.9, 7.3), but every
//             load, tokens or not: where paths with and without loads meet, the wait for the next rows is for the fewer in
//             flight (with the value loads left out too, 64 x 4096 tokens took 59.8 us instead of 56.4).
//   softmax : online per head and step; the four lanes of a head agree on the maxima of the four steps (three
//             swaps of lane halves gather them, three bring them back), each keeps the partial sums of its own tokens;
//             accumulators are rescaled when the maximum moves.
//   values  : out^T[d, h] = sum_t (code[t, d] - zero[t]) w[t, h]: the weights are already laid
//             out as the column operand (tokens 4 (l >> 4) + i of head l & 15); the row
//             operand wants four TOKENS of one d per lane, so the V codes are loaded four
//             bytes per lane and token (lane = d group l & 15 of 8 head dimensions, tokens
//             4 (l >> 4) + i), transposed as bytes in registers and unpacked two tokens at a
//             time; tile j of the eight result tiles holds d = 8 (row) + j, so lane l ends
//             with d = 32 (l >> 4) + 8 e + j of head l & 15.
//             The weights must fit fp16 whatever the scales are:
//             w = p * v_scale * 2^15 / R, R the largest v_scale this wavefront has met so far
//             (fixed per group of 64 tokens; when a new group raises it, the accumulators are
//             rescaled, as for the running maximum of the scores): at most 2^15, and a normal
//             fp16 number down to 2^-29 of that.  One fp16 number per weight is not enough (its rounding alone shows
//             as 1e-2 of the small outputs of a head): w travels as fp16 hi + fp16 lo, one
//             16x16x16 MFMA for each against the same value operand.
//             The zero point leaves BEFORE the contraction, so the sums carry no offset that a long context
//             would have to cancel: bits 0..3 of a half word are the (subnormal) fp16 number code 2^-24, bits 4..7 code
//             2^-20, and one packed fma makes (code - zero) 2^-9 of either, exactly.  Zero points beyond +-1000
//             (rows whose values all sit far on one side of zero) are taken out up to that
//             bound, the rest leaves through sum_t w * rest as in the per-head kernel.
//   scales  : lane l reads the scale and zero point of token l of the group (one cache line
//             per array) and parks what the steps need in LDS, where a step reads its four tokens' worth as broadcasts.
// What bounds it: the chain of instructions of a wavefront (the grid leaves one to three per SIMD).  A group takes about 5300
// cycles alone on its SIMD, 630 to 770 of vector ALU instructions at 4 cycles, and 80 MFMAs at 16 of which the scheduling below
// hides most.  Alone, 64 heads on 8, lengths from T / 4 to T, us, against one step after the other with its own maximum, clamped
// addresses and loads that waited for the scales: 16 sequences of 4096 25.2 -> 23.0, 128 of 2048 58.1 -> 50.2, 64 of
// 1024 21.7 -> 19.3, 100 of 500 21.4 -> 17.8, 1 of 16384 16.0 -> 14.9.  Every sum keeps its order: the same bits.
// ONCE: the K rows are loaded with the hint that nothing reads them again; the V rows are not, since a 128-byte line of them holds two
// tokens, which two of a wavefront's loads take.
template <bool ONCE>
__global__ __launch_bounds__(kGqaWaves * 64)
void decode_attention_kv4_gqa_kernel(const __half *__restrict__ q, int H, int Hkv, int64_t Tmax,
                                     const int32_t *__restrict__ seq_len,
                                     const uint8_t *__restrict__ kq, const __half *__restrict__ ks,
                                     const int16_t *__restrict__ kz, const uint8_t *__restrict__ vq,
                                     const __half *__restrict__ vs, const int16_t *__restrict__ vz,
                                     float sm_scale, __half *__restrict__ out, int groups_per_split,
                                     float *__restrict__ part)
{
    constexpr int D = 128;
    constexpr int kWaves = kGqaWaves;
    __shared__ __align__(16) float s_meta[kWaves][3][kTokens];
    __shared__ __align__(16) _Float16 s_zero[kWaves][kTokens];
    __shared__ __align__(16) float s_rest[kWaves][kTokens];
    __shared__ float  s_m[kWaves][kGqaMaxHeads], s_l[kWaves][kGqaMaxHeads];
    extern __shared__ __align__(16) float s_acc[];        // [kWaves][Gq][kGqaHeadPitch]

    const int Gq = H / Hkv;
    const int b = blockIdx.x / Hkv, kvh = blockIdx.x % Hkv;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int x = lane & 15, c = lane >> 4;
    // (every argument is fetched before the first wait for any: the compiler would leave most for after the length)
    asm volatile("" : : "s"(q), "s"(kq), "s"(ks), "s"(kz), "s"(vq), "s"(vs), "s"(vz), "s"(sm_scale), "s"(groups_per_split));
    int T = seq_len[b];
    T = T < 0 ? 0 : (T > Tmax ? (int)Tmax : T);
    const int64_t base = ((int64_t)b * Hkv + kvh) * Tmax;
    const uint8_t *kb = kq + base * (D / 2), *vb = vq + base * (D / 2);
    const __half  *ksb = ks + base, *vsb = vs + base;
    const int16_t *kzb = kz + base, *vzb = vz + base;

    const int g_first = blockIdx.y * groups_per_split;
    const int g_end   = min((T + kTokens - 1) / kTokens, g_first + groups_per_split);
    int  G     = g_first + wave;
    const bool alive = G < g_end;                        // then T >= 1: clamped addresses are valid
    const int  t_last = min(T, g_end * kTokens) - 1;     // loads never leave this split's tokens

    uint4 kst[4];
    struct Rows { uint32_t v0, v1, v2, v3; };
    Rows vst[4];
    const float k_mul = sm_scale * 1.44269504088896340736f;   // scores in units of log2: exp2 below
    // A step is 16 rows of 64 bytes.  Rows past t_last (masked tokens, steps past the end) lie past the end of the buffer that
    // the descriptors state: they read as 0 and touch no memory.
    const uint32_t k_lane = 64u * x + 16u * c, v_lane = 64u * (4u * c) + 4u * x;
    const auto k_rows = __builtin_amdgcn_make_buffer_rsrc((void *)kb, 0, 64u * (uint32_t)(t_last + 1), 0x00020000);
    const auto v_rows = __builtin_amdgcn_make_buffer_rsrc((void *)vb, 0, 64u * (uint32_t)(t_last + 1), 0x00020000);
    auto k_of = [&](int tile) {
        return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(k_rows, (uint32_t)tile * (kTile * 64u) + k_lane, 0, ONCE ? 2 : 0));
    };
    auto v_of = [&](int tile) {
        const uint32_t t0 = (uint32_t)tile * (kTile * 64u) + v_lane;
        return Rows{__builtin_amdgcn_raw_buffer_load_b32(v_rows, t0, 0, 0), __builtin_amdgcn_raw_buffer_load_b32(v_rows, t0 + 64u, 0, 0),
                    __builtin_amdgcn_raw_buffer_load_b32(v_rows, t0 + 128u, 0, 0), __builtin_amdgcn_raw_buffer_load_b32(v_rows, t0 + 192u, 0, 0)};
    };
    // scales and zero points of token `lane` of group g, raw
    struct Meta { __half ks, vs; int16_t kz, vz; };
    auto fetch_meta = [&](int g) {
        int t = g * kTokens + lane;
        t = t <= t_last ? t : t_last;
        return Meta{ksb[(uint32_t)t], vsb[(uint32_t)t], kzb[(uint32_t)t], vzb[(uint32_t)t]};
    };
    v4f acc[8];                           // acc[j][e] <-> out[head x][d = 32c + 8e + j], in units of R / 2^6
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    float m_run = -INFINITY, l_run = 0.0f, off_run = 0.0f;    // l and off: this lane's tokens only
    float R = 0.0f;                       // largest v_scale met so far (the same in every lane)
    unsigned c_zero = 0u;
    asm volatile("" : "+s"(c_zero));
    bool  has_rest = false;               // some zero point of the current group was clamped
    // ... as k_scale sm_scale log2 e, 16 + k_zero, v_scale * 2^15 / R and (16 - (16 + v_zero clamped to +-1000)) / 2^9 into
    // LDS, what the clamp cut off (/ 2^9) beside it
    auto install_meta = [&](const Meta &mt) {
        const float v_s = __half2float(mt.vs);
        const float Rn  = fmaxf(R, max_across_chunks(row16_max(v_s), c_zero));
        if (Rn > R) {                     // the same decision in every lane; rare after the first groups
            const float down = R / Rn;    // 0 the first time
            off_run *= down;
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] *= down;
            R = Rn;
        }
        const float rinv  = R > 0.0f ? 32768.0f / R : 0.0f;
        const float v_off = 16.0f + (float)mt.vz;
        const float v_cut = fminf(fmaxf(v_off, -1000.0f), 1000.0f);
        s_meta[wave][0][lane] = __half2float(mt.ks) * k_mul;
        s_meta[wave][1][lane] = 16.0f + (float)mt.kz;
        s_meta[wave][2][lane] = v_s * rinv;
        s_zero[wave][lane] = (_Float16)((16.0f - v_cut) * (1.0f / 512.0f));
        s_rest[wave][lane] = (v_off - v_cut) * (1.0f / 512.0f);
        has_rest = __ballot(v_off != v_cut) != 0;
    };
    if (alive) {
        // every first load leaves before any is waited for, in the order in which they are needed
        const bool live = x < Gq;
        uint4 qraw[4];                        // 64 bytes as four loads
        {
            const __half *qv = q + ((int64_t)b * H + (int64_t)kvh * Gq + (live ? x : 0)) * D + 32 * c;
#pragma unroll
            for (int j = 0; j < 4; ++j) qraw[j] = *reinterpret_cast<const uint4 *>(qv + 8 * j);
        }
        const Meta first = fetch_meta(G);
#pragma unroll
        for (int i = 0; i < 4; ++i) kst[i] = k_of(4 * G + i);
#pragma unroll
        for (int i = 0; i < 4; ++i) vst[i] = v_of(4 * G + i);
        __builtin_amdgcn_sched_barrier(0);    // (or the waits for the scales move between the loads)
        install_meta(first);

        // q of head x as the column operand: MFMA j of a step contracts, for chunk c, the head
        // dimensions 32c + 8j + {0, 4, 1, 5, 2, 6, 3, 7} (the order unpack8_16 delivers)
        v8h qb[4];
        float qsum = 0.0f;
        {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float e[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) e[i] = live ? half_of(qraw, 8 * j + (i >> 1) + 4 * (i & 1)) : 0.0f;
                qb[j] = v8h{(_Float16)e[0], (_Float16)e[1], (_Float16)e[2], (_Float16)e[3],
                            (_Float16)e[4], (_Float16)e[5], (_Float16)e[6], (_Float16)e[7]};
                qsum += ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7]));
            }
            qsum += __shfl_xor(qsum, 16, 64);
            qsum += __shfl_xor(qsum, 32, 64);
        }

        uint32_t c_mask = 0x03C003C0u, c_magic = 0x4C004C00u;
        asm volatile("" : "+s"(c_mask));
        asm volatile("" : "+v"(c_magic));

        const h2 c_even = {(_Float16)32768.0f, (_Float16)32768.0f}, c_odd = {(_Float16)2048.0f, (_Float16)2048.0f};
        while (G < g_end) {
            const int Gn = G + kWaves;                    // past the end: clamped, unused loads
            const Meta meta_next = fetch_meta(Gn);
            const int steps = (T - G * kTokens + kTile - 1) / kTile;      // those that hold tokens: four and more but for a sequence's last group
            // ---- scores of the four steps
            v4f sa[4];
            auto products = [&](int i) __attribute__((always_inline)) {
                const uint32_t kw[4] = {kst[i].x, kst[i].y, kst[i].z, kst[i].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    uint32_t pr[4];
                    unpack8_16_mfma(kw[j], c_mask, c_magic, pr);
                    sa[i] = __builtin_amdgcn_mfma_f32_16x16x32_f16(quad_operand(pr[0], pr[1], pr[2], pr[3]), qb[j], sa[i], 0, 0, 0);
                }
            };
            sa[0] = sa[1] = sa[2] = sa[3] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
            products(0);
            if (steps > 1) {
                products(1);
                products(2);
                products(3);
            }
            float sc[4][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                kst[i] = k_of(4 * Gn + i);
                const float4 ks4 = *reinterpret_cast<const float4 *>(&s_meta[wave][0][16 * i + 4 * c]);
                const float4 kz4 = *reinterpret_cast<const float4 *>(&s_meta[wave][1][16 * i + 4 * c]);
                sc[i][0] = ks4.x * fmaf(-kz4.x, qsum, sa[i][0]);
                sc[i][1] = ks4.y * fmaf(-kz4.y, qsum, sa[i][1]);
                sc[i][2] = ks4.z * fmaf(-kz4.z, qsum, sa[i][2]);
                sc[i][3] = ks4.w * fmaf(-kz4.w, qsum, sa[i][3]);
            }
            if ((G + 1) * kTokens > T) {                  // the end of the sequence: a weight of 0 from there on
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (G * kTokens + 16 * i + 4 * c + e >= T) sc[i][e] = -INFINITY;
            }
            // ---- online softmax per head, step by step: the four lanes of a head take the same decisions
            float mx[4], m[5];
#pragma unroll
            for (int i = 0; i < 4; ++i) mx[i] = fmaxf(fmaxf(sc[i][0], sc[i][1]), fmaxf(sc[i][2], sc[i][3]));
            spread(swap_max<32>(swap_max<16>(mx[0], mx[1]), swap_max<16>(mx[2], mx[3])), mx);
            m[0] = m_run;
#pragma unroll
            for (int i = 0; i < 4; ++i) m[i + 1] = fmaxf(m[i], mx[i]);
            m_run = m[4];
            float w[4][4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 vs4 = *reinterpret_cast<const float4 *>(&s_meta[wave][2][16 * i + 4 * c]);
                const float vs_[4] = {vs4.x, vs4.y, vs4.z, vs4.w};
                if (m[i + 1] > m[i]) l_run *= __builtin_amdgcn_exp2f(m[i] - m[i + 1]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float p = __builtin_amdgcn_exp2f(sc[i][e] - m[i + 1]);
                    l_run += p;
                    w[i][e] = p * vs_[e];
                }
            }
            // ---- values
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (i == 0 || i < steps) {
                    if (__any(m[i + 1] > m[i])) {
                        const float alpha = m[i + 1] > m[i] ? __builtin_amdgcn_exp2f(m[i] - m[i + 1]) : 1.0f;   // 0 on the first step
                        off_run *= alpha;
#pragma unroll
                        for (int j = 0; j < 8; ++j) acc[j] *= alpha;
                    }
                    // w = hi + lo: hi by the packed conversion (which truncates: any rounding will do, lo
                    // takes what hi leaves), two tokens per instruction
                    const h2 hi01 = __builtin_bit_cast(h2, __builtin_amdgcn_cvt_pkrtz(w[i][0], w[i][1]));
                    const h2 hi23 = __builtin_bit_cast(h2, __builtin_amdgcn_cvt_pkrtz(w[i][2], w[i][3]));
                    const h2 lo01 = __builtin_bit_cast(h2, __builtin_amdgcn_cvt_pkrtz(w[i][0] - (float)hi01[0], w[i][1] - (float)hi01[1]));
                    const h2 lo23 = __builtin_bit_cast(h2, __builtin_amdgcn_cvt_pkrtz(w[i][2] - (float)hi23[0], w[i][3] - (float)hi23[1]));
                    if (has_rest) {               // rare: the part of a zero point the operands cannot carry
                        const float *rs = &s_rest[wave][16 * i + 4 * c];   // (hi + lo is w to 2^-22)
#pragma unroll
                        for (int e = 0; e < 4; ++e) off_run = fmaf(w[i][e], rs[e], off_run);
                    }
                    const v4h pb_hi = {hi01[0], hi01[1], hi23[0], hi23[1]}, pb_lo = {lo01[0], lo01[1], lo23[0], lo23[1]};
                    const v4h z4 = *reinterpret_cast<const v4h *>(&s_zero[wave][16 * i + 4 * c]);
                    const h2 z01 = {z4[0], z4[1]}, z23 = {z4[2], z4[3]};

                    // byte transpose (token i of this lane = dword v_i), then two tokens per unpack
                    const uint32_t w0 = vst[i].v0, w1 = vst[i].v1, w2 = vst[i].v2, w3 = vst[i].v3;
                    // v_perm_b32 picks each result byte out of eight: 0-3 the second operand's, 4-7 the first's
                    constexpr uint32_t kZipLo = 0x05010400u;          // [b.0 a.0 b.1 a.1] of perm(a, b)
                    constexpr uint32_t kZipHi = 0x07030602u;          // [b.2 a.2 b.3 a.3]
                    // L01 = [t0.b0 t1.b0 t0.b1 t1.b1], H01 = [t0.b2 t1.b2 t0.b3 t1.b3] (byte 0 first)
                    const uint32_t L01 = __builtin_amdgcn_perm(w1, w0, kZipLo), H01 = __builtin_amdgcn_perm(w1, w0, kZipHi);
                    const uint32_t L23 = __builtin_amdgcn_perm(w3, w2, kZipLo), H23 = __builtin_amdgcn_perm(w3, w2, kZipHi);
                    // Y_b = [t0.b t2.b t1.b t3.b]: the codes of tokens 0 and 1 sit 16 bits apart, as do 2 and 3
                    uint32_t Y[4];
                    Y[0] = __builtin_amdgcn_perm(L23, L01, kZipLo);
                    Y[1] = __builtin_amdgcn_perm(L23, L01, kZipHi);
                    Y[2] = __builtin_amdgcn_perm(H23, H01, kZipLo);
                    Y[3] = __builtin_amdgcn_perm(H23, H01, kZipHi);
#pragma unroll
                    for (int bt = 0; bt < 4; ++bt) {
                        const uint32_t up = Y[bt] >> 8;
                        const h2 e01 = __builtin_elementwise_fma(__builtin_bit_cast(h2, Y[bt] & 0x000F000Fu), c_even, z01);
                        const h2 o01 = __builtin_elementwise_fma(__builtin_bit_cast(h2, Y[bt] & 0x00F000F0u), c_odd, z01);
                        const h2 e23 = __builtin_elementwise_fma(__builtin_bit_cast(h2, up & 0x000F000Fu), c_even, z23);
                        const h2 o23 = __builtin_elementwise_fma(__builtin_bit_cast(h2, up & 0x00F000F0u), c_odd, z23);
                        const v4h ve = {e01[0], e01[1], e23[0], e23[1]}, vo = {o01[0], o01[1], o23[0], o23[1]};     // even / odd d of byte bt
                        acc[2 * bt]     = __builtin_amdgcn_mfma_f32_16x16x16f16(ve, pb_hi, acc[2 * bt], 0, 0, 0);
                        acc[2 * bt + 1] = __builtin_amdgcn_mfma_f32_16x16x16f16(vo, pb_hi, acc[2 * bt + 1], 0, 0, 0);
                        acc[2 * bt]     = __builtin_amdgcn_mfma_f32_16x16x16f16(ve, pb_lo, acc[2 * bt], 0, 0, 0);
                        acc[2 * bt + 1] = __builtin_amdgcn_mfma_f32_16x16x16f16(vo, pb_lo, acc[2 * bt + 1], 0, 0, 0);
                    }
                    // an MFMA takes the matrix core 16 cycles: three vector instructions between one and the next, as far as they go
                    __builtin_amdgcn_sched_group_barrier(0x002, 40, 0);
#pragma unroll
                    for (int n = 0; n < 16; ++n) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
                    }
                }
                vst[i] = v_of(4 * Gn + i);                // (on every path: the compiler counts the loads in flight)
            }
            if (has_rest) {                               // what the operands could not carry of the zero points
                float off = off_run;
                off += __shfl_xor(off, 16, 64);
                off += __shfl_xor(off, 32, 64);
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] -= off;
                off_run = 0.0f;
            }
            install_meta(meta_next);                      // every read of this group's entries is done
            G = Gn;
        }
    }

    // ---- the wavefronts merge through LDS: out = sum_w e^(m_w - M) acc_w / sum_w e^(m_w - M) l_w
    l_run += __shfl_xor(l_run, 16, 64);
    l_run += __shfl_xor(l_run, 32, 64);
    if (x < Gq) {
        float *dst = s_acc + ((size_t)wave * Gq + x) * kGqaHeadPitch + 33 * c;
#pragma unroll
        for (int j = 0; j < 8; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) dst[8 * e + j] = acc[j][e] * (R * (1.0f / 64.0f));
        if (c == 0) {
            s_m[wave][x] = m_run;
            s_l[wave][x] = l_run;
        }
    }
    __syncthreads();
#pragma unroll 4
    for (int idx = tid; idx < Gq * D; idx += kWaves * 64) {
        const int hh = idx >> 7, d = idx & (D - 1);
        float M = s_m[0][hh];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) M = fmaxf(M, s_m[w][hh]);
        float num = 0.0f, den = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const float e = s_m[w][hh] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(s_m[w][hh] - M);
            num += e * s_acc[((size_t)w * Gq + hh) * kGqaHeadPitch + 33 * (d >> 5) + (d & 31)];
            den += e * s_l[w][hh];
        }
        const int64_t head = (int64_t)b * H + (int64_t)kvh * Gq + hh;
        if (part == nullptr) {
            out[head * D + d] = __float2half_rn(den > 0.0f ? num / den : 0.0f);
        } else {                          // partials in natural-log units, as the merge kernel reads them
            float *dst = part + (head * gridDim.y + blockIdx.y) * (D + 2);
            dst[2 + d] = num;
            if (d == 0) {
                dst[0] = M * 0.69314718055994530942f;
                dst[1] = den;
            }
        }
    }
}

// Second pass of a split launch: the partials of one (sequence, head) merge as the
// wavefronts did, out = sum_s e^(M_s - M) num_s / sum_s e^(M_s - M) den_s.  At most 64 splits:
// lane s of the first wavefront takes split s, so the maxima are one load per lane and the
// weights e^(M_s - M) are computed once; then thread d sums its column over the splits with
// independent loads (a loop that waits for each split's maximum in turn costs the memory
// latency 2 S times).
__global__ __launch_bounds__(128)
void decode_attention_merge_kernel(const float *__restrict__ part, int S, __half *__restrict__ out)
{
    constexpr int D = 128;
    __shared__ float s_e[64];
    __shared__ float s_den;
    const float *src = part + (int64_t)blockIdx.x * S * (D + 2);
    const int tid = threadIdx.x;
    // the first splits' values leave before the weights are known: a load behind the barrier costs a latency of its own (attention and
    // merge, 128 cache heads in 4 splits 23.0 -> 22.7 us, 512 heads in 2 15.3 -> 14.8, 32 heads in 40 23.2 -> 22.2)
    constexpr int AHEAD = 8;
    float ahead[AHEAD];
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) ahead[s] = src[(s < S ? s : S - 1) * (D + 2) + 2 + tid];
    if (tid < 64) {
        const float ms = tid < S ? src[tid * (D + 2)] : -INFINITY;
        const float dn = tid < S ? src[tid * (D + 2) + 1] : 0.0f;
        float M = row16_max(ms);
        M = fmaxf(M, __shfl_xor(M, 16, 64));
        M = fmaxf(M, __shfl_xor(M, 32, 64));
        const float e = ms == -INFINITY ? 0.0f : __expf(ms - M);
        float den = row16_sum(e * dn);
        den += __shfl_xor(den, 16, 64);
        den += __shfl_xor(den, 32, 64);
        s_e[tid] = e;
        if (tid == 0) s_den = den;
    }
    __syncthreads();
    float num = 0.0f;
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) num = s < S ? fmaf(s_e[s], ahead[s], num) : num;
#pragma unroll 8
    for (int s = AHEAD; s < S; ++s) num = fmaf(s_e[s], src[s * (D + 2) + 2 + tid], num);
    const float den = s_den;
    out[(int64_t)blockIdx.x * D + tid] = __float2half_rn(den > 0.0f ? num / den : 0.0f);
}

}  // namespace

namespace atom_internal {

// Shape of the launch.  B * H workgroups of four wavefronts fill the GPU from about five per
// compute unit; a grid of at most 384 workgroups first gets 16 wavefronts per workgroup (the token range is
// shared inside the workgroup, which merges through LDS: no second kernel), and below 256
// workgroups the token range is also split over several workgroups whose partials meet in
// decode_attention_merge_kernel.  Never less than one 64-token group per wavefront and split.
//
// With 2 to 16 query heads per cache head the grouped-query kernel runs instead: one workgroup of
// four wavefronts per (sequence, cache head), the token range split until about 512 workgroups
// exist.
struct AttentionShape { int waves, splits; bool gqa; };
AttentionShape decode_attention_shape(int B, int H, int Hkv, int64_t Tmax)
{
    const int64_t groups = (Tmax + kTokens - 1) / kTokens;
    const int     Gq     = H / Hkv;
    if (Gq >= 2 && Gq <= kGqaMaxHeads) {
        const int64_t bk = (int64_t)B * Hkv;
        // about 512 workgroups, two per compute unit where three fit.  No target is the best one everywhere (64 heads on 8,
        // lengths from T / 4 to T, attention and merge, us, targets of 256, 512, 768, 1024, 1536): 16 x 4096 tokens 23.9, 22.5, 24.5,
        // 24.5, 24.6; 16 x 16384 67.8, 58.3, 58.2, 57.5, 58.6; 32 x 4096 36.0, 34.4, 33.6, 35.2, 36.1; 32 x 2048 21.2, 22.7, 23.1,
        // 24.9, 24.9; 1 x 16384 12.8, 14.9 from 512 on; and from 257 cache heads on, not split, 48 x 4096 49.2, 49.3, 43.6, 43.2, 44.0
        int64_t want = 512 / bk, cap = groups / kGqaWaves;    // no split from 257 workgroups on
        if (want > cap) want = cap;
        if (want > 64) want = 64;
        if (want < 1) want = 1;
        // every split a whole number of rounds of the four wavefronts
        const int64_t per = ((groups + want - 1) / want + kGqaWaves - 1) / kGqaWaves * kGqaWaves;
        return {kGqaWaves, (int)((groups + per - 1) / per), true};
    }
    const int64_t bh     = (int64_t)B * H;
    if (bh > 384 || groups < 16) {
        int64_t want = (1280 + bh - 1) / bh, cap = groups / 4;
        if (want > cap) want = cap;
        if (want > 64) want = 64;
        return {4, want < 1 ? 1 : (int)want, false};
    }
    // 256 x 16 wavefronts = four per SIMD: a round.  Of several sequences the shorter ones leave their last workgroups empty, and one more split than fits is
    // the better side (40 heads, T / 4 to T: 2 x 16000 tokens 30.1 us in four, 33.9 in three; 3 x 8000 26.3 in three, 28.9 in two); a lone
    // sequence has no shorter ones (1 x 40 heads in seven and six: 8192 tokens 25.7, 18.9, 16000 38.8, 26.1).
    // With more than three quarters of a round of heads the second of two splits is mostly a round of its own: its start costs more than it shares out, but the
    // longer the tokens of a workgroup, the less, and a batch of one long and otherwise short sequences waits for the long one alone.  Two splits over one, with all sequences
    // equally long / T / 4 to T (mean of eight orders) / one of T and the others T / 16: 7 x 32 heads: 4096 tokens 1.27 / 1.16 / 0.90, 6144 1.24 / 1.10 / 0.85,
    // 8192 1.24 / 1.08 / 0.76, 12000 1.19 / 1.02 / 0.73, 16000 1.10 / 0.94 / 0.66; 6 x 40: 6144 1.25 / 1.16 / 0.85, 12000 1.17 / 1.08 / 0.75, 16000 1.13 / 1.10 /
    // 0.72; 51 x 5: 8192 1.23 / 1.15 / 0.78, 12000 1.17 / 1.14 / 0.75, 16000 1.13 / 1.09 / 0.73; 5 x 40: 4096 1.30 / 1.11 / 0.75, 6144 1.29 / 1.03 / 0.84, 8192
    // 1.24 / 0.99 / 0.78, 12000 1.20 / 0.92 / 0.68.  The line is where the three cancel: 96 groups at 200 heads, 136 at 224, 162 at 240, 187 at
    // 255.  Up to 2048 tokens the splits, and with them the order of the sums, are what they were (7 x 32 heads, 2048: 22.7, in one 17.4).
    int64_t want = (256 + bh - 1) / bh, cap = groups / 16;
    if (groups > 32 && (B == 1 || (bh > 192 && 3 * groups <= 5 * bh - 712))) want = bh <= 256 ? 256 / bh : 1;
    if (want > cap) want = cap;
    if (want > 64) want = 64;
    return {16, want < 1 ? 1 : (int)want, false};
}

size_t decode_attention_workspace_bytes(int B, int H, int Hkv, int64_t Tmax)
{
    const int S = decode_attention_shape(B, H, Hkv, Tmax).splits;
    return S > 1 ? (size_t)B * H * S * (128 + 2) * sizeof(float) : 0;
}

// A cache that the last-level cache (256 MB) does not keep until the next step is read with the hint that nothing reads it
// again: the memory then delivers 7.1 instead of 6.3 TB/s (a plain read of 400 MB and more).  Append and attention, lengths from T / 4 to
// T, us, without and with the hint; in MB the codes of all Tmax rows: 32 heads, 64 x 2048 (537 MB) 77.8, 68.7; 128 x 2048 139.2,
// 130.0; 90 x 1024 (377) 56.6, 54.1; 60 x 1024 (252) 42.1, 40.3; 40 x 1024 (168) 32.7, 31.9; 28 x 1024 (117) 28.6, 28.5;
// 20 x 1024 (84) 23.1, 23.3; 40 heads, 8 x 10000 (410) 64.1, 60.6; 85 x 161 (70) 24.7, 25.3; 64 heads on 8, 128 x 2048 (268) 56.3, 54.2.
// The line goes by capacity: how full the cache is, only the device knows.  Little filled (attention alone, 128 x 2048, 32 heads, 100 to 300
// tokens, 105 MB): with four such caches in turn, as layers of a model, 34.8, 33.8; one and the same cache again and again, out of the
// last-level cache, 32.2, 33.1.
// Query heads that share a cache head outside the grouped-query kernel (more than 16 of them) read the same rows one after the other: no
// hint (64 heads on 2, 64 x 8192: 435, with the hint 513; 32 on 1, 128 x 8192 373, 426).
static bool attention_reads_once(int B, int H, int Hkv, int64_t Tmax, bool gqa)
{
    return (gqa || H == Hkv) && (int64_t)B * Hkv * Tmax * 128 >= (int64_t)1 << 27;
}

// The same for a call's sizes, as its test asks it.
extern "C" int atom_internal_attention_reads_once(int32_t B, int32_t H, int32_t Hkv, int64_t Tmax)
{
    return attention_reads_once(B, H, Hkv, Tmax, decode_attention_shape(B, H, Hkv, Tmax).gqa);
}

hipError_t launch_decode_attention_kv4(const void *q, int B, int H, int Hkv, int64_t Tmax,
                                       const int32_t *seq_len, const void *kq, const void *ks,
                                       const void *kz, const void *vq, const void *vs,
                                       const void *vz, float sm_scale, void *out, void *workspace,
                                       hipStream_t stream)
{
    const AttentionShape sh = decode_attention_shape(B, H, Hkv, Tmax);
    const int S      = sh.splits;
    const int groups = (int)((Tmax + kTokens - 1) / kTokens);
    int tps = S > 1 ? (groups + S - 1) / S : (groups > 0 ? groups : 1);
    if (sh.gqa) tps = (tps + kGqaWaves - 1) / kGqaWaves * kGqaWaves;   // whole rounds of the wavefronts
    float *part = S > 1 ? (float *)workspace : nullptr;
    const bool once = attention_reads_once(B, H, Hkv, Tmax, sh.gqa);
    if (sh.gqa) {
        const size_t lds = (size_t)kGqaWaves * (H / Hkv) * kGqaHeadPitch * sizeof(float);   // <= 34 KB
        auto kern = once ? &decode_attention_kv4_gqa_kernel<true> : &decode_attention_kv4_gqa_kernel<false>;
        hipLaunchKernelGGL(kern, dim3((unsigned)(B * Hkv), (unsigned)S),
                           dim3(kGqaWaves * 64), lds, stream, (const __half *)q, H, Hkv, Tmax, seq_len,
                           (const uint8_t *)kq, (const __half *)ks, (const int16_t *)kz, (const uint8_t *)vq,
                           (const __half *)vs, (const int16_t *)vz, sm_scale, (__half *)out, tps, part);
    } else {
        auto kern = sh.waves == 4 ? (once ? &decode_attention_kv4_kernel<4, true> : &decode_attention_kv4_kernel<4, false>)
                                  : (once ? &decode_attention_kv4_kernel<16, true> : &decode_attention_kv4_kernel<16, false>);
        hipLaunchKernelGGL(kern, dim3((unsigned)(B * H), (unsigned)S), dim3((unsigned)(64 * sh.waves)),
                           0, stream, (const __half *)q, H, Hkv, Tmax, seq_len, (const uint8_t *)kq,
                           (const __half *)ks, (const int16_t *)kz, (const uint8_t *)vq,
                           (const __half *)vs, (const int16_t *)vz, sm_scale, (__half *)out, tps, part);
    }
    hipError_t err = hipGetLastError();
    if (err != hipSuccess || S == 1) return err;
    hipLaunchKernelGGL(decode_attention_merge_kernel, dim3((unsigned)(B * H)), dim3(128), 0, stream,
                       (const float *)part, S, (__half *)out);
    return hipGetLastError();
}

// Scratch for callers that cannot allocate: one array per GPU, in the library's own device
// image, held until the process ends.  Host code never passes the array's name to a kernel (there
// it is only a handle for the symbol): the device address is looked up once per device with that
// device current, and only that pointer is used afterwards.
namespace {
constexpr size_t kStaticScratchBytes = (size_t)4 << 20;
__device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
std::atomic<void *> scratch_ptr[kMaxDevices];
}  // namespace

size_t static_scratch_bytes() { return kStaticScratchBytes; }

hipError_t static_scratch(void **ptr)
{
    int dev = -1;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return err;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    void *p = scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        err = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (err != hipSuccess) return err;
        if (!p) return hipErrorInvalidSymbol;
        scratch_ptr[dev].store(p, std::memory_order_release);
    }
    *ptr = p;
    return hipSuccess;
}

}  // namespace atom_internal
