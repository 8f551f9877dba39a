// Definitions shared by the FP6 group-GEMM kernels (atom_gemm_f6.hip, atom_gemm_f6_thin.hip, atom_gemm_f6_walk.hip): the unit
// images of the packed operands, the kernel parameters, the matrix instructions and the order control.
#ifndef ATOM_GEMM_F6_H
#define ATOM_GEMM_F6_H

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "atom_gemm_common.h"

namespace atom_gemm_f6 {

using namespace atom_gemm;

typedef int      v8i  __attribute__((ext_vector_type(8)));
typedef int      v12i __attribute__((ext_vector_type(12)));
typedef unsigned v6u  __attribute__((ext_vector_type(6)));
typedef unsigned v2u  __attribute__((ext_vector_type(2)));
typedef unsigned v4u  __attribute__((ext_vector_type(4)));
typedef float    v16f __attribute__((ext_vector_type(16)));
typedef _Float16 v32h __attribute__((ext_vector_type(32)));
typedef _Float16 v4h  __attribute__((ext_vector_type(4)));
typedef float    v2f  __attribute__((ext_vector_type(2)));
typedef _Float16 v2h  __attribute__((ext_vector_type(2)));

constexpr int IMG4 = 6656;                // bytes of an INT4 group image of one unit
constexpr int IMG8 = 8704;                // bytes of an INT8 group image of one unit
constexpr int kU8  = 9216;                // pitch of the INT8 images in LDS where they are fetched during the K loop
constexpr int SC4  = 6144;                // offset of the scales inside an INT4 image
constexpr int SC8  = 8192;

__host__ __device__ constexpr int round_kb(int x) { return (x + 1023) / 1024 * 1024; }

struct F6Params {
    const uint8_t *a_pk, *w_pk;           // unit images of the activations / weights
    uint16_t *y; int32_t *partials;
    int64_t M, N, ldy;
    int     a_units, w_units, G4, G8;
    int64_t ustride;
};

// s_waitcnt immediate: vmcnt(n), lgkmcnt(0), expcnt untouched
__host__ __device__ constexpr int wait_imm(int n) { return (n & 15) | (7 << 4) | (0 << 8) | ((n >> 4) << 14); }

// A lane's operands of the two MFMAs of a group, as the three 128-bit fragment reads deliver them:
// registers 0-5 feed the first MFMA (channels 0-63 of the group), registers 6-11 the second.
template <int S>
__device__ __forceinline__ v16f mfma_f6(const v12i &a, const v12i &b, v16f c)
{
    // cbsz = blgp = 3: both operands E3M2 (six registers each); no scales: the form of the instruction without them
    const v8i a8 = __builtin_shufflevector(a, a, 6 * S, 6 * S + 1, 6 * S + 2, 6 * S + 3, 6 * S + 4, 6 * S + 5, -1, -1);
    const v8i b8 = __builtin_shufflevector(b, b, 6 * S, 6 * S + 1, 6 * S + 2, 6 * S + 3, 6 * S + 4, 6 * S + 5, -1, -1);
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a8, b8, c, 3, 3, 0, 0, 0, 0);
}

// Order control.  MFMAs and fused multiply-adds have no side effects, so instruction selection
// is free to let them drift towards their consumers, which bunches each MFMA with the
// multiply-adds that wait for it.  An empty volatile asm that takes a value as an in/out operand
// is ordered with the other volatile statements and with the scheduling fences: whatever produces
// the value stays above it, whatever consumes it stays below.
#define ATOM_F6_PIN(x) asm volatile("" : "+v"(x))
#define ATOM_F6_SLOT_END()                         \
    do {                                           \
        asm volatile("" ::: "memory");             \
        __builtin_amdgcn_sched_barrier(0);         \
    } while (0)

// One LDS-DMA request: every active lane moves 16 bytes from base + voff into LDS, lane l to lds + 16 l.
__device__ __forceinline__ void dma16(uint32_t lds, uint32_t voff, const uint8_t *base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(__builtin_amdgcn_readfirstlane((int)lds)), "v"(voff), "s"(base) : "memory", "m0");
}

// The same for the lanes of a (uniform) mask only; every lane of the wavefront is active around it.
__device__ __forceinline__ void dma16_masked(uint32_t lds, uint32_t voff, const uint8_t *base, uint64_t mask)
{
    const uint64_t m = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(mask >> 32)) << 32 |
                       (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)mask);
    asm volatile("s_mov_b32 m0, %0\n\ts_mov_b64 exec, %3\n\tglobal_load_lds_dwordx4 %1, %2\n\ts_mov_b64 exec, -1"
                 :: "s"(__builtin_amdgcn_readfirstlane((int)lds)), "v"(voff), "s"(base), "s"(m) : "memory", "m0");
}

// The kernels for one INT8 group and at least seven INT4 groups, with at least a tile's units of either operand:
// few tiles (atom_gemm_f6_thin.hip; tile 0: 64 x 64, 1: 64 x 128, 2: 128 x 128) and many (atom_gemm_f6_walk.hip; tile 0:
// 128 x 128, 1: 256 x 128, 2: 256 x 192, 3: 128 x 384, 4: 256 x 256, 5: 192 x 128).
hipError_t launch_thin(const F6Params &p, int tile, hipStream_t stream);
hipError_t launch_walk(const F6Params &p, int tile, hipStream_t stream);

}  // namespace atom_gemm_f6
#endif
