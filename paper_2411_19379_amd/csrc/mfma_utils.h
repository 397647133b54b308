// Device helpers of the fp16 / bf16 matrix-core scans (scan_mfma.hip, scan_resident.hip): operand types and products, LDS
// transpose reads, buffer descriptors, wave sums, conversions.
#pragma once

#include "device_utils.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(4))) _Float16 f16x4;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) float f32x2;

constexpr int kQ = kMfmaTileTokens;  // 64 tokens per tile
constexpr int kN = 128;              // d_state
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ s16x4 lds_tr4(const void *p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(p));
}

// 8 k-values of a transposed operand: two groups of 4 consecutive rows of a row-major tile of 16-bit elements.
// The 16 lanes of a group pass the addresses of 4 rows x (4 lanes x 4 elements); lane i of the group receives
// column i of that 4x16 block.
__device__ __forceinline__ uint4 lds_frag_tr(const void *p_lo, const void *p_hi)
{
    const s16x4 lo = lds_tr4(p_lo), hi = lds_tr4(p_hi);
    return __builtin_bit_cast(uint4, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ uint32_t pack2_f16(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
}

__device__ __forceinline__ float f16_lo(uint32_t u) { return (float)__builtin_bit_cast(f16x2, u)[0]; }
__device__ __forceinline__ float f16_hi(uint32_t u) { return (float)__builtin_bit_cast(f16x2, u)[1]; }
__device__ __forceinline__ float bf16_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t u) { return __uint_as_float(u & 0xffff0000u); }

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

// Loads and stores of the tile loop go through buffer descriptors: a wave-uniform base and size in scalar registers,
// one 32-bit byte offset per lane and a uniform offset, so that no address arithmetic runs on the vector ALUs.  The
// loads are issued phases ahead of their use; the scheduling fences at the phase ends keep them where they are
// written.  Every access stays inside its descriptor's range.  The one use of the hardware's range check is a
// descriptor of size zero, through which a wave that has no next tile issues its look-ahead loads: they return
// zeros without touching memory (and their base address is valid memory in any case).
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void *base, uint32_t bytes)
{
    // raw buffer (stride 0) of `bytes` bytes; the flags word selects 32-bit data, as for any untyped access on gfx9
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ uint4 buf_load16(rsrc_t r, uint32_t lane_off, uint32_t uniform_off)
{
    const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane_off, (int)uniform_off, 0);
    return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void buf_store16(rsrc_t r, uint32_t lane_off, uint32_t uniform_off, const uint4 &d)
{
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = {d.x, d.y, d.z, d.w};
    __builtin_amdgcn_raw_buffer_store_b128(v, r, (int)lane_off, (int)uniform_off, 0);
}

#define SSM_DPP(old, v, ctrl, row_mask, bound)                                                        \
    __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, (float)(old)),       \
                                                          __builtin_bit_cast(int, (float)(v)), (ctrl), \
                                                          (row_mask), 0xF, (bound)))
// Inclusive prefix sum over the 64 lanes of a wave with DPP row shifts and the two row broadcasts.
__device__ __forceinline__ float wave_inclusive_sum(float v)
{
    v += SSM_DPP(0.f, v, 0x111, 0xF, true);   // row_shr:1
    v += SSM_DPP(0.f, v, 0x112, 0xF, true);   // row_shr:2
    v += SSM_DPP(0.f, v, 0x114, 0xF, true);   // row_shr:4
    v += SSM_DPP(0.f, v, 0x118, 0xF, true);   // row_shr:8
    v += SSM_DPP(0.f, v, 0x142, 0xA, false);  // row_bcast:15 into rows 1 and 3
    v += SSM_DPP(0.f, v, 0x143, 0xC, false);  // row_bcast:31 into rows 2 and 3
    return v;
}

__device__ __forceinline__ float read_lane(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

__device__ __forceinline__ f32x16 zero16()
{
    const f32x16 z = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    return z;
}

__device__ __forceinline__ f32x16 mfma_bf16(uint4 a, uint4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                   0);
}

__device__ __forceinline__ f32x16 mfma_f16(uint4 a, uint4 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0,
                                                  0);
}

// Four neighbouring elements of a cached state (element index idx) in its storage type.
__device__ __forceinline__ float4 load_state4(const void *base, size_t idx, int state_dtype)
{
    if (state_dtype == SSM_ST_F16) {
        const f16x4 h = *reinterpret_cast<const f16x4 *>(static_cast<const _Float16 *>(base) + idx);
        return make_float4((float)h[0], (float)h[1], (float)h[2], (float)h[3]);
    }
    if (state_dtype == SSM_ST_BF16) {
        const uint2 u = *reinterpret_cast<const uint2 *>(static_cast<const bf16_t *>(base) + idx);
        return make_float4(bf16_lo(u.x), bf16_hi(u.x), bf16_lo(u.y), bf16_hi(u.y));
    }
    return *reinterpret_cast<const float4 *>(static_cast<const float *>(base) + idx);
}

__device__ __forceinline__ void store_state4(void *base, size_t idx, float4 v, int state_dtype)
{
    if (state_dtype == SSM_ST_F16) {
        const f16x4 h = {(_Float16)v.x, (_Float16)v.y, (_Float16)v.z, (_Float16)v.w};
        *reinterpret_cast<f16x4 *>(static_cast<_Float16 *>(base) + idx) = h;
    } else if (state_dtype == SSM_ST_BF16) {
        *reinterpret_cast<uint2 *>(static_cast<bf16_t *>(base) + idx) =
            make_uint2(pack2_bf16(v.x, v.y), pack2_bf16(v.z, v.w));
    } else {
        *reinterpret_cast<float4 *>(static_cast<float *>(base) + idx) = v;
    }
}

// 8 bf16 -> 8 fp16 (exact for values whose exponent fp16 can hold)
__device__ __forceinline__ uint4 bf16x8_to_f16x8(uint4 v)
{
    return make_uint4(pack2_f16(bf16_lo(v.x), bf16_hi(v.x)), pack2_f16(bf16_lo(v.y), bf16_hi(v.y)),
                      pack2_f16(bf16_lo(v.z), bf16_hi(v.z)), pack2_f16(bf16_lo(v.w), bf16_hi(v.w)));
}

// The 16 raw scores of a lane (accumulator image of a 32x32 block of Gm^T, fp16) as floats.
__device__ __forceinline__ void unpack_scores(const uint4 &raw0, const uint4 &raw1, float (&v)[16])
{
    const uint32_t rw[8] = {raw0.x, raw0.y, raw0.z, raw0.w, raw1.x, raw1.y, raw1.z, raw1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        v[2 * e] = f16_lo(rw[e]);
        v[2 * e + 1] = f16_hi(rw[e]);
    }
}

__device__ __forceinline__ void pack_scores(const float (&v)[16], uint4 &g0, uint4 &g1)
{
    g0 = make_uint4(pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]), pack2_bf16(v[4], v[5]), pack2_bf16(v[6], v[7]));
    g1 = make_uint4(pack2_bf16(v[8], v[9]), pack2_bf16(v[10], v[11]), pack2_bf16(v[12], v[13]), pack2_bf16(v[14], v[15]));
}

}  // namespace
