// Small device helpers shared by the scan kernels (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "plan.h"

typedef uint16_t bf16_t;  // raw bfloat16 bits

__device__ __forceinline__ float bf16_to_f32(bf16_t v)
{
    return __uint_as_float((uint32_t)v << 16);
}

// round to nearest even; NaN stays NaN
__device__ __forceinline__ bf16_t f32_to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u)
        return (bf16_t)((u >> 16) | 0x0040u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

template <typename IO> struct IoTraits;
template <> struct IoTraits<float> {
    static __device__ __forceinline__ float load(const float *p) { return *p; }
    static __device__ __forceinline__ void store(float *p, float v) { *p = v; }
};
template <> struct IoTraits<bf16_t> {
    static __device__ __forceinline__ float load(const bf16_t *p) { return bf16_to_f32(*p); }
    static __device__ __forceinline__ void store(bf16_t *p, float v) { *p = f32_to_bf16(v); }
};

// One element of a cached state in its storage type (ssm_state_dtype_t); the running state is always fp32 and a
// reduced-precision checkpoint is that fp32 value rounded once, to nearest even.
__device__ __forceinline__ float state_load(const void *base, size_t idx, int state_dtype)
{
    if (state_dtype == SSM_ST_F16)
        return (float)static_cast<const _Float16 *>(base)[idx];
    if (state_dtype == SSM_ST_BF16)
        return bf16_to_f32(static_cast<const bf16_t *>(base)[idx]);
    return static_cast<const float *>(base)[idx];
}

__device__ __forceinline__ void state_store(void *base, size_t idx, float v, int state_dtype)
{
    if (state_dtype == SSM_ST_F16)
        static_cast<_Float16 *>(base)[idx] = (_Float16)v;
    else if (state_dtype == SSM_ST_BF16)
        static_cast<bf16_t *>(base)[idx] = f32_to_bf16(v);
    else
        static_cast<float *>(base)[idx] = v;
}

// A word or a table entry at a uniform address that no kernel of the call writes: read with scalar loads, which wait for no
// vector memory access in flight.  (In a loop that stores, the compiler reads such entries with vector loads; the tile table
// in the loops of the fp32 and split-operand scans: 141.5 -> 138.2 us for 2048 tokens of 80 heads in fp32, 57.1 -> 55.7 for
// 8 requests with d_state 16.)
template <typename T> __device__ __forceinline__ T scalar_load(const T *p)
{
    static_assert(sizeof(T) % 4 == 0, "whole words");
    typedef const uint32_t __attribute__((address_space(4))) constant_u32;
    const constant_u32 *c = (const constant_u32 *)(uint64_t)p;
    uint32_t w[sizeof(T) / 4];
#pragma unroll
    for (unsigned k = 0; k < sizeof(T) / 4; ++k)
        w[k] = c[k];
    T v;
    __builtin_memcpy(&v, w, sizeof(T));
    return v;
}

// The per-call state pointers of a batch.  Up to kStatePtrsInArgs of them travel in the kernel's own arguments; a larger
// batch reads them from a device array that another launch has filled.  (A launch of its own for a few pointers costs 1
// to 5 us in front of every call; 64 pointers are half a KiB of arguments, which costs nothing measurable.)
constexpr int kStatePtrsInArgs = 64;
struct StatePtrs {
    const void *const *table;         // device array; null: the pointers are in p
    const void *p[kStatePtrsInArgs];  // all null if there are none
    // Read with scalar loads and known to point to device memory: chosen between two addresses, the pointer itself and all
    // that is accessed through it would take FLAT instructions (128 sequences rolled forward by 4 tokens, 128 heads, fp16
    // states: 249 -> 237 us per call).
    __device__ __forceinline__ const void *of(int seq) const
    {
        typedef const uint64_t __attribute__((address_space(1))) global_u64;
        typedef const void __attribute__((address_space(1))) global_void;
        uint64_t u;
        if (table)
            u = ((global_u64 *)(uint64_t)table)[seq];
        else
            u = (uint64_t)p[seq & (kStatePtrsInArgs - 1)];
        return (const void *)(global_void *)u;
    }
};

// Arguments common to the scan kernels.  Pointers are device pointers.
struct ScanArgs {
    const void *x;
    const void *dt;
    const float *A;
    const void *B;
    const void *C;
    const float *D;
    void *y;
    void *state_out;                // [n_ckpt,H,P,N] in the state type
    const void *const *init_ptrs;   // [batch] pointers to [H,P,N] in the state type, or NULL
    const SsmTile *tiles;
    const SsmSeq *seqs;
    const SsmScanSeq *scan_seqs;    // matrix-core scan only
    int32_t H, P, N, G;
    int32_t p_split;
    int32_t state_dtype;            // ssm_state_dtype_t
    const void *const *host_ptrs = nullptr;  // the same pointers as a host array
    int32_t n_host_ptrs = 0;                 // its entries, if at most kStatePtrsInArgs: then the device array is not needed
    const int32_t *order = nullptr;          // [batch] the plan's sequences by decreasing number of tokens
    bool states_overlap = false;             // an initial state shares memory with state_out; asked only for cut sequences
};

inline StatePtrs state_ptrs_of(const void *const *device_table, const void *const *host, int n)
{
    StatePtrs s = {};
    if (host && n > 0)
        for (int i = 0; i < n; ++i)
            s.p[i] = host[i];
    else
        s.table = device_table;
    return s;
}

// Launchers implemented next to their kernels.
hipError_t launch_scan_valu(const ssm_plan *plan, const ScanArgs &args, hipStream_t stream);
// the fp32 matrix-core scan behind it, which is also the roll-forward over more than a few tokens: of all sequences, or
// of the `n_seqs` longest ones
bool scan_f32_supports(const ssm_shape_t &s);
hipError_t launch_scan_f32(const ssm_plan *plan, const ScanArgs &args, bool roll, int n_seqs, hipStream_t stream);
hipError_t launch_scan_mfma(const ssm_plan *plan, const ScanArgs &args, void *workspace, hipStream_t stream);
// `d_pieces`: the plan's table of pieces
hipError_t launch_scan_resident(const ssm_plan *plan, const ScanArgs &args, const SsmPiece *d_pieces, void *workspace,
                                hipStream_t stream);
// events to record after the first and after the second kernel of the matrix-core scan on the calling thread
// (nullptr: none)
hipEvent_t ssm_profile_event(int which);
bool state_advance_supports(const ssm_shape_t &s);
bool state_advance_mixes(const ssm_plan *plan);
hipError_t launch_state_advance(const ssm_plan *plan, const ScanArgs &args, void *const *d_state_ptrs,
                                hipStream_t stream);
bool conv1d_supports(int channels, int K, int io_dtype);
hipError_t launch_conv1d_prefill(const ssm_plan *plan, const SsmTile *d_tiles, const SsmSeq *d_seqs, int channels,
                                 int K, const void *in, const float *w, const float *bias,
                                 const void *const *d_init_ptrs, void *out, void *state_out, int act,
                                 hipStream_t stream, const void *const *host_ptrs = nullptr, int n_host_ptrs = 0, bool states_overlap = false);
