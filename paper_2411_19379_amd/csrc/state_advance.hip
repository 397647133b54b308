// Roll-forward of cached states (Section 4.1: a kernel that rolls a checkpointed state forward by a few tokens to
// reach an exact position; with one token per sequence it is the decode step).  Every sequence of the batch brings
// its own [H,P,N] state (fp32, or fp16 / bf16 as a cache stores it), which is advanced IN PLACE by the sequence's
// tokens with the token recurrence itself,
//
//     a = exp(dt A),   S[p,n] = a S[p,n] + (dt x[p]) B[n],   y[p] = sum_n C[n] S[p,n] + D x[p],
//
// in fp32 on the vector ALUs: for a handful of tokens the work is reading and writing the state once (2 x 4 MiB per
// sequence at H=128, P=64, N=128), i.e. HBM-bound streaming, and the chunked machinery of the scan buys nothing.
//
// One workgroup of 256 threads owns (sequence, head, slice of state rows).  A state row of N floats is spread over
// N/4 neighbouring lanes (16 bytes each, so every state access is a contiguous run of 16-byte pieces); a thread keeps
// up to 8 rows in registers across the sequence's tokens.  y needs the sum over a row: a DPP prefix sum inside the
// lane group, taken from the group's last lane.
#include "device_utils.h"

namespace {

constexpr int kAdvThreads = 256;
constexpr int kAdvMaxRows = 8;  // state rows per thread
// A longer sequence is rolled forward by the matrix-core kernels of scan_valu.hip (fp32 as here): the token loop is one
// chain of dependent loads and sums, 1 to 2 us a token.  Three sequences of 17 to 256 tokens at 128 heads: 466 -> 37 us.
// The sequence's own length decides and nothing else of the batch, so that its bits do not depend on its neighbours; a
// batch with both kinds takes two launches (workgroups of the other kind's sequences leave this kernel's at once).
// Where the line lies, token recurrence against matrix cores, us per call (heads x 64 channels, d_state 128):
//   bf16, 128 heads, fp32 states   1 sequence 4 tokens 12 / 7    8 x 5 tokens 22 / 23    64 x 5 137 / 159   64 x 8 185 / 165
//   bf16, 80 heads, fp16 states    1 x 4  12 / 6                 8 x 5  18 / 14          64 x 4 63 / 72     64 x 5  73 / 72
//   fp32, 80 heads                 1 x 5  14 / 9    8 x 5  18 / 21   8 x 7  21 / 21      64 x 5 79 / 105    64 x 8 102 / 107
// With smaller states the matrix cores win from 2 to 5 tokens on at any number of sequences.
constexpr int kAdvMaxTokens = 4;
constexpr int kAdvMaxTokensF32Wide = 7;  // fp32 storage and d_state 128: the fp32 instruction is the slowest
inline int advance_max_tokens(const ssm_shape_t &s)
{
    return s.io_dtype == SSM_DT_F32 && s.d_state >= 128 ? kAdvMaxTokensF32Wide : kAdvMaxTokens;
}
// States of more than this per call pass by the caches (non-temporal loads and stores): in a serving program every layer's
// states come by between two steps, so what a call leaves in the 256 MiB memory-side cache is gone before it is read again
// and only displaces.  The price is paid by a program whose states do stay there, one that advances few layers in turn.
// One token per sequence at 128 heads x 64 x 128, us per call through the caches / past them:
//                    132 MiB   192 MiB   256 MiB   320 MiB of states
//   fp32   other    59 / 49   84 / 72  106 / 94  136 / 119     (other: each call advances other ones of 1 GiB of buffers)
//          same     45 / 48   63 / 71   83 / 93  118 / 118     (same: the same buffers in every call)
//   bf16   other    85 / 72  117 / 108 155 / 144 197 / 181
//          same     66 / 73   90 / 107 142 / 144 192 / 181
//   fp16   other    79 / 73  114 / 107 148 / 142 188 / 178
//          same     58 / 73   80 / 106 129 / 142 187 / 177
// In fp32 and bf16 the limit is where a second call's states no longer fit the cache beside the first's.  In fp16 the gain
// is small and the price high, so there it lies where not even the same states stay cached.
constexpr long long kAdvStreamBytes = 128ll << 20, kAdvStreamBytesF16 = 272ll << 20;
constexpr float kAdvLog2e = 1.4426950408889634f;

#define ADV_DPP(v, ctrl, row_mask)                                                                            \
    __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, (float)(v)), (ctrl),     \
                                                          (row_mask), 0xF, true))

// Sum over each group of LPR neighbouring lanes (LPR a power of two, groups aligned); valid in the last lane of a group.
template <int LPR>
__device__ __forceinline__ float group_sum_in_last_lane(float v)
{
    if (LPR >= 2)
        v += ADV_DPP(v, 0x111, 0xF);  // row_shr:1
    if (LPR >= 4)
        v += ADV_DPP(v, 0x112, 0xF);  // row_shr:2
    if (LPR >= 8)
        v += ADV_DPP(v, 0x114, 0xF);  // row_shr:4
    if (LPR >= 16)
        v += ADV_DPP(v, 0x118, 0xF);  // row_shr:8
    if (LPR >= 32)
        v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x142, 0xA, 0xF,
                                                                   false));  // row_bcast:15 into rows 1 and 3
    if (LPR >= 64)
        v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x143, 0xC, 0xF,
                                                                   false));  // row_bcast:31 into rows 2 and 3
    return v;
}

template <typename IO> struct Vec4;
template <> struct Vec4<float> {
    static __device__ __forceinline__ float4 load(const float *p) { return *reinterpret_cast<const float4 *>(p); }
};
template <> struct Vec4<bf16_t> {
    static __device__ __forceinline__ float4 load(const bf16_t *p)
    {
        const uint2 u = *reinterpret_cast<const uint2 *>(p);
        return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                           __uint_as_float(u.y & 0xffff0000u));
    }
};

// Storage type of the cached states: fp32, or fp16 / bf16 as a cache keeps them (Section 5.1: FP16 everywhere;
// Appendix A.1: 2 bytes per state element), which halves the bytes this kernel moves.  Arithmetic stays fp32; a
// reduced-precision state is rounded once, to nearest even, when it is written back.
enum { ADV_STATE_F32 = SSM_ST_F32, ADV_STATE_F16 = SSM_ST_F16, ADV_STATE_BF16 = SSM_ST_BF16 };
// NT: loads and stores that keep nothing in the caches (see kAdvStreamBytes).
typedef float adv_f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t adv_u32x2 __attribute__((ext_vector_type(2)));
template <bool NT, typename V> __device__ __forceinline__ V adv_load(const void *p)
{
    if constexpr (NT)
        return __builtin_nontemporal_load(static_cast<const V *>(p));
    return *static_cast<const V *>(p);
}
template <bool NT, typename V> __device__ __forceinline__ void adv_store(void *p, V v)
{
    if constexpr (NT)
        __builtin_nontemporal_store(v, static_cast<V *>(p));
    else
        *static_cast<V *>(p) = v;
}
template <int ST> struct StateVec;
template <> struct StateVec<ADV_STATE_F32> {
    typedef float elem;
    template <bool NT> static __device__ __forceinline__ float4 load(const elem *p)
    {
        const adv_f32x4 v = adv_load<NT, adv_f32x4>(p);
        return make_float4(v[0], v[1], v[2], v[3]);
    }
    template <bool NT> static __device__ __forceinline__ void store(elem *p, float4 v)
    {
        const adv_f32x4 u = {v.x, v.y, v.z, v.w};
        adv_store<NT>(p, u);
    }
};
template <> struct StateVec<ADV_STATE_F16> {
    typedef _Float16 elem;
    typedef __attribute__((ext_vector_type(4))) _Float16 h4;
    template <bool NT> static __device__ __forceinline__ float4 load(const elem *p)
    {
        const h4 h = __builtin_bit_cast(h4, adv_load<NT, adv_u32x2>(p));
        return make_float4((float)h[0], (float)h[1], (float)h[2], (float)h[3]);
    }
    template <bool NT> static __device__ __forceinline__ void store(elem *p, float4 v)
    {
        const h4 h = {(_Float16)v.x, (_Float16)v.y, (_Float16)v.z, (_Float16)v.w};
        adv_store<NT>(p, __builtin_bit_cast(adv_u32x2, h));
    }
};
template <> struct StateVec<ADV_STATE_BF16> {
    typedef bf16_t elem;
    template <bool NT> static __device__ __forceinline__ float4 load(const elem *p)
    {
        const adv_u32x2 u = adv_load<NT, adv_u32x2>(p);
        return make_float4(__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xffff0000u), __uint_as_float(u[1] << 16),
                           __uint_as_float(u[1] & 0xffff0000u));
    }
    template <bool NT> static __device__ __forceinline__ void store(elem *p, float4 v)
    {
        const adv_u32x2 u = {(uint32_t)f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16),
                             (uint32_t)f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16)};
        adv_store<NT>(p, u);
    }
};

struct AdvanceArgs {
    const void *x, *dt, *B, *C;
    const float *A, *D;
    void *y;                   // may be null
    StatePtrs states;          // [batch] device pointers, each [H,P,N] in the state type; null = leave the sequence alone
    const SsmTile *tiles;
    const SsmSeq *seqs;
    int H, P, N, G;
    int rows_per_thread;       // 1..kAdvMaxRows
    int slices;                // workgroups per (sequence, head)
    int most_tokens;           // longer sequences belong to another launch (Mixed); 0: there are none
    bool stream;               // the states pass by the caches
};

// Mixed: the batch also has sequences that another launch advances (a look at the tile table that a decode step does without).
template <typename IO, int LPR, int ST, bool NT, bool Mixed>
__global__ __launch_bounds__(kAdvThreads) void ssm_advance_kernel(AdvanceArgs a)
{
    typedef typename StateVec<ST>::elem state_t;
    constexpr int kRowsPerPass = kAdvThreads / LPR;
    const int H = a.H, P = a.P, N = a.N, G = a.G;
    const int slice = blockIdx.x % a.slices;
    const int h = (blockIdx.x / a.slices) % H;
    const int seq = blockIdx.x / (a.slices * H);
    const int g = h / (H / G);
    const int c = threadIdx.x % LPR;   // this thread holds state columns 4c .. 4c+3
    const int rs = threadIdx.x / LPR;  // row slot inside a pass
    const int R = a.rows_per_thread;
    const int p_first = slice * kRowsPerPass * R + rs;  // rows p_first + kRowsPerPass * r

    state_t *state = static_cast<state_t *>(const_cast<void *>(a.states.of(seq)));
    const SsmSeq sq = a.seqs[seq];
    if (sq.tile_end <= sq.tile_begin || state == nullptr)
        return;  // nothing to advance; the whole workgroup leaves
    if constexpr (Mixed) {
        const SsmTile last = a.tiles[sq.tile_end - 1];
        if (last.tok0 + last.len - a.tiles[sq.tile_begin].tok0 > a.most_tokens)
            return;
    }

    const IO *x = static_cast<const IO *>(a.x);
    const IO *dt = static_cast<const IO *>(a.dt);
    const IO *Bg = static_cast<const IO *>(a.B);
    const IO *Cg = static_cast<const IO *>(a.C);
    IO *y = static_cast<IO *>(a.y);
    const float Ah = a.A[h] * kAdvLog2e;
    const float Dh = a.D[h];

    float4 S[kAdvMaxRows];
#pragma unroll
    for (int r = 0; r < kAdvMaxRows; ++r) {
        const int p = p_first + kRowsPerPass * r;
        S[r] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (r < R && p < P)
            S[r] = StateVec<ST>::template load<NT>(state + ((size_t)h * P + p) * N + 4 * c);
    }

    for (int ti = sq.tile_begin; ti < sq.tile_end; ++ti) {
        const SsmTile t = a.tiles[ti];
        for (int i = 0; i < t.len; ++i) {
            const size_t tok = (size_t)t.tok0 + i;
            const float dtv = IoTraits<IO>::load(dt + tok * H + h);
            const float decay = __builtin_amdgcn_exp2f(dtv * Ah);
            const float4 b4 = Vec4<IO>::load(Bg + (tok * G + g) * N + 4 * c);
            const float4 c4 = Vec4<IO>::load(Cg + (tok * G + g) * N + 4 * c);
#pragma unroll
            for (int r = 0; r < kAdvMaxRows; ++r) {
                const int p = p_first + kRowsPerPass * r;
                // the row guard is uniform over a lane group, and groups never straddle DPP rows they do not own
                const bool live = r < R && p < P;
                const float xv = live ? IoTraits<IO>::load(x + (tok * H + h) * P + p) : 0.f;
                const float dx = dtv * xv;
                S[r].x = decay * S[r].x + dx * b4.x;
                S[r].y = decay * S[r].y + dx * b4.y;
                S[r].z = decay * S[r].z + dx * b4.z;
                S[r].w = decay * S[r].w + dx * b4.w;
                if (y != nullptr && r < R) {  // uniform over the wave: every lane takes part in the DPP steps
                    const float part = c4.x * S[r].x + c4.y * S[r].y + c4.z * S[r].z + c4.w * S[r].w;
                    const float row = group_sum_in_last_lane<LPR>(part);
                    if (live && c == LPR - 1)
                        IoTraits<IO>::store(y + (tok * H + h) * P + p, row + Dh * xv);
                }
            }
        }
    }

#pragma unroll
    for (int r = 0; r < kAdvMaxRows; ++r) {
        const int p = p_first + kRowsPerPass * r;
        if (r < R && p < P)
            StateVec<ST>::template store<NT>(state + ((size_t)h * P + p) * N + 4 * c, S[r]);
    }
}

template <typename IO, int LPR, int ST, bool NT>
void launch_nt(const AdvanceArgs &a, dim3 grid, hipStream_t stream)
{
    if (a.most_tokens > 0)
        hipLaunchKernelGGL((ssm_advance_kernel<IO, LPR, ST, NT, true>), grid, dim3(kAdvThreads), 0, stream, a);
    else
        hipLaunchKernelGGL((ssm_advance_kernel<IO, LPR, ST, NT, false>), grid, dim3(kAdvThreads), 0, stream, a);
}

template <typename IO, int LPR, int ST>
void launch_st(const AdvanceArgs &a, dim3 grid, hipStream_t stream)
{
    if (a.stream)
        launch_nt<IO, LPR, ST, true>(a, grid, stream);
    else
        launch_nt<IO, LPR, ST, false>(a, grid, stream);
}

template <typename IO, int LPR>
void launch_lpr(const AdvanceArgs &a, int batch, int state_type, hipStream_t stream)
{
    const dim3 grid((unsigned)(batch * a.H * a.slices));
    switch (state_type) {
    case ADV_STATE_F16: launch_st<IO, LPR, ADV_STATE_F16>(a, grid, stream); break;
    case ADV_STATE_BF16: launch_st<IO, LPR, ADV_STATE_BF16>(a, grid, stream); break;
    default: launch_st<IO, LPR, ADV_STATE_F32>(a, grid, stream); break;
    }
}

template <typename IO>
hipError_t launch_io(AdvanceArgs &a, int batch, int state_type, hipStream_t stream)
{
    const int lpr = a.N / 4;
    const int rows_per_pass = kAdvThreads / lpr;
    int R = (a.P + rows_per_pass - 1) / rows_per_pass;
    if (R > kAdvMaxRows)
        R = kAdvMaxRows;
    a.rows_per_thread = R;
    a.slices = (a.P + rows_per_pass * R - 1) / (rows_per_pass * R);
    switch (lpr) {
    case 1: launch_lpr<IO, 1>(a, batch, state_type, stream); break;
    case 2: launch_lpr<IO, 2>(a, batch, state_type, stream); break;
    case 4: launch_lpr<IO, 4>(a, batch, state_type, stream); break;
    case 8: launch_lpr<IO, 8>(a, batch, state_type, stream); break;
    case 16: launch_lpr<IO, 16>(a, batch, state_type, stream); break;
    case 32: launch_lpr<IO, 32>(a, batch, state_type, stream); break;
    case 64: launch_lpr<IO, 64>(a, batch, state_type, stream); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

// True if the roll-forward kernel handles this shape: d_state a power of two between 4 and 256.
bool state_advance_supports(const ssm_shape_t &s)
{
    const int n = s.d_state;
    return n >= 4 && n <= 256 && (n & (n - 1)) == 0;
}

// How many sequences of the plan are rolled forward by the matrix-core kernels: the first ones of plan->order.
static int longer_ones(const ssm_plan *plan)
{
    return scan_f32_supports(plan->shape) ? ssm_plan_longer_than(plan, advance_max_tokens(plan->shape)) : 0;
}

// True if a roll-forward of the plan takes both kinds of kernels and so needs the order of its sequences on the GPU.
bool state_advance_mixes(const ssm_plan *plan)
{
    const int n_long = longer_ones(plan);
    return n_long > 0 && n_long < ssm_plan_longer_than(plan, 0);
}

// Advance the state of every sequence of the plan in place by the sequence's tokens; `d_state_ptrs` is a device array
// of plan->batch device pointers to states in the plan's state type (not needed if args.host_ptrs is set).  y may be null.
// args.order is needed where both kinds of kernels are (state_advance_mixes).
// Checkpoints of the plan are ignored (the result is the in-place state after the last token).
hipError_t launch_state_advance(const ssm_plan *plan, const ScanArgs &args, void *const *d_state_ptrs,
                                hipStream_t stream)
{
    const int state_type = args.state_dtype;
    if (!state_advance_supports(plan->shape) || state_type < ADV_STATE_F32 || state_type > ADV_STATE_BF16)
        return hipErrorInvalidValue;
    if (plan->batch == 0 || plan->tiles.empty())
        return hipSuccess;
    const int busy = ssm_plan_longer_than(plan, 0);
    const int n_long = longer_ones(plan);
    if (n_long > 0) {
        ScanArgs roll = args;
        roll.init_ptrs = d_state_ptrs;
        const hipError_t e = launch_scan_f32(plan, roll, true, n_long == busy ? plan->batch : n_long, stream);
        if (e != hipSuccess || n_long == busy)
            return e;
    }
    AdvanceArgs a;
    a.x = args.x;
    a.dt = args.dt;
    a.B = args.B;
    a.C = args.C;
    a.A = args.A;
    a.D = args.D;
    a.y = args.y;
    a.states = state_ptrs_of(d_state_ptrs, args.host_ptrs, args.n_host_ptrs);
    a.tiles = args.tiles;
    a.seqs = args.seqs;
    a.most_tokens = n_long > 0 ? advance_max_tokens(plan->shape) : 0;
    a.H = args.H;
    a.P = args.P;
    a.N = args.N;
    a.G = args.G;
    long long advanced = busy - n_long;
    for (int r = n_long; args.host_ptrs && r < busy; ++r)
        advanced -= args.host_ptrs[plan->order[r]] == nullptr;
    const long long bytes = advanced * a.H * a.P * a.N * (state_type == ADV_STATE_F32 ? 4 : 2);
    a.stream = bytes > (state_type == ADV_STATE_F16 ? kAdvStreamBytesF16 : kAdvStreamBytes);
    return plan->shape.io_dtype == SSM_DT_F32 ? launch_io<float>(a, plan->batch, state_type, stream)
                                              : launch_io<bf16_t>(a, plan->batch, state_type, stream);
}
