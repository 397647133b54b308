// Causal depthwise convolution in front of the SSM scan, with cached-state resume and state checkpoints (the
// conv_1d state of Appendix A.1, "Memory footprint").  For channel c, kernel width K <= 4 and the sequence-local
// token t:
//
//     out[t,c] = act( bias[c] + sum_{j<K} w[c,j] z[t-K+1+j, c] ),   act = identity or SiLU
//
// where z is the sequence's input, continued to the left by the cached prefix's last inputs (or zeros).  The state
// after p tokens is the last K inputs of every channel, oldest first, in the storage type of the input (a copy of
// inputs, so nothing is lost); a resumed sequence passes such a state back.
//
// The work is streaming: 2 bytes in and 2 bytes out per (token, channel) in bf16.  It uses the tile table of the
// scan's plan, whose tiles never cross a sequence boundary and end at every checkpoint: one workgroup takes one tile
// and a block of channels, a thread walks the tile's tokens for 16 bytes' worth of neighbouring channels with the
// last K inputs in registers, so every access is a contiguous run of 16-byte pieces.  The K-1 tokens in front of a
// tile are read again (from the previous tile's tokens, or from the cached state at the start of a sequence).
//
// Memory bounds it, with the vector units not far behind: 32768 tokens of 10240 channels in bf16 with SiLU, 1.34 GB, take
// 270 us, 5.0 TB/s.  Rounding each output in integer arithmetic instead of by the conversion instruction is 9 us more, and
// requesting a group's rows only when the group before is done another 13 us.
#include "mfma_utils.h"

namespace {

constexpr int kConvThreads = 256;
constexpr int kConvMaxK = 4;
// Rows of a group.  177 VGPRs, two waves per SIMD; 4 rows (133 VGPRs, three) 282 us where 8 take 270 (below), 12 rows 275.
constexpr int kAhead = 8;
constexpr int kConvMostParts = 8;  // tiles have up to 64 tokens
constexpr int kConvWorkgroups = 512;

__device__ __forceinline__ uint4 load16(const void *p) { return *static_cast<const uint4 *>(p); }

template <typename IO> struct ConvVec;
template <> struct ConvVec<float> {
    static constexpr int kLanes = 4;  // channels per thread: 16 bytes
    static __device__ __forceinline__ void unpack(const uint4 &u, float *v)
    {
        v[0] = __uint_as_float(u.x), v[1] = __uint_as_float(u.y), v[2] = __uint_as_float(u.z), v[3] = __uint_as_float(u.w);
    }
    static __device__ __forceinline__ void store(float *p, const float *v)
    {
        *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
    }
};
template <> struct ConvVec<bf16_t> {
    static constexpr int kLanes = 8;
    static __device__ __forceinline__ void unpack(const uint4 &u, float *v)
    {
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[2 * e] = __uint_as_float(w[e] << 16);
            v[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
        }
    }
    static __device__ __forceinline__ void store(bf16_t *p, const float *v)
    {
        *reinterpret_cast<uint4 *>(p) =
            make_uint4(pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]), pack2_bf16(v[4], v[5]), pack2_bf16(v[6], v[7]));
    }
};

struct ConvArgs {
    const void *in;                 // [T,Cch] storage type
    const float *w;                 // [Cch,K]
    const float *bias;              // [Cch] or null
    void *out;                      // [T,Cch] storage type
    StatePtrs init;                 // [batch] device pointers (null = zeros) to [Cch,K] storage type
    void *state_out;                // [n_ckpt,Cch,K] storage type
    const SsmTile *tiles;
    const SsmSeq *seqs;
    int Cch, act, n_tiles, blocks_per_tile;
    int parts;                      // a tile's tokens are dealt to this many workgroups per channel block
};

template <typename IO, int K>
__global__ __launch_bounds__(kConvThreads, 2) void ssm_conv1d_kernel(ConvArgs a)
{
    constexpr int V = ConvVec<IO>::kLanes;
    const int cb = blockIdx.x % a.blocks_per_tile, part_of_all = blockIdx.x / a.blocks_per_tile;
    const int tile = part_of_all / a.parts, part = part_of_all % a.parts;
    const int c0 = (cb * kConvThreads + threadIdx.x) * V;  // first channel of this thread
    const int Cch = a.Cch;
    if (tile >= a.n_tiles || c0 >= Cch)
        return;  // no barriers in this kernel: threads may leave on their own
    SsmTile t = a.tiles[tile];
    const int seq_tok0 = a.tiles[a.seqs[t.seq].tile_begin].tok0;
    if (a.parts > 1) {  // from here on the part is the tile: whole groups, the last part writes the checkpoint
        const int own = (t.len + a.parts * kAhead - 1) / (a.parts * kAhead) * kAhead, skip = part * own;
        if (skip >= t.len)
            return;
        const bool last = t.len - skip <= own;
        t.tok0 += skip;
        t.len = last ? t.len - skip : own;
        t.ckpt_slot = last ? t.ckpt_slot : -1;
    }
    const int lp = t.tok0 - seq_tok0;  // tokens of this sequence in front of the tile

    const IO *__restrict__ in = static_cast<const IO *>(a.in);  // the caller keeps in and out apart
    IO *__restrict__ out = static_cast<IO *>(a.out);
    const IO *init = static_cast<const IO *>(a.init.of(t.seq));

    float wk[K][V], bias[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        bias[e] = a.bias ? a.bias[c0 + e] : 0.f;
#pragma unroll
        for (int j = 0; j < K; ++j)
            wk[j][e] = a.w[(size_t)(c0 + e) * K + j];
    }

    // hist[j] = the input j+1 tokens in front of the current one (j = 0 newest); K entries so that the state,
    // which also holds the input K-1 places back from its last token, can be written from registers
    float hist[K][V];
    // [channel][entry] of the thread's channels: K pieces of 16 bytes (element by element 64 one-token sequences took 24 us
    // where they take 11)
    float state[K * V];
#pragma unroll
    for (int p = 0; p < K; ++p)
        if (init && lp < K)
            ConvVec<IO>::unpack(load16(init + (size_t)c0 * K + p * V), state + p * V);
#pragma unroll
    for (int j = 0; j < K; ++j) {
#pragma unroll
        for (int e = 0; e < V; ++e)
            hist[j][e] = 0.f;
        const int back = j + 1;  // tokens back from the tile's first token
        if (lp - back >= 0) {
            ConvVec<IO>::unpack(load16(in + (size_t)(t.tok0 - back) * Cch + c0), hist[j]);
        } else if (init) {
            // sequence-local index lp - back < 0 is entry K + lp - back of the cached state
#pragma unroll
            for (int m = 0; m < K; ++m)
                if (m == K + lp - back)
#pragma unroll
                    for (int e = 0; e < V; ++e)
                        hist[j][e] = state[e * K + m];
        }
    }

    // Groups of kAhead tokens: while one is worked on, the rows of the next are on their way.
    uint4 row[kAhead], next[kAhead];
    auto request = [&](int i0) {  // past the end: the last row again, unused
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            next[u] = load16(in + ((size_t)t.tok0 + (i0 + u < t.len ? i0 + u : t.len - 1)) * Cch + c0);
    };
    auto token = [&](int i, const uint4 &raw) {
        float cur[V], v[V];
        ConvVec<IO>::unpack(raw, cur);
#pragma unroll
        for (int e = 0; e < V; ++e) {
            float acc = bias[e];
            // oldest first, as the definition is written: w[c,j] meets the input K-1-j places back
#pragma unroll
            for (int j = 0; j < K - 1; ++j)
                acc += wk[j][e] * hist[K - 2 - j][e];
            acc += wk[K - 1][e] * cur[e];
            if (a.act == 1)
                acc = acc * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-1.4426950408889634f * acc));
            v[e] = acc;
        }
        ConvVec<IO>::store(out + ((size_t)t.tok0 + i) * Cch + c0, v);
#pragma unroll
        for (int j = K - 1; j > 0; --j)
#pragma unroll
            for (int e = 0; e < V; ++e)
                hist[j][e] = hist[j - 1][e];
#pragma unroll
        for (int e = 0; e < V; ++e)
            hist[0][e] = cur[e];
    };
    request(0);
    for (int i0 = 0; i0 < t.len; i0 += kAhead) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            row[u] = next[u];
        if (i0 + kAhead < t.len)
            request(i0 + kAhead);
        if (i0 + kAhead <= t.len) {
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                token(i0 + u, row[u]);
        } else {
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                if (i0 + u < t.len)
                    token(i0 + u, row[u]);
        }
    }

    if (t.ckpt_slot >= 0) {
        // the last K inputs, oldest first: hist[K-1] .. hist[0]
        IO *st = static_cast<IO *>(a.state_out) + ((size_t)t.ckpt_slot * Cch + c0) * K;
#pragma unroll
        for (int e = 0; e < V; ++e)
#pragma unroll
            for (int m = 0; m < K; ++m)
                state[e * K + m] = hist[K - 1 - m][e];
#pragma unroll
        for (int p = 0; p < K; ++p)
            ConvVec<IO>::store(st + p * V, state + p * V);
    }
}

}  // namespace

// True if the convolution kernel handles the request: width 1..4 and channel rows that are whole 16-byte pieces.
bool conv1d_supports(int channels, int K, int io_dtype)
{
    const int v = io_dtype == SSM_DT_F32 ? 4 : 8;
    return K >= 1 && K <= kConvMaxK && channels > 0 && channels % v == 0;
}

// Launch over the tiles of `plan` (any shape: only its tile table, sequence table and storage type are used).
// `d_init_ptrs` is null or a device array of plan->batch device pointers; `state_out` may be null if the plan has no
// checkpoints.  `states_overlap`: an initial state shares memory with `state_out`.
hipError_t launch_conv1d_prefill(const ssm_plan *plan, const SsmTile *d_tiles, const SsmSeq *d_seqs, int channels,
                                 int K, const void *in, const float *w, const float *bias,
                                 const void *const *d_init_ptrs, void *out, void *state_out, int act,
                                 hipStream_t stream, const void *const *host_ptrs, int n_host_ptrs, bool states_overlap)
{
    if (!conv1d_supports(channels, K, plan->shape.io_dtype))
        return hipErrorInvalidValue;
    const int n_tiles = (int)plan->tiles.size();
    if (n_tiles == 0)
        return hipSuccess;
    const int v = plan->shape.io_dtype == SSM_DT_F32 ? 4 : 8;
    ConvArgs a;
    a.in = in;
    a.w = w;
    a.bias = bias;
    a.out = out;
    a.init = state_ptrs_of(d_init_ptrs, host_ptrs, n_host_ptrs);
    a.state_out = state_out;
    a.tiles = d_tiles;
    a.seqs = d_seqs;
    a.Cch = channels;
    a.act = act;
    a.n_tiles = n_tiles;
    a.blocks_per_tile = (channels + kConvThreads * v - 1) / (kConvThreads * v);
    // Few tiles leave most of the chip idle, and each is a serial walk: they are cut into parts, of no less than a group of
    // rows for tiles of average length, up to kConvWorkgroups workgroups in all.  Whole tiles and in parts, bf16: 500 tokens
    // of 5376 channels 23 and 8 us, 2048 25 and 17 (1024 workgroups: 21), 4096 26 and 24 (32); 32768 tokens of 10240
    // channels, 2560 workgroups, 270 and, cut in two, 274.  Not where a state is updated in place: a whole tile's walk has
    // read the state in front of it before it writes the one behind, but the last part may write it before the first reads.
    a.parts = 1;
    while (!states_overlap && a.parts < kConvMostParts && (int64_t)n_tiles * a.blocks_per_tile * a.parts * 2 <= kConvWorkgroups &&
           plan->total_tokens > (int64_t)n_tiles * a.parts * kAhead)
        a.parts *= 2;
    const dim3 grid((unsigned)n_tiles * (unsigned)a.parts * (unsigned)a.blocks_per_tile);
    const bool f32 = plan->shape.io_dtype == SSM_DT_F32;
#define SSM_CONV_LAUNCH(KW)                                                                                  \
    case KW:                                                                                                 \
        if (f32)                                                                                             \
            hipLaunchKernelGGL((ssm_conv1d_kernel<float, KW>), grid, dim3(kConvThreads), 0, stream, a);      \
        else                                                                                                 \
            hipLaunchKernelGGL((ssm_conv1d_kernel<bf16_t, KW>), grid, dim3(kConvThreads), 0, stream, a);     \
        break;
    switch (K) {
        SSM_CONV_LAUNCH(1)
        SSM_CONV_LAUNCH(2)
        SSM_CONV_LAUNCH(3)
        SSM_CONV_LAUNCH(4)
    default: return hipErrorInvalidValue;
    }
#undef SSM_CONV_LAUNCH
    return hipGetLastError();
}
