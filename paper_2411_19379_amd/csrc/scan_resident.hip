// Matrix-core scan for gfx950 whose running state stays in the accumulators: d_state 128, bf16 x/dt/B/C/y, cached states
// in fp32, fp16 or bf16; layers with 64, 128 or 256 channels per head and groups that are a multiple of 256 channels wide.
//
// The per-tile algebra is that of scan_mfma.hip (tiles of q <= 64 tokens, fp16 operands of the two long contractions,
// bf16 ones of Gm.x, everything else fp32).  What differs is who does what:
//
// * One workgroup per (piece of a sequence, 256 neighbouring channels of the H x P channels of a token), the channels of
//   one group.  Wave w owns 32 of them and their state, 32 x 128 fp32 in 64 accumulator registers, for the whole piece:
//   the state update accumulates onto it, and it never passes through LDS.
// * B and C of a tile are read from device memory once per workgroup, converted to fp16 on their way to LDS, and the raw
//   scores C_i.B_j are computed once per workgroup: there is no operand preparation in front and no workspace for it.
// * A workgroup's part of a token row of x or y is 512 neighbouring bytes (128 in the other scan).
// * What a sequence-serial recurrence leaves idle is filled by cutting long sequences into pieces.  A first kernel,
//   ssm_segment_state_kernel, computes what the segments of every piece that is continued add to the state, as far as it
//   has not decayed below 2^-150 by the end of the piece; a piece of the second kernel,
//   ssm_scan_resident_kernel, starts from the sum of the segments in front of it.  So y is written once, from the true
//   state.  For pieces with many segments in front of them ssm_group_states_kernel sums these up in eights.  An infinity or
//   NaN does not decay: a last kernel, ssm_not_finite_kernel, which leaves at once if there is none, takes those in the state
//   at the end of a piece to the rest of the sequence.
//
// Time per call, this scan and the other: 128 heads, 131072 tokens 1430 us and 1850, 16 x 8192 1282 and 1689, 32 x 1024
// 353 and 485; 80 heads, 16 requests of 500 to 7700 tokens 522 and 564; 16 heads, 32768 tokens 85 and 118.  At 128 heads
// the scan kernel of 131072 tokens and 32 checkpoints takes 1280 us and moves 5.06 GB, 4.0 TB/s, the segments' 171 us and
// 0.65 GB.  What bounds it is the serial work of a tile on a compute unit, 3.9 us with a few units busy and 5.0 us with all.
// Counters of that call, per tile and wave: 547 vector, 41 matrix, 124 LDS, 13 memory instructions; vector units busy 45 % of
// the time, matrix cores 27 %, LDS 45 % (22 % of it bank conflicts), waves waiting 41 %, to issue 20 %: no unit is full, two
// waves per SIMD and two barriers per tile do not cover what each waits for.
//
// Lane layouts.  Everything a lane holds in runs is in natural order, eight neighbours at a time: the transpose reads that
// fetch a B^T or x^T operand pick the four 4-column groups of a 16-column block in the order 0, 2, 1, 3, so that
// accumulator row rho = 8 a + 4 q + r stands for index 16 (a / 2) + 8 q + 4 (a % 2) + r (pi(rho) below), and the results
// of one product are the operand of the next as they are.
#include <mutex>
#include <type_traits>

#include "mfma_utils.h"

namespace {

// Workgroup barrier that orders LDS traffic only: device memory accesses stay in flight.  Device memory written by these
// kernels is never read back by the same launch.
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

constexpr int kWaves = kResidentChannels / 32;
constexpr int kThreads = 64 * kWaves;
// Row strides in LDS: four rows of a transpose read meet on no bank; the pieces of a row of C, which go to the same lane of
// 16 operands, spread over the banks.
constexpr int LDB = kN + 24, LDX = kResidentChannels + 24, LDC = 64 + 1;
constexpr float kCutoffLog2 = -150.f;         // a finite state that has decayed below this adds nothing to others of its size
constexpr int kRowsBC = kThreads / 16, kPassesBC = kQ / kRowsBC;  // rows of B and C per pass of the workgroup
constexpr int kLanesX = kResidentChannels / 8, kRowsX = kThreads / kLanesX, kPassesX = kQ / kRowsX;  // and of x

struct ResidentTables {  // of one wave's head
    float ei[kQ];        // e^{l_i}
    float wt[kQ];        // e^{l_q - l_j} dt_j
    float ri[kQ];        // e^{l_i - l_31}
    float cf[kQ];        // e^{l_31 - l_j} dt_j
};
struct ResidentTile {
    _Float16 Bs[kQ][LDB];  // rows of B
    uint4 Cf[16][LDC];     // C as operands: [token half * 8 + k-step of 16 state indices][lane]
    bf16_t XY[kQ][LDX];    // x, token major; later y.  While a tile is worked on a wave touches its own columns only
    uint32_t dt[kQ][2];    // steps of the workgroup's up to four heads
};
struct ResidentLds {
    ResidentTile tile[2];
    uint4 Gs[3][2][64];             // raw score blocks as accumulator images, fp16
    uint4 none[2][2][64];           // zeros in the place of the first two
    ResidentTables tb[kWaves];
};
constexpr int kWindows = 2 * kWaves;  // of 64 tokens, looked back over at a time
struct SegmentLds {
    _Float16 Bs[kQ][LDB];
    bf16_t XY[kQ][LDX];
    uint32_t dt[kQ][2];
    float wt[kWaves][kQ];
    int from[kWaves];
    float window[kWindows][4];
};

struct ResidentArgs {
    const bf16_t *x, *dt, *B, *C;
    const float *A, *D;
    bf16_t *y;
    void *state_out;
    StatePtrs init;
    const SsmTile *tiles;
    const SsmPiece *pieces;  // of this launch, in launch order
    // per slot: what the segment adds to the state, as accumulator images.  Behind the segments' slots those of the groups
    float4 *carry;
    float *decay;            // per (slot, head): the total log2 decay; minus infinity if the slot holds nothing
    int n_segments, n_groups;
    // per piece that another one continues and 32 channels: whether the state at its end holds a value that is not finite;
    // if it does, that state, as accumulator images
    int *spoiled;
    float4 *spoil;
    int H, P, G, blocks, n_items;
    int kept;                // the cached states of cut sequences have been copied to `spoil`, 32 channels in each one's place
};

// pi: which of 32 columns or rows an operand lane stands for.
__device__ __forceinline__ int operand_index(int i)
{
    return (i & 19) | ((i & 4) << 1) | ((i & 8) >> 1);
}

// The operands of one tile on their way from device memory to LDS, 16 bytes of a token row at a time, and the steps of the
// workgroup's heads, every wave those of eight tokens.  Rows past the end of a partial tile re-read its last row: their
// step counts as zero, so any finite x and C will do; B is cleared there.  A tile that is not there is read through descriptors of size zero,
// which return zeros without touching memory.
struct TileRegs {
    uint4 b[kPassesBC], c[kPassesBC], x[kPassesX];
    uint32_t dt[2];
};
struct TileLoader {
    const unsigned char *x, *B, *C, *dt;  // of the workgroup's channels, group and heads, token 0
    uint32_t x_row, bc_row, dt_row;       // bytes per token row
    int heads;                            // of the workgroup: 4, 2 or 1
    int row, col;                         // the thread's row and column (of 8 elements) of a B or C row
    int xr, xc;                           // and of an x row
    int dt_tok;
    uint32_t x_own, bc_own, dt_own;       // byte offsets of the thread's row and column
    // of the tile to load
    rsrc_t xs, bs, cs, ds;
    uint32_t x_most, bc_most, dt_most;    // byte offset of the last row
    __device__ __forceinline__ void start(const SsmTile &t, bool live)
    {
        const uint32_t last = (uint32_t)(t.len - 1);
        x_most = last * x_row, bc_most = last * bc_row, dt_most = last * dt_row;
        xs = make_rsrc(x + (size_t)t.tok0 * x_row, live ? x_most + kResidentChannels * 2 : 0);
        bs = make_rsrc(B + (size_t)t.tok0 * bc_row, live ? bc_most + kN * 2 : 0);
        cs = make_rsrc(C + (size_t)t.tok0 * bc_row, live ? bc_most + kN * 2 : 0);
        ds = make_rsrc(dt + (size_t)t.tok0 * dt_row, live ? dt_most + 2 * heads : 0);
    }
    __device__ __forceinline__ static uint32_t least(uint32_t a, uint32_t b) { return a < b ? a : b; }
    // 16 bytes of row `up` + the thread's own, whose offset (with the column) is `own`: a uniform part and a part per lane.  A
    // lane past the last row reads the last 16 of the last row's `bytes`.
    __device__ __forceinline__ static uint4 row16(const rsrc_t &r, uint32_t own, uint32_t up, uint32_t most, uint32_t bytes)
    {
        up = least(up, most);
        return buf_load16(r, least(own, most - up + bytes - 16), up);
    }
    __device__ __forceinline__ void load_x(TileRegs &r, int m) const
    {
        r.x[m] = row16(xs, x_own, kRowsX * m * x_row, x_most, kResidentChannels * 2);
    }
    __device__ __forceinline__ void load_b(TileRegs &r, int m) const
    {
        r.b[m] = row16(bs, bc_own, kRowsBC * m * bc_row, bc_most, kN * 2);
    }
    __device__ __forceinline__ void load_c(TileRegs &r, int m) const
    {
        r.c[m] = row16(cs, bc_own, kRowsBC * m * bc_row, bc_most, kN * 2);
    }
    __device__ __forceinline__ void load_dt(TileRegs &r) const
    {
        const uint32_t off = least(dt_own, dt_most);
        if (heads == 4) {
            const auto u = __builtin_amdgcn_raw_buffer_load_b64(ds, (int)off, 0, 0);
            r.dt[0] = u[0], r.dt[1] = u[1];
        } else if (heads == 2) {
            r.dt[0] = __builtin_amdgcn_raw_buffer_load_b32(ds, (int)off, 0, 0);
        } else {
            r.dt[0] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(ds, (int)off, 0, 0);
        }
    }
    template <bool kC> __device__ __forceinline__ void load(TileRegs &r, const SsmTile &t)
    {
        start(t, true);
#pragma unroll
        for (int m = 0; m < kPassesX; ++m)
            load_x(r, m);
#pragma unroll
        for (int m = 0; m < kPassesBC; ++m) {
            load_b(r, m);
            if constexpr (kC)
                load_c(r, m);
        }
        load_dt(r);
    }
};
// Zeros in the rows of B behind a partial tile, which the loader fills with its last row: that row may hold infinities (or
// values above the fp16 range), and 0 x inf is NaN.  Behind the thread's own stores to the same rows.
__device__ __forceinline__ void clear_rows_behind(_Float16 (*Bs)[LDB], const TileLoader &ld, int len)
{
    if (__builtin_expect(len < kQ, 0)) {
        const uint32_t zero = (uint32_t)len >> 16;  // a constant would occupy four registers throughout
#pragma unroll
        for (int m = 0; m < kPassesBC; ++m)
            if (ld.row + kRowsBC * m >= len)
                *reinterpret_cast<uint4 *>(&Bs[ld.row + kRowsBC * m][ld.col]) = make_uint4(zero, zero, zero, zero);
    }
}
__device__ __forceinline__ TileLoader make_loader(const ResidentArgs &a, int c0, int g)
{
    TileLoader l;
    const int tid = threadIdx.x;
    l.heads = kResidentChannels > a.P ? kResidentChannels / a.P : 1;
    l.x = reinterpret_cast<const unsigned char *>(a.x) + (size_t)c0 * 2;
    l.B = reinterpret_cast<const unsigned char *>(a.B) + (size_t)g * kN * 2;
    l.C = reinterpret_cast<const unsigned char *>(a.C) + (size_t)g * kN * 2;
    l.dt = reinterpret_cast<const unsigned char *>(a.dt) + (size_t)(c0 / a.P) * 2;
    l.x_row = (uint32_t)a.H * a.P * 2;
    l.bc_row = (uint32_t)a.G * kN * 2;
    l.dt_row = (uint32_t)a.H * 2;
    l.row = tid >> 4, l.col = 8 * (tid & 15);
    l.xr = tid / kLanesX, l.xc = 8 * (tid % kLanesX);
    l.dt_tok = 8 * (tid >> 6) + (tid & 7);
    l.x_own = l.xr * l.x_row + l.xc * 2, l.bc_own = l.row * l.bc_row + l.col * 2, l.dt_own = l.dt_tok * l.dt_row;
    return l;
}
// The step of token `lane` of head `hd` of the workgroup.
__device__ __forceinline__ float step_of(const uint32_t (*dt)[2], int lane, int hd, int len)
{
    const uint32_t u = dt[lane][hd >> 1];
    return lane < len ? __uint_as_float((hd & 1) ? u & 0xffff0000u : u << 16) : 0.f;
}

// l log2(e), rounded before anything is subtracted from it, as in the other scan: both give a token the same weight.
__device__ __forceinline__ float to_log2(float l)
{
#pragma clang fp contract(off)
    return l * kLog2e;
}

// The accumulator images of a slot or of a continued piece, from channel cw on, in float4 units: + 16 * 64 per 32 channels,
// + (4 nb + a) 64 + lane.
__device__ __forceinline__ size_t carry_at(const ResidentArgs &a, int slot, int cw)
{
    return ((size_t)slot * ((size_t)a.H * a.P / 32) + cw / 32) * (16 * 64);
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniform(float v) { return read_lane(v, 0); }

// What of the masks does not depend on the tile: element 4 a + r of a lane is key 16 (a / 2) + 8 q + 4 (a % 2) + r.
struct LaneMask {
    int diag;         // i - 8 q
    // pairs of elements as packed, all ones where the key is not behind the query: within 16 tokens, and whether the query
    // is one of the later 16 of the block
    uint32_t on[4], later;
};
__device__ __forceinline__ LaneMask make_mask(int i, int q)
{
    LaneMask m;
    m.diag = i - 8 * q;
    m.later = i >= 16 ? 0xffffffffu : 0u;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int j = 8 * q + 2 * e;
        m.on[e] = (j <= (i & 15) ? 0x0000ffffu : 0u) | (j + 1 <= (i & 15) ? 0xffff0000u : 0u);
    }
    return m;
}
// A quarter (elements 4 a .. 4 a + 3) of a diagonal block of raw scores, decayed by f, D added on the diagonal, masked and
// packed: two words of an operand of Gm.x.
__device__ __forceinline__ uint2 mask_quarter(uint32_t raw0, uint32_t raw1, const float (&f)[4], int a, const LaneMask &m,
                                              float Dh)
{
    const int e0 = 16 * (a >> 1) + 4 * (a & 1);
    const float v0 = __builtin_fmaf(f16_lo(raw0), f[0], e0 + 0 == m.diag ? Dh : 0.f);
    const float v1 = __builtin_fmaf(f16_hi(raw0), f[1], e0 + 1 == m.diag ? Dh : 0.f);
    const float v2 = __builtin_fmaf(f16_lo(raw1), f[2], e0 + 2 == m.diag ? Dh : 0.f);
    const float v3 = __builtin_fmaf(f16_hi(raw1), f[3], e0 + 3 == m.diag ? Dh : 0.f);
    const uint32_t lo = pack2_bf16(v0, v1), hi = pack2_bf16(v2, v3), on0 = m.on[2 * (a & 1)], on1 = m.on[2 * (a & 1) + 1];
    return a < 2 ? make_uint2(lo & (on0 | m.later), hi & (on1 | m.later)) : make_uint2(lo & on0 & m.later, hi & on1 & m.later);
}

// x^T of 32 channels as fp16 operands weighted by decay: the weights are those of tokens 16 ks + 8 q + e.
__device__ __forceinline__ uint4 weighted(const uint4 &xv, const float4 &w0, const float4 &w1)
{
    return make_uint4(pack2_f16(w0.x * bf16_lo(xv.x), w0.y * bf16_hi(xv.x)), pack2_f16(w0.z * bf16_lo(xv.y), w0.w * bf16_hi(xv.y)),
                      pack2_f16(w1.x * bf16_lo(xv.z), w1.y * bf16_hi(xv.z)), pack2_f16(w1.z * bf16_lo(xv.w), w1.w * bf16_hi(xv.w)));
}

// ================================================================ what a segment adds to the state
// One workgroup per (segment, 256 channels).  First every wave looks back over the steps of its head from the end of the
// piece, where the segment's contribution is used: what has decayed below the cutoff by there is left out, which for decay
// rates as trained models have them is all but some thirty tiles.  From the earliest token that counts for one of its heads
// the workgroup then walks forwards like the scan, without outputs.
template <int ST>
__global__ __launch_bounds__(kThreads, 4) void ssm_segment_state_kernel(ResidentArgs a)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    SegmentLds &L = *reinterpret_cast<SegmentLds *>(lds_raw);
    const int item = ssm_launch_item(blockIdx.x, a.n_items);
    if (item < 0)
        return;
    const SsmPiece p = scalar_load(a.pieces + item / a.blocks);
    const int lane = threadIdx.x & 63, w = uniform((int)threadIdx.x >> 6);
    const int c0 = item % a.blocks * kResidentChannels, cw = c0 + 32 * w;
    const int h = uniform(cw / a.P), g = c0 / (a.H / a.G * a.P);
    const float Ah = scalar_load(a.A + h);
    const SsmTile first = scalar_load(a.tiles + p.tile_begin), end = scalar_load(a.tiles + p.stop - 1);

    // The first token that counts for this wave's head; two more than the cutoff, because the sum that whoever uses the slot
    // compares may differ by rounding.  The waves share the work: each sums the steps of all heads of the workgroup over
    // windows of 64 tokens.
    int from = end.tok0 + end.len;
    bool cut = false;
    {
        const int heads = kResidentChannels > a.P ? kResidentChannels / a.P : 1, hd = h - c0 / a.P;
        const bf16_t *dt = a.dt + c0 / a.P;
        float sum = 0.f;
        for (int to = from; to > first.tok0; to -= 64 * kWindows) {
            lds_barrier();  // the sums before have been read
#pragma unroll
            for (int u = 0; u < kWindows; u += kWaves) {
                const int tok = to - 64 * (u + w) - 1 - lane;
                uint32_t d[2] = {0, 0};
                if (tok >= first.tok0) {
                    const void *at = dt + (size_t)tok * a.H;
                    if (heads == 4) {
                        const uint2 v = *static_cast<const uint2 *>(at);
                        d[0] = v.x, d[1] = v.y;
                    } else if (heads == 2) {
                        d[0] = *static_cast<const uint32_t *>(at);
                    } else {
                        d[0] = *static_cast<const bf16_t *>(at);
                    }
                }
                const float s0 = read_lane(wave_inclusive_sum(bf16_lo(d[0])), 63), s1 = read_lane(wave_inclusive_sum(bf16_hi(d[0])), 63);
                const float s2 = read_lane(wave_inclusive_sum(bf16_lo(d[1])), 63), s3 = read_lane(wave_inclusive_sum(bf16_hi(d[1])), 63);
                if (lane == 0)
                    *reinterpret_cast<float4 *>(L.window[u + w]) = make_float4(s0, s1, s2, s3);
            }
            lds_barrier();
            for (int u = 0; u < kWindows && !cut && from > first.tok0; ++u) {
                sum += uniform(L.window[u][hd]) * Ah * kLog2e;
                from -= 64;
                cut = sum < kCutoffLog2 - 2.f;
            }
            bool all = cut;
            if (lane == 0)
                L.from[w] = cut;
            lds_barrier();
#pragma unroll
            for (int v = 0; v < kWaves; ++v)
                all = all && L.from[v] != 0;
            if (uniform((int)all))
                break;  // the whole workgroup: every wave has read the same values
        }
        lds_barrier();
        from = uniform(from > first.tok0 ? from : first.tok0);
    }
    if (lane == 0)
        L.from[w] = from;
    lds_barrier();
    int earliest = L.from[0];
#pragma unroll
    for (int v = 1; v < kWaves; ++v)
        earliest = L.from[v] < earliest ? L.from[v] : earliest;
    earliest = uniform(earliest);
    // tiles that end before it
    int k = p.tile_begin;
    for (int k0 = p.tile_begin; k0 < p.tile_end; k0 += 64) {
        bool before = false;
        if (k0 + lane < p.tile_end) {
            const SsmTile u = a.tiles[k0 + lane];
            before = u.tok0 + u.len <= earliest;
        }
        k += (int)read_lane(wave_inclusive_sum(before ? 1.f : 0.f), 63);
    }
    k = uniform(k);
    if (k >= p.tile_end) {  // the whole workgroup; nobody gets as far as these slots
        if (lane == 0 && cw % a.P == 0)
            a.decay[(size_t)p.slot * a.H + h] = -__builtin_inff();
        return;
    }

    const int q = lane >> 5, g4 = lane >> 4;
    const int tr_row = 8 * (g4 >> 1) + ((lane & 15) >> 2), tr_col = 16 * (g4 & 1) + 4 * ((lane & 1) * 2 + ((lane >> 1) & 1));
    TileLoader ld = make_loader(a, c0, g);
    TileRegs regs;
    SsmTile t = scalar_load(a.tiles + k);
    ld.load<false>(regs, t);
    f32x16 S[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
        S[nb] = zero16();
    const void *init = p.back == 0 && !cut ? a.init.of(p.seq) : nullptr;
    if (init) {  // (+ 0: the sum waits for the loads here; else the wait would be in the loop, for loads ahead as well)
        const size_t row = ((size_t)cw + operand_index(lane & 31)) * kN + 8 * q;
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float4 v = load_state4(init, row + 32 * nb + 16 * (e >> 1) + 4 * (e & 1), ST);
                S[nb][4 * e + 0] = v.x + 0.f;
                S[nb][4 * e + 1] = v.y + 0.f;
                S[nb][4 * e + 2] = v.z + 0.f;
                S[nb][4 * e + 3] = v.w + 0.f;
            }
    }
    float decay = 0.f;  // of the tiles that count, log2
    for (; k < p.tile_end; ++k) {
        SsmTile t_next = t;
        if (k + 1 < p.tile_end)
            t_next = scalar_load(a.tiles + k + 1);
#pragma unroll
        for (int m = 0; m < kPassesBC; ++m)
            *reinterpret_cast<uint4 *>(&L.Bs[ld.row + kRowsBC * m][ld.col]) = bf16x8_to_f16x8(regs.b[m]);
#pragma unroll
        for (int m = 0; m < kPassesX; ++m)
            *reinterpret_cast<uint4 *>(&L.XY[ld.xr + kRowsX * m][ld.xc]) = regs.x[m];
        if (lane < 8)
            *reinterpret_cast<uint2 *>(L.dt[ld.dt_tok]) = make_uint2(regs.dt[0], regs.dt[1]);
        clear_rows_behind(L.Bs, ld, t.len);
        lds_barrier();
        if (k + 1 < p.tile_end)
            ld.load<false>(regs, t_next);
        if (t.tok0 + t.len > from) {  // uniform in the wave
            const float dtj = step_of(L.dt, lane, h - c0 / a.P, t.len);
            const float ell2 = wave_inclusive_sum(dtj * Ah) * kLog2e, last = read_lane(ell2, 63);
            L.wt[w][lane] = exp2_fast(last - ell2) * dtj;
            __builtin_amdgcn_wave_barrier();
            const float dl = exp2_fast(last);
            decay += last;
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    S[nb][e] *= dl;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                const bf16_t *px = &L.XY[16 * ks + tr_row][32 * w + tr_col];
                uint4 b[4];
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) {
                    const _Float16 *pb = &L.Bs[16 * ks + tr_row][32 * nb + tr_col];
                    b[nb] = lds_frag_tr(pb, pb + 4 * LDB);
                }
                const uint4 xw = weighted(lds_frag_tr(px, px + 4 * LDX), *reinterpret_cast<const float4 *>(&L.wt[w][16 * ks + 8 * q]),
                                          *reinterpret_cast<const float4 *>(&L.wt[w][16 * ks + 8 * q + 4]));
#pragma unroll
                for (int nb = 0; nb < 4; ++nb)
                    S[nb] = mfma_f16(b[nb], xw, S[nb]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        lds_barrier();
        t = t_next;
    }
    float4 *out = a.carry + carry_at(a, p.slot, cw) + lane;
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            out[(4 * nb + e) * 64] = make_float4(S[nb][4 * e], S[nb][4 * e + 1], S[nb][4 * e + 2], S[nb][4 * e + 3]);
    if (lane == 0 && cw % a.P == 0)
        a.decay[(size_t)p.slot * a.H + h] = decay;
}

// ================================================================ sums of segments
// One workgroup per (group of kGroupSlots slots, 32 channels): what the group's segments add to the state at the end of the last
// one.  The pieces at least another group behind it start from this sum instead of the slots.  With decay so slow that every
// segment counts in all that follows, 33000 tokens of 8 heads (129 slots in front of the last piece) take 170 us without and
// 90 us with it; where the next group of slots alone decays below the cutoff, nothing is read.  A group may hold slots of two
// sequences: nobody reads that one.
constexpr int kGroupThreads = 256;
__global__ __launch_bounds__(kGroupThreads) void ssm_group_states_kernel(ResidentArgs a)
{
    const int units = a.H * a.P / 32, group = blockIdx.x / units, cw = 32 * (blockIdx.x % units);
    const int h = cw / a.P, first = group * kGroupSlots;
    auto decay_of = [&](int slot) { return scalar_load(a.decay + (size_t)slot * a.H + h); };
    float behind = 0.f;
#pragma unroll
    for (int s = first + kGroupSlots; s < first + 2 * kGroupSlots; ++s)
        behind += decay_of(s < a.n_segments ? s : a.n_segments - 1);  // all loads at once
    if (first + 2 * kGroupSlots > a.n_segments)
        behind = -__builtin_inff();
    // f[s]: from the end of slot `first` + s to the end of the group
    float f[kGroupSlots], all = 0.f;
#pragma unroll
    for (int s = kGroupSlots - 1; s >= 0; --s) {
        f[s] = all;
        all += decay_of(first + s);
    }
    const bool made = behind >= kCutoffLog2 - 2.f && all > -__builtin_inff();  // neither if one is NaN
    if (threadIdx.x == 0 && cw % a.P == 0)
        a.decay[(size_t)(a.n_segments + group) * a.H + h] = made ? all : -__builtin_inff();
    if (!made)
        return;
    for (int m = threadIdx.x; m < 16 * 64; m += kGroupThreads) {
        float4 v[kGroupSlots];
#pragma unroll
        for (int s = 0; s < kGroupSlots; ++s)
            v[s] = a.carry[carry_at(a, first + s, cw) + m];
        float4 sum = v[kGroupSlots - 1];
#pragma unroll
        for (int s = kGroupSlots - 2; s >= 0; --s) {
            const float scale = exp2_fast(f[s]);
            sum.x = __builtin_fmaf(scale, v[s].x, sum.x);
            sum.y = __builtin_fmaf(scale, v[s].y, sum.y);
            sum.z = __builtin_fmaf(scale, v[s].z, sum.z);
            sum.w = __builtin_fmaf(scale, v[s].w, sum.w);
        }
        a.carry[carry_at(a, a.n_segments + group, cw) + m] = sum;
    }
}

// ================================================================ the scan
// One workgroup per (piece, 256 channels).  The tiles alternate between two LDS buffers: while one is worked on, the rows
// of the next are converted into the other and those of the one after are requested.  Two barriers per tile: operands in
// place (and the tile before done), raw scores in place.
//
// Why 8 waves x 32 channels: workgroups of 128 channels, two per unit, convert and score B and C twice as often, and waves
// of 64 channels leave no registers for the rows in flight; both measured slower.
template <int ST>
__global__ __launch_bounds__(kThreads, 2) void ssm_scan_resident_kernel(ResidentArgs a)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    ResidentLds &L = *reinterpret_cast<ResidentLds *>(lds_raw);
    const int item = ssm_launch_item(blockIdx.x, a.n_items);
    if (item < 0)
        return;
    const SsmPiece p = scalar_load(a.pieces + item / a.blocks);
    const int lane = threadIdx.x & 63, w = uniform((int)threadIdx.x >> 6);
    const int c0 = item % a.blocks * kResidentChannels, cw = c0 + 32 * w;
    const int h = uniform(cw / a.P), g = c0 / (a.H / a.G * a.P);
    const float Ah = scalar_load(a.A + h);
    const int i = lane & 31, q = lane >> 5, g4 = lane >> 4, pi = operand_index(i);
    const int tr_row = 8 * (g4 >> 1) + ((lane & 15) >> 2), tr_col = 16 * (g4 & 1) + 4 * ((lane & 1) * 2 + ((lane >> 1) & 1));
    TileLoader ld = make_loader(a, c0, g);
    const int hd = h - c0 / a.P;  // the wave's head in the workgroup
    unsigned char *yh = reinterpret_cast<unsigned char *>(a.y) + (size_t)c0 * 2;
    ResidentTables &W = L.tb[w];
    // + 32 nb + 16 (a / 2) + 4 (a % 2): this lane's 4 state values of element group a
    const size_t state_row = ((size_t)cw + pi) * kN + 8 * q;

    TileRegs regs;
    SsmTile t = scalar_load(a.tiles + p.tile_begin), t_next = t;
    ld.load<true>(regs, t);

    f32x16 S[4];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
        S[nb] = zero16();
    if (p.back > 0) {
        // what the pieces in front add, the nearest first, until it has decayed to nothing.  Farther away whole groups of slots,
        // where there is such a sum
        float f = 0.f;
        for (int m = 0, step = 1; m < p.back && f >= kCutoffLog2; m += step) {
            const float scale = exp2_fast(f);
            int slot = p.slot - m;
            step = 1;
            if (a.n_groups > 0 && m >= kGroupSlots && p.back - m >= kGroupSlots && slot % kGroupSlots == kGroupSlots - 1) {
                const int group = a.n_segments + slot / kGroupSlots;
                if (scalar_load(a.decay + (size_t)group * a.H + h) > -__builtin_inff()) {
                    slot = group;
                    step = kGroupSlots;
                }
            }
            const float4 *in = a.carry + carry_at(a, slot, cw) + lane;
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float4 v = in[(4 * nb + e) * 64];
                    S[nb][4 * e + 0] = __builtin_fmaf(scale, v.x, S[nb][4 * e + 0]);
                    S[nb][4 * e + 1] = __builtin_fmaf(scale, v.y, S[nb][4 * e + 1]);
                    S[nb][4 * e + 2] = __builtin_fmaf(scale, v.z, S[nb][4 * e + 2]);
                    S[nb][4 * e + 3] = __builtin_fmaf(scale, v.w, S[nb][4 * e + 3]);
                }
            f += scalar_load(a.decay + (size_t)slot * a.H + h);
        }
    } else if (const void *init = a.init.of(p.seq)) {
        size_t row = state_row;
        if (a.kept && p.tile_end < p.stop) {
            init = a.spoil + carry_at(a, p.first, cw);
            row -= (size_t)cw * kN;
        }
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float4 v = load_state4(init, row + 32 * nb + 16 * (e >> 1) + 4 * (e & 1), ST);
                S[nb][4 * e + 0] = v.x + 0.f;
                S[nb][4 * e + 1] = v.y + 0.f;
                S[nb][4 * e + 2] = v.z + 0.f;
                S[nb][4 * e + 3] = v.w + 0.f;
            }
    }

    const LaneMask mask = make_mask(i, q);
    const uint32_t yoff = ld.x_own;
    uint4 yr[kPassesX];
    auto read_y = [&](const ResidentTile &T) {
#pragma unroll
        for (int m = 0; m < kPassesX; ++m)
            yr[m] = *reinterpret_cast<const uint4 *>(&T.XY[ld.xr + kRowsX * m][ld.xc]);
    };
    auto store_y = [&](int tok0, int len) {
        const rsrc_t ys = make_rsrc(yh + (size_t)tok0 * ld.x_row, (uint32_t)(len - 1) * ld.x_row + kResidentChannels * 2);
        if (len == kQ) {
#pragma unroll
            for (int m = 0; m < kPassesX; ++m)
                buf_store16(ys, yoff, kRowsX * m * ld.x_row, yr[m]);
        } else {
#pragma unroll
            for (int m = 0; m < kPassesX; ++m)
                if (ld.xr + kRowsX * m < len)
                    buf_store16(ys, yoff, kRowsX * m * ld.x_row, yr[m]);
        }
    };
    // A tile's rows from registers to LDS, a piece at a time; the registers then take the same piece of another tile.  A
    // thread writes x where it has read y.
    auto stage_x = [&](ResidentTile &T, int m) {
        *reinterpret_cast<uint4 *>(&T.XY[ld.xr + kRowsX * m][ld.xc]) = regs.x[m];
    };
    auto stage_b = [&](ResidentTile &T, int m) {
        *reinterpret_cast<uint4 *>(&T.Bs[ld.row + kRowsBC * m][ld.col]) = bf16x8_to_f16x8(regs.b[m]);
    };
    auto stage_c = [&](ResidentTile &T, int m) {
        // token `row`, state indices col .. col + 7: lane (row % 32, (col / 8) % 2) of operand (row / 32, col / 16)
        const int row = ld.row + kRowsBC * m;
        T.Cf[(row >> 5) * 8 + (ld.col >> 4)][(row & 31) + 4 * (ld.col & 8)] = bf16x8_to_f16x8(regs.c[m]);
    };
    auto stage_dt = [&](ResidentTile &T) {
        if (lane < 8)
            *reinterpret_cast<uint2 *>(T.dt[ld.dt_tok]) = make_uint2(regs.dt[0], regs.dt[1]);
    };
    // the eight pieces of a tile
    auto stage = [&](ResidentTile &T, int m) {
        if (m < 4)
            stage_x(T, m);
        else if (m & 1)
            stage_c(T, (m - 4) >> 1);
        else
            stage_b(T, (m - 4) >> 1);
        if (m == 7)
            stage_dt(T);
    };
    auto request = [&](int m) {
        if (m < 4)
            ld.load_x(regs, m);
        else if (m & 1)
            ld.load_c(regs, (m - 4) >> 1);
        else
            ld.load_b(regs, (m - 4) >> 1);
        if (m == 7)
            ld.load_dt(regs);
    };
    static_assert(kPassesX == 4 && kPassesBC == 2, "eight pieces");

    for (int m = threadIdx.x; m < 4 * 64; m += kThreads)
        L.none[0][0][m] = make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int m = 0; m < 8; ++m)
        stage(L.tile[0], m);
    clear_rows_behind(L.tile[0].Bs, ld, t.len);
    const bool two = p.tile_begin + 1 < p.tile_end;
    if (two)
        t_next = scalar_load(a.tiles + p.tile_begin + 1);
    ld.start(t_next, two);
#pragma unroll
    for (int m = 0; m < 8; ++m)
        request(m);
    int y_tok0 = 0, y_len = 0;  // the tile whose y waits in the other buffer
    for (int k = p.tile_begin; k < p.tile_end; ++k) {
        ResidentTile &T = L.tile[(k - p.tile_begin) & 1], &O = L.tile[~(k - p.tile_begin) & 1];
        SsmTile t_after = t_next;
        if (k + 2 < p.tile_end)
            t_after = scalar_load(a.tiles + k + 2);
        const float Dh = scalar_load(a.D + h);  // read per tile: what is made of it would fill 16 registers
        lds_barrier();  // the tile is in place, the one before is done and its y in the other buffer
        auto x_operand = [&](int ks) {
            return lds_frag_tr(&T.XY[16 * ks + tr_row][32 * w + tr_col], &T.XY[16 * ks + tr_row + 4][32 * w + tr_col]);
        };
        auto float4_at = [&](const float *v) { return *reinterpret_cast<const float4 *>(v); };
        // ---------------- raw score blocks Gm^T[j, i] = B_j . C_i: block 0 keys and queries 0..31, block 1 keys and queries
        // 32..63, block 2 keys 0..31 and queries 32..63
        if (w < 3) {
            const int row = (w == 1 ? 32 : 0) + pi;
            f32x16 acc = zero16();
            uint4 bo[2], co[2];
            auto load = [&](int ks) {
                bo[ks & 1] = *reinterpret_cast<const uint4 *>(&T.Bs[row][16 * ks + 8 * q]);
                co[ks & 1] = T.Cf[(w == 0 ? 0 : 8) + ks][lane];
            };
            load(0);
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) {
                if (ks < 7)
                    load(ks + 1);
                acc = mfma_f16(bo[ks & 1], co[ks & 1], acc);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int hf = 0; hf < 2; ++hf)
                L.Gs[w][hf][lane] =
                    make_uint4(pack2_f16(acc[8 * hf + 0], acc[8 * hf + 1]), pack2_f16(acc[8 * hf + 2], acc[8 * hf + 3]),
                               pack2_f16(acc[8 * hf + 4], acc[8 * hf + 5]), pack2_f16(acc[8 * hf + 6], acc[8 * hf + 7]));
        }
        // ---------------- S.C from the state in front of the tokens, 16 state indices at a time; between the products the
        // factor tables, y of the tile before, and x^T of the wave's channels weighted by decay
        uint4 cf[2][2];
        auto load_c = [&](int ks) {
            cf[ks & 1][0] = T.Cf[ks][lane];
            cf[ks & 1][1] = T.Cf[8 + ks][lane];
        };
        load_c(0);
        load_c(1);
        if (y_len)
            read_y(O);
        // The token's step, the log2 decay up to and including it, that of token 31, the total.
        const float dtj = step_of(T.dt, lane, hd, t.len);
        const float ell2 = to_log2(wave_inclusive_sum(dtj * Ah)), mid = read_lane(ell2, 31), last = read_lane(ell2, 63);
        // The factors e^{l_i - l_31} and e^{l_31 - l_j} of the diagonal blocks must stay inside the fp32 exponent range
        // (2^+-100 is far inside).  If they do not, or a step is NaN, the blocks' scores and factors are zeros here, and what
        // the blocks contribute is added behind the others; the factors of the third block are at most 1 whatever the decay.
        const bool fast = mid > -100.f && last - mid > -100.f;
        const uint4 *diag = fast ? &L.Gs[0][0][lane] : &L.none[0][0][lane];
        float dl = 0.f;
        f32x16 Y[2] = {zero16(), zero16()};  // [token half]
        uint4 xw[4], xb;
        float4 wb[2];
        auto load_x = [&](int ks) {
            xb = x_operand(ks);
            wb[0] = float4_at(&W.wt[16 * ks + 8 * q]);
            wb[1] = float4_at(&W.wt[16 * ks + 8 * q + 4]);
        };
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            const f32x16 &Sb = S[ks >> 1];
            const int e = 8 * (ks & 1);
            const uint4 s16 = make_uint4(pack2_f16(Sb[e + 0], Sb[e + 1]), pack2_f16(Sb[e + 2], Sb[e + 3]),
                                         pack2_f16(Sb[e + 4], Sb[e + 5]), pack2_f16(Sb[e + 6], Sb[e + 7]));
            Y[0] = mfma_f16(s16, cf[ks & 1][0], Y[0]);
            Y[1] = mfma_f16(s16, cf[ks & 1][1], Y[1]);
            if (ks + 2 < 8)
                load_c(ks + 2);
            if (ks == 0) {
                W.wt[lane] = exp2_fast(last - ell2) * dtj;
                __builtin_amdgcn_wave_barrier();  // LDS executes a wave's accesses in order
            }
            if (ks == 1) {
                W.ei[lane] = exp2_fast(ell2);
                W.ri[lane] = exp2_fast(ell2 - mid);
            }
            if (ks == 2) {
                W.cf[lane] = exp2_fast(mid - ell2) * dtj;
                dl = exp2_fast(last);  // padded tokens have dt = 0, so this is e^{l_len}
            }
            if (ks >= 4)
                xw[ks - 4] = weighted(xb, wb[0], wb[1]);
            if (ks >= 3 && ks < 7)
                load_x(ks - 3);
            __builtin_amdgcn_sched_barrier(0);
            if (ks == 0 && y_len)
                store_y(y_tok0, y_len);
            if (ks == 2 && __builtin_expect(!fast, 0)) {
                const float key = W.cf[lane];
                W.ri[lane & 31] = 0.f;
                // NaN where a step of the first half is; the queries' factor of the third block is then NaN too
                if (lane >= 32 || key != key)
                    W.cf[lane] = 0.f;
            }
        }
        lds_barrier();  // the raw scores are in place
        // ---------------- the decayed state accumulates the update, two blocks of 32 state indices x 16 tokens at a time;
        // between the products the decay mask (+ D on the diagonal), which makes the operands of Gm.x:
        // e^{l_i-l_j} dt_j = e^{l_i-l_31} * e^{l_31-l_j} dt_j from two factor tables
        auto decay_state = [&](int nb) {
#pragma unroll
            for (int e = 0; e < 16; ++e)
                S[nb][e] *= dl;
        };
        uint4 bt[2];
        auto load_b = [&](int st) {
            const int n2 = st >> 2 << 1, ks = st & 3;
#pragma unroll
            for (int u = 0; u < 2; ++u)
                bt[u] = lds_frag_tr(&T.Bs[16 * ks + tr_row][32 * (n2 + u) + tr_col],
                                    &T.Bs[16 * ks + tr_row + 4][32 * (n2 + u) + tr_col]);
        };
        auto update = [&](int st) {
#pragma unroll
            for (int u = 0; u < 2; ++u)
                S[(st >> 2 << 1) + u] = mfma_f16(bt[u], xw[st & 3], S[(st >> 2 << 1) + u]);
        };
        const auto key_of = [&](int a) { return 16 * (a >> 1) + 8 * q + 4 * (a & 1); };
        const float ri[2] = {W.ri[i], W.ri[32 + i]}, ei[2] = {W.ei[i], W.ei[32 + i]};
        float4 key = float4_at(&W.cf[key_of(0)]);
        uint4 raw = diag[0], g = make_uint4(0, 0, 0, 0);
        load_b(0);
        ld.start(t_after, k + 2 < p.tile_end);
        decay_state(0);
        decay_state(1);
#pragma unroll
        for (int e = 0; e < 16; ++e)
            Y[0][e] *= ei[0];
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int st = 0; st < 8; ++st) {
            const int blk = st >> 2, a = st & 3, nx = st + 1;
            update(st);
            if (nx < 8)
                load_b(nx);
            if (a & 1)
                xb = x_operand(2 * blk + (a >> 1));
            const float f[4] = {ri[blk] * key.x, ri[blk] * key.y, ri[blk] * key.z, ri[blk] * key.w};
            key = nx < 8 ? float4_at(&W.cf[32 * (nx >> 2) + key_of(nx & 3)]) : float4_at(&W.cf[key_of(0)]);
            const uint2 two = (a & 1) ? mask_quarter(raw.z, raw.w, f, a, mask, Dh) : mask_quarter(raw.x, raw.y, f, a, mask, Dh);
            if (a & 1) {
                g.z = two.x, g.w = two.y;
                raw = nx < 8 ? diag[nx / 2 * 64] : L.Gs[2][0][lane];
                Y[blk] = mfma_bf16(xb, g, Y[blk]);  // Gm.x is added onto e^{l_i} (S C_i)
            } else {
                g.x = two.x, g.y = two.y;
            }
            if (st == 0)
                decay_state(2);
            if (st == 1)
                decay_state(3);
            if (st == 2 || st == 3)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    Y[1][8 * (st & 1) + e] *= ei[1];
            stage(O, st);  // the next tile into the other buffer, the rows of the one after requested
            request(st);
            __builtin_amdgcn_sched_barrier(0);
        }
        // keys 0..31, queries 32..63: unmasked
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            auto pair = [&](uint32_t r, float u, float v) {
                return pack2_bf16(f16_lo(r) * (ri[1] * u), f16_hi(r) * (ri[1] * v));
            };
            const float4 k1 = float4_at(&W.cf[key_of(2 * ks + 1)]);
            xb = x_operand(ks);
            g = make_uint4(pair(raw.x, key.x, key.y), pair(raw.y, key.z, key.w), pair(raw.z, k1.x, k1.y), pair(raw.w, k1.z, k1.w));
            if (ks == 0) {
                key = float4_at(&W.cf[key_of(2)]);
                raw = L.Gs[2][1][lane];
            }
            Y[1] = mfma_bf16(xb, g, Y[1]);
        }
        __builtin_amdgcn_sched_barrier(0);
        // ---------------- the diagonal blocks of a tile that decays by too much for the factors: one exponential per score.
        // x is still in place here, so the tile takes one walk whatever its decay (walks over windows of tokens that
        // together decay by less, each leaving its y over x for the next, took 16 x 8192 tokens of 128 heads with A = -16 and
        // dt = 0.1 5.9 ms instead of 1.28, and made a y that is not finite 0 x inf in the state).
        if (__builtin_expect(!fast, 0)) {
            const float step = step_of(T.dt, lane, hd, t.len), l = to_log2(wave_inclusive_sum(step * Ah));
            W.ei[lane] = l;  // both tables have been read
            W.wt[lane] = l - __builtin_amdgcn_logf(step);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                const float li = W.ei[32 * blk + i];
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) {
                    const uint4 r = L.Gs[blk][hf][lane];
                    const float4 c0 = float4_at(&W.wt[32 * blk + key_of(2 * hf)]), c1 = float4_at(&W.wt[32 * blk + key_of(2 * hf + 1)]);
                    const float f0[4] = {exp2_fast(li - c0.x), exp2_fast(li - c0.y), exp2_fast(li - c0.z), exp2_fast(li - c0.w)};
                    const float f1[4] = {exp2_fast(li - c1.x), exp2_fast(li - c1.y), exp2_fast(li - c1.z), exp2_fast(li - c1.w)};
                    const uint2 g0 = mask_quarter(r.x, r.y, f0, 2 * hf, mask, 0.f), g1 = mask_quarter(r.z, r.w, f1, 2 * hf + 1, mask, 0.f);
                    Y[blk] = mfma_bf16(x_operand(2 * blk + hf), make_uint4(g0.x, g0.y, g1.x, g1.y), Y[blk]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // ---------------- y over the wave's own columns of x: elements 8 hf .. 8 hf + 7 are channels 16 hf + 8 q .. + 7 of
        // token 32 ih + i
#pragma unroll
        for (int ih = 0; ih < 2; ++ih)
#pragma unroll
            for (int hf = 0; hf < 2; ++hf)
                *reinterpret_cast<uint4 *>(&T.XY[32 * ih + i][32 * w + 16 * hf + 8 * q]) = make_uint4(
                    pack2_bf16(Y[ih][8 * hf + 0], Y[ih][8 * hf + 1]), pack2_bf16(Y[ih][8 * hf + 2], Y[ih][8 * hf + 3]),
                    pack2_bf16(Y[ih][8 * hf + 4], Y[ih][8 * hf + 5]), pack2_bf16(Y[ih][8 * hf + 6], Y[ih][8 * hf + 7]));
        if (t.ckpt_slot >= 0) {
            const size_t slot_row = (size_t)t.ckpt_slot * a.H * a.P * kN + state_row;
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    store_state4(a.state_out, slot_row + 32 * nb + 16 * (e >> 1) + 4 * (e & 1),
                                 make_float4(S[nb][4 * e], S[nb][4 * e + 1], S[nb][4 * e + 2], S[nb][4 * e + 3]), ST);
        }
        clear_rows_behind(O.Bs, ld, t_next.len);
        y_tok0 = t.tok0;
        y_len = t.len;
        t = t_next;
        t_next = t_after;
    }
    lds_barrier();
    read_y(L.tile[(p.tile_end - p.tile_begin - 1) & 1]);
    store_y(y_tok0, y_len);
    // read and made again here: what the loop does not need would fill registers there that the rows in flight need
    const int me = ssm_launch_item(blockIdx.x, a.n_items), me_cw = me % a.blocks * kResidentChannels + 32 * w;
    const int ln = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
    const SsmPiece done = a.pieces[me / a.blocks];
    if (done.tile_end < done.stop) {
        float sum = 0.f;  // NaN if one of them is not finite
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                sum = __builtin_fmaf(S[nb][e], 0.f, sum);
        const bool spoiled = __any(sum != 0.f);
        const int own = done.first + done.part;
        if (ln == 0)
            a.spoiled[(size_t)own * (a.H * a.P / 32) + me_cw / 32] = spoiled;
        if (spoiled) {
            float4 *out = a.spoil + carry_at(a, own, me_cw) + ln;
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    out[(4 * nb + e) * 64] = make_float4(S[nb][4 * e], S[nb][4 * e + 1], S[nb][4 * e + 2], S[nb][4 * e + 3]);
        }
    }
}

// ================================================================ states that are updated in place
// One workgroup per (piece, 256 channels), in front of the scan and only for calls whose cached states share memory with the
// checkpoints.  The first piece of a cut sequence reads the cached state while the last one may already write its successor to
// the same place: the first piece takes a copy, in the memory that holds its last state only behind the scan.
template <int ST>
__global__ __launch_bounds__(256) void ssm_keep_states_kernel(ResidentArgs a)
{
    const int item = ssm_launch_item(blockIdx.x, a.n_items);
    if (item < 0)
        return;
    const SsmPiece p = scalar_load(a.pieces + item / a.blocks);
    const void *init = a.init.of(p.seq);
    if (p.part > 0 || p.tile_end == p.stop || !init)
        return;
    constexpr int kBytes = 32 * kN * (ST == SSM_ST_F32 ? 4 : 2);
    const int c0 = item % a.blocks * kResidentChannels;
    for (int u = 0; u < kResidentChannels / 32; ++u) {
        const uint4 *from = reinterpret_cast<const uint4 *>(static_cast<const unsigned char *>(init) + (size_t)(c0 / 32 + u) * kBytes);
        uint4 *to = reinterpret_cast<uint4 *>(a.spoil + carry_at(a, p.first, c0 + 32 * u));
        for (int m = threadIdx.x; m < kBytes / 16; m += 256)
            to[m] = from[m];
    }
}

// ================================================================ values that are not finite
// One workgroup per (piece, 256 channels).  A state element that is infinite or NaN stays so, but a piece starts without what
// has decayed.  Where an earlier piece of the sequence ended with such elements, they are added to the piece's checkpoints
// and, through C, to its outputs; where the piece started with them, that changes nothing.  Without any, which is all that
// ever happens with sound inputs, the workgroup reads a flag per earlier piece and 32 channels and leaves: 3 us with the launch
// (32768 tokens of 16 heads 81 -> 84 us).  To look for such elements in the segments instead would mean to read all of x and B
// a second time.
constexpr int kRestThreads = 256;
struct RestLds {
    float P[32][kN];  // the elements that are not finite, else 0
    int any[kResidentChannels / 32];
};
template <int ST>
__global__ __launch_bounds__(kRestThreads) void ssm_not_finite_kernel(ResidentArgs a)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    RestLds &L = *reinterpret_cast<RestLds *>(lds_raw);
    const int item = ssm_launch_item(blockIdx.x, a.n_items), tid = threadIdx.x;
    if (item < 0)
        return;
    const SsmPiece p = scalar_load(a.pieces + item / a.blocks);
    if (p.part == 0)
        return;
    const int c0 = item % a.blocks * kResidentChannels, groups = a.H * a.P / 32;
    constexpr int kGroups = kResidentChannels / 32;
    auto spoiled = [&](int m, int u) { return a.spoiled[(size_t)(p.first + m) * groups + c0 / 32 + u]; };
    static_assert(kGroups == 8, "two words of four flags");
    int seen[kGroups] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int m = tid; m < p.part; m += kRestThreads) {
        const int4 *f = reinterpret_cast<const int4 *>(a.spoiled + (size_t)(p.first + m) * groups + c0 / 32);
        const int4 lo = f[0], hi = f[1];
        seen[0] |= lo.x, seen[1] |= lo.y, seen[2] |= lo.z, seen[3] |= lo.w;
        seen[4] |= hi.x, seen[5] |= hi.y, seen[6] |= hi.z, seen[7] |= hi.w;
    }
    if (tid < kGroups)
        L.any[tid] = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kGroups; ++u)
        if (seen[u])
            L.any[u] = 1;
    __syncthreads();
    const bf16_t *C = a.C + (size_t)(c0 / (a.H / a.G * a.P)) * kN;
    const SsmTile begin = scalar_load(a.tiles + p.tile_begin), end = scalar_load(a.tiles + p.tile_end - 1);
    for (int u = 0; u < kGroups; ++u) {
        if (!L.any[u])
            continue;  // the whole workgroup
        const int cw = c0 + 32 * u;
        for (int m = tid; m < 16 * 64; m += kRestThreads) {
            const int lane = m & 63, nb = m >> 8, e = (m >> 6) & 3;
            float sum[4] = {0.f, 0.f, 0.f, 0.f};
            for (int k = 0; k < p.part; ++k)
                if (spoiled(k, u)) {
                    const float4 v = a.spoil[carry_at(a, p.first + k, cw) + m];
                    const float vs[4] = {v.x, v.y, v.z, v.w};
                    for (int r = 0; r < 4; ++r)
                        sum[r] += vs[r] * 0.f != 0.f ? vs[r] : 0.f;
                }
            for (int r = 0; r < 4; ++r)
                L.P[operand_index(lane & 31)][32 * nb + 16 * (e >> 1) + 4 * (e & 1) + 8 * (lane >> 5) + r] = sum[r];
        }
        __syncthreads();
        const int ch = tid & 31;
        for (int tok = begin.tok0 + (tid >> 5); tok < end.tok0 + end.len; tok += kRestThreads / 32) {
            float sum = 0.f;
            for (int n = 0; n < kN; ++n)
                if (L.P[ch][n] != 0.f)
                    sum += L.P[ch][n] * bf16_to_f32(C[(size_t)tok * a.G * kN + n]);
            bf16_t *y = a.y + (size_t)tok * a.H * a.P + cw + ch;
            if (sum != 0.f)
                *y = f32_to_bf16(bf16_to_f32(*y) + sum);
        }
        for (int k = p.tile_begin; k < p.tile_end; ++k) {
            const int slot = a.tiles[k].ckpt_slot;
            if (slot < 0)
                continue;
            for (int m = tid; m < 32 * kN; m += kRestThreads) {
                const size_t at = ((size_t)slot * a.H * a.P + cw) * kN + m;
                if ((&L.P[0][0])[m] != 0.f)
                    state_store(a.state_out, at, state_load(a.state_out, at, ST) + (&L.P[0][0])[m], ST);
            }
        }
        __syncthreads();
    }
}

template <int ST>
hipError_t launch_resident_st(const ssm_plan *plan, ResidentArgs a, const SsmPiece *d_pieces, hipStream_t stream)
{
    static std::once_flag attr_once[64];
    static hipError_t attr_err[64];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return e;
    if (dev < 0 || dev >= 64)
        return hipErrorInvalidDevice;
    std::call_once(attr_once[dev], [&]() {
        attr_err[dev] = hipFuncSetAttribute(reinterpret_cast<const void *>(ssm_scan_resident_kernel<ST>),
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(ResidentLds));
    });
    if (attr_err[dev] != hipSuccess)
        return attr_err[dev];
    if (a.kept) {
        a.pieces = d_pieces;
        a.n_items = plan->n_pieces * a.blocks;
        hipLaunchKernelGGL(ssm_keep_states_kernel<ST>, dim3((unsigned)ssm_launch_blocks(a.n_items)), dim3(256), 0, stream, a);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    if (plan->n_segments > 0) {
        a.pieces = d_pieces + plan->n_pieces;
        a.n_items = plan->n_segments * a.blocks;
        hipLaunchKernelGGL(ssm_segment_state_kernel<ST>, dim3((unsigned)ssm_launch_blocks(a.n_items)), dim3(kThreads),
                           sizeof(SegmentLds), stream, a);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    if (plan->n_groups > 0) {
        hipLaunchKernelGGL(ssm_group_states_kernel, dim3((unsigned)plan->n_groups * (unsigned)(a.H * a.P / 32)),
                           dim3(kGroupThreads), 0, stream, a);
        if ((e = hipGetLastError()) != hipSuccess)
            return e;
    }
    if (hipEvent_t mark = ssm_profile_event(0))
        if ((e = hipEventRecord(mark, stream)) != hipSuccess)
            return e;
    a.pieces = d_pieces;
    a.n_items = plan->n_pieces * a.blocks;
    hipLaunchKernelGGL(ssm_scan_resident_kernel<ST>, dim3((unsigned)ssm_launch_blocks(a.n_items)), dim3(kThreads),
                       sizeof(ResidentLds), stream, a);
    if ((e = hipGetLastError()) != hipSuccess)
        return e;
    if (hipEvent_t mark = ssm_profile_event(1))
        if ((e = hipEventRecord(mark, stream)) != hipSuccess)
            return e;
    if (plan->n_continued > 0) {
        hipLaunchKernelGGL(ssm_not_finite_kernel<ST>, dim3((unsigned)ssm_launch_blocks(a.n_items)), dim3(kRestThreads),
                           sizeof(RestLds), stream, a);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace

hipError_t launch_scan_resident(const ssm_plan *plan, const ScanArgs &args, const SsmPiece *d_pieces, void *workspace,
                                hipStream_t stream)
{
    if (plan->n_pieces == 0)
        return hipSuccess;
    ResidentArgs a;
    a.x = static_cast<const bf16_t *>(args.x);
    a.dt = static_cast<const bf16_t *>(args.dt);
    a.B = static_cast<const bf16_t *>(args.B);
    a.C = static_cast<const bf16_t *>(args.C);
    a.A = args.A;
    a.D = args.D;
    a.y = static_cast<bf16_t *>(args.y);
    a.state_out = args.state_out;
    a.init = state_ptrs_of(args.init_ptrs, args.host_ptrs, args.n_host_ptrs);
    a.tiles = args.tiles;
    const SsmPieceWorkspace w = ssm_piece_workspace(plan);
    unsigned char *base = static_cast<unsigned char *>(workspace);
    a.carry = reinterpret_cast<float4 *>(base);
    a.spoil = reinterpret_cast<float4 *>(base + w.spoil);
    a.decay = reinterpret_cast<float *>(base + w.decay);
    a.spoiled = reinterpret_cast<int *>(base + w.spoiled);
    a.H = args.H;
    a.P = args.P;
    a.G = args.G;
    a.blocks = args.H * args.P / kResidentChannels;
    a.n_items = 0;
    a.n_segments = plan->n_segments;
    a.n_groups = plan->n_groups;
    a.kept = args.states_overlap && plan->n_continued > 0 && (args.init_ptrs || args.host_ptrs);
    a.pieces = nullptr;
    switch (args.state_dtype) {
    case SSM_ST_F16: return launch_resident_st<SSM_ST_F16>(plan, a, d_pieces, stream);
    case SSM_ST_BF16: return launch_resident_st<SSM_ST_BF16>(plan, a, d_pieces, stream);
    default: return launch_resident_st<SSM_ST_F32>(plan, a, d_pieces, stream);
    }
}
