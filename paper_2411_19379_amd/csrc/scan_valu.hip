// fp32 scan kernels: f32 or bf16 storage, all arithmetic in fp32 (decay exponents summed in fp64).  They are the path of
// the fp32 mode, of the shapes the fp16 / bf16 matrix-core kernel does not cover, and of the roll-forward over more
// than a few tokens.
//
// All work tile by tile; per tile of q tokens (at most 16, or 32 for the split operands) starting after token s, with
// l_i = A * sum_{k<=i} dt_k inside the tile:
//
//   y_i  = e^{l_i} (S_s C_i) + sum_{j<=i} (C_i.B_j) e^{l_i-l_j} dt_j x_j + D x_i
//   S_e  = e^{l_q} S_s + sum_j e^{l_q-l_j} dt_j x_j B_j^T
//
// which is the token recurrence of ssm_prefill.h unrolled over the tile.  Where d_state is 16, 32, 64 or 128 and headdim
// a multiple of 16 the contractions run on the matrix cores: with fp32 instructions for f32 storage (ssm_scan_f32_kernel),
// with bf16 ones on split operands for bf16 storage (ssm_scan_split_kernel, units of 32 tokens).  Any other shape takes
// the vector ALUs (ssm_scan_valu_kernel).
#include "device_utils.h"

namespace {

// ================================================================ matrix cores, fp32
// One workgroup per (sequence, head, NC slices of 16 channels); its waves take the sequence's tiles of 16 tokens
// round-robin and each computes all of its tile with v_mfma_f32_16x16x4_f32.  The running state lives in LDS and goes
// from the wave of tile k - 1 to the wave of tile k; a counter says how many tiles have left their state there, and
// that hand-off (wait, read, multiply-add, write, publish) is the only thing that orders the waves: no barrier in the
// loop, the tile-local state is complete before a wave starts to wait, and NW tiles are in flight per workgroup.
//
// Layouts.  With kq = lane / 16 and li = lane % 16, an operand holds (row or column li, k = kq), a result element r
// (row 4 kq + r, column li).  The three contractions are ordered so that what one leaves in its result registers is
// what the next wants as an operand, with the k index permuted the same way on both sides:
//   S^T[n, ch] += B^T[n, tok] (w x)[tok, ch]      row i of block nb is state index NB i + nb
//   Gm^T[j, i]  = B[j, n] C^T[n, i]               result r: key token 4 kq + r, query token li
//   Y[i, ch]    = C[i, n] S^T[n, ch] + Gm[i, j] x[j, ch]
// so a lane reads B and C as runs of NB or 4 NB neighbouring state indices straight from device memory, x once for
// all its uses, and nothing passes through LDS but the state and three 16-entry tables of decay factors.
//
// What bounds it: the matrix cores, whose fp32 rate is a sixteenth of their bf16 one (NC (8 NB + 4) + 4 NB products of
// 32 cycles per tile; the 4 NB of the scores are the same for every slice, hence NC > 1), and the chain of hand-offs.
// Against the vector-ALU kernel below (one workgroup per head, five barriers per 16 tokens, dot products from LDS), per
// call: 80 heads x 64 channels, d_state 128, 2048 tokens 8180 -> 141 us; 4 heads x 16 channels, d_state 16, 256 tokens
// 64 -> 12 us.
constexpr int kF32SpinLimit = 1 << 16;  // polls of the hand-off counter before a wave gives up waiting (milliseconds)
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((address_space(3))) int lds_int_t;

// Wait for this wave's own LDS traffic (LDS executes a wave's accesses in order).
__device__ __forceinline__ void lds_wait()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// The hand-off counter is an LDS word read and written with DS instructions (through a generic pointer the accesses
// would be FLAT and wait for outstanding loads from device memory too).  The wait is bounded: every wave ends.
__device__ __forceinline__ void f32_wait_counter(const int *counter, int want)
{
    const volatile lds_int_t *c = (const volatile lds_int_t *)counter;
    int polls = 0;
    while (__builtin_amdgcn_readfirstlane(*c) < want) {
        if (++polls > kF32SpinLimit)
            break;
        __builtin_amdgcn_s_sleep(1);
    }
    asm volatile("" ::: "memory");  // what follows in the source reads LDS after the counter
}
__device__ __forceinline__ void f32_publish_counter(int *counter, int value, int lane)
{
    asm volatile("" ::: "memory");  // LDS executes a wave's accesses in order
    if (lane == 0)
        *(volatile lds_int_t *)counter = value;
}

struct F32Args {
    const void *x, *dt, *B, *C;
    const float *A, *D;
    void *y;                        // may be null (roll-forward without outputs)
    void *state_out;                // [n_ckpt,H,P,N] in the state type (scan)
    StatePtrs init;                 // [batch]: the states the scan starts from, or those the roll-forward advances
    bool roll;                      // roll-forward in place
    const SsmTile *tiles;
    const SsmSeq *seqs;
    const int32_t *order;           // the launch's k-th sequence is order[first + k]; null: first + k
    int first;
    int H, P, G, slices, state_dtype;
};

// NV values (a multiple of 4, or 1 or 2); p is aligned to the run's size, at most 16 bytes
template <int NV> __device__ __forceinline__ void load_run(const float *p, float *v)
{
    if (NV == 1) {
        v[0] = *p;
    } else if (NV == 2) {
        const float2 f = *reinterpret_cast<const float2 *>(p);
        v[0] = f.x, v[1] = f.y;
    } else {
#pragma unroll
        for (int e = 0; e < NV; e += 4) {
            const float4 f = *reinterpret_cast<const float4 *>(p + e);
            v[e] = f.x, v[e + 1] = f.y, v[e + 2] = f.z, v[e + 3] = f.w;
        }
    }
}
// Four neighbouring elements of a cached state (index a multiple of four).
typedef __attribute__((ext_vector_type(4))) _Float16 st_f16x4;
__device__ __forceinline__ float4 state_load4(const void *base, size_t idx, int st)
{
    if (st == SSM_ST_F16) {
        const st_f16x4 v = *reinterpret_cast<const st_f16x4 *>(static_cast<const _Float16 *>(base) + idx);
        return make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
    }
    if (st == SSM_ST_BF16) {
        const uint2 u = *reinterpret_cast<const uint2 *>(static_cast<const bf16_t *>(base) + idx);
        return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                           __uint_as_float(u.y & 0xffff0000u));
    }
    return *reinterpret_cast<const float4 *>(static_cast<const float *>(base) + idx);
}
__device__ __forceinline__ void state_store4(void *base, size_t idx, float4 v, int st)
{
    if (st == SSM_ST_F16) {
        const st_f16x4 h = {(_Float16)v.x, (_Float16)v.y, (_Float16)v.z, (_Float16)v.w};
        *reinterpret_cast<st_f16x4 *>(static_cast<_Float16 *>(base) + idx) = h;
    } else if (st == SSM_ST_BF16) {
        *reinterpret_cast<uint2 *>(static_cast<bf16_t *>(base) + idx) =
            make_uint2((uint32_t)f32_to_bf16(v.x) | ((uint32_t)f32_to_bf16(v.y) << 16),
                       (uint32_t)f32_to_bf16(v.z) | ((uint32_t)f32_to_bf16(v.w) << 16));
    } else {
        *reinterpret_cast<float4 *>(static_cast<float *>(base) + idx) = v;
    }
}

#define F32_DPP64(v, ctrl)                                                                                         \
    [&]() {                                                                                                        \
        const uint64_t u_ = __builtin_bit_cast(uint64_t, (double)(v));                                             \
        const uint32_t lo_ = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u_, (ctrl), 0xF, 0xF, true);  \
        const uint32_t hi_ = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(u_ >> 32), (ctrl), 0xF, 0xF, true);    \
        return __builtin_bit_cast(double, ((uint64_t)hi_ << 32) | lo_);                                            \
    }()
// Inclusive prefix sum over each row of 16 lanes.
__device__ __forceinline__ double row_inclusive_sum(double v)
{
    v += F32_DPP64(v, 0x111);
    v += F32_DPP64(v, 0x112);
    v += F32_DPP64(v, 0x114);
    v += F32_DPP64(v, 0x118);
    return v;
}

__device__ __forceinline__ f32x4 mfma_f32(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bool finite(float v) { return __builtin_fabsf(v) < __builtin_inff(); }

struct F32Wave {          // private to one wave
    double ell[16];       // l_i
    float ei[16];         // e^{l_i}
    float wt[16];         // e^{l_q - l_j} dt_j
    float dt[16];
    int first_bad[64];
};
template <int NB, int NC, int NW> struct F32Lds {
    float4 S[NC][NB][64];  // [slice][four of a lane's 4 NB state elements][lane]
    int done;
    int pad[3];
    F32Wave wv[NW];
};

// Waves per SIMD: what the registers of the common path leave room for (the paths for values that are not finite would
// take a wave away).
constexpr int f32_waves_per_simd(int nb, int nc)
{
    return nb == 8 ? 2 : nb * nc == 8 ? 3 : nb * nc == 4 ? 4 : 5;
}
template <int NB, int NC, int NW>
__global__ __launch_bounds__(64 * NW, f32_waves_per_simd(NB, NC)) void ssm_scan_f32_kernel(F32Args a)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    F32Lds<NB, NC, NW> &L = *reinterpret_cast<F32Lds<NB, NC, NW> *>(lds_raw);
    constexpr int N = 16 * NB;
    const int H = a.H, P = a.P, G = a.G, st = a.state_dtype;
    const int slice = blockIdx.x % a.slices;
    const int h = (blockIdx.x / a.slices) % H;
    const int rank = a.first + (int)(blockIdx.x / (unsigned)(a.slices * H)), seq = a.order ? a.order[rank] : rank;
    const int g = h / (H / G);
    const int lane = threadIdx.x & 63, li = lane & 15, kq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool roll = a.roll;
    const SsmSeq sq = a.seqs[seq];
    const void *from = a.init.of(seq);
    if (sq.tile_end <= sq.tile_begin || (roll && !from))
        return;  // nothing to scan; the whole workgroup leaves
    // The scan takes the plan's tiles, which end at checkpoints; the roll-forward knows no checkpoints and cuts the
    // sequence's tokens itself.
    int tok_begin = 0, n_tok = 0, n_tiles = sq.tile_end - sq.tile_begin;
    if (roll) {
        const SsmTile last = a.tiles[sq.tile_end - 1];
        tok_begin = a.tiles[sq.tile_begin].tok0;
        n_tok = last.tok0 + last.len - tok_begin;
        n_tiles = (n_tok + 15) / 16;
    }
    const float *x = static_cast<const float *>(a.x), *dt = static_cast<const float *>(a.dt);
    const float *Bg = static_cast<const float *>(a.B) + (size_t)g * N, *Cg = static_cast<const float *>(a.C) + (size_t)g * N;
    float *y = static_cast<float *>(a.y);
    const float Ah = a.A[h], Dh = a.D[h];
    // channel li of slice c, state indices 4 NB kq .. 4 NB kq + 4 NB - 1
    const size_t state_row = ((size_t)h * P + 16 * NC * slice + li) * N + 4 * NB * kq;
    const size_t GN = (size_t)G * N, HP = (size_t)H * P;
    const size_t xcol = (size_t)h * P + 16 * NC * slice + li;

    // One wave alone keeps the state in its registers: what it starts from arrives while the first tile is computed.
    float4 sp[NC][NB];
    auto start_at = [&](int c, int f4) {
        return from ? state_load4(from, state_row + (size_t)16 * c * N + 4 * f4, st) : make_float4(0.f, 0.f, 0.f, 0.f);
    };
    if constexpr (NW == 1) {
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int f4 = 0; f4 < NB; ++f4)
                sp[c][f4] = start_at(c, f4);
    } else {
        for (int b = w; b < NC * NB; b += NW)
            L.S[b / NB][b % NB][lane] = start_at(b / NB, b % NB);
        if (threadIdx.x == 0)
            L.done = 0;
        __syncthreads();  // the only one: the starting state and the counter are in place
    }

    F32Wave &W = L.wv[w];
    for (int k = w; k < n_tiles; k += NW) {
        int tok0, len, ckpt = -1;
        if (roll) {
            tok0 = tok_begin + 16 * k;
            len = n_tok - 16 * k < 16 ? n_tok - 16 * k : 16;
        } else {
            const SsmTile t = scalar_load(a.tiles + sq.tile_begin + k);
            tok0 = t.tok0, len = t.len, ckpt = t.ckpt_slot;
        }
        // rows past the end of a partial tile re-read its last row
        const size_t row = (size_t)tok0 + (li < len ? li : len - 1);
        const float dtl = li < len ? dt[row * H + h] : 0.f;
        float Cf[4 * NB], Bf[4 * NB], Bt[4][NB], xv[NC][4];
        load_run<4 * NB>(Bg + row * GN + 4 * NB * kq, Bf);
        load_run<4 * NB>(Cg + row * GN + 4 * NB * kq, Cf);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const size_t tok = (size_t)tok0 + (4 * kq + r < len ? 4 * kq + r : len - 1);
            load_run<NB>(Bg + tok * GN + NB * li, Bt[r]);
#pragma unroll
            for (int c = 0; c < NC; ++c)
                xv[c][r] = x[tok * HP + xcol + 16 * c];
        }
        const double ell = row_inclusive_sum((double)dtl * (double)Ah);  // padded tokens add nothing
        if (lane < 16) {
            W.ell[li] = ell;
            W.dt[li] = dtl;
        }
        lds_wait();
        const double last = W.ell[15];
        if (lane < 16) {
            W.ei[li] = expf((float)ell);
            W.wt[li] = expf((float)(last - ell)) * dtl;
        }
        const float dl = expf((float)last);
        lds_wait();
        const float4 wt4 = *reinterpret_cast<const float4 *>(&W.wt[4 * kq]);
        const float wt[4] = {wt4.x, wt4.y, wt4.z, wt4.w};

        if (len < 16) {  // rows past the end add nothing: their weights are zero, but what was read may not be finite
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const bool in = 4 * kq + r < len;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    Bt[r][nb] = in ? Bt[r][nb] : 0.f;
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    xv[c][r] = in ? xv[c][r] : 0.f;
            }
        }
        f32x4 Sl[NC * NB];  // [slice][block]
#pragma unroll
        for (int c = 0; c < NC * NB; ++c)
            Sl[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    Sl[c * NB + nb] = mfma_f32(Bt[r][nb], wt[r] * xv[c][r], Sl[c * NB + nb]);
        // masked, decayed scores of key 4 kq + r and query li; four partial sums, so that the products do not wait for
        // each other
        float gm[4];
        if (y) {
            f32x4 part[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                part[r] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int f = 0; f < NB; ++f)
                    part[r] = mfma_f32(Bf[r * NB + f], Cf[r * NB + f], part[r]);
            }
            const float4 dt4 = *reinterpret_cast<const float4 *>(&W.dt[4 * kq]);
            const float dtj[4] = {dt4.x, dt4.y, dt4.z, dt4.w};
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float e = expf((float)(ell - W.ell[4 * kq + r])) * dtj[r];
                const float sc = (part[0][r] + part[1][r]) + (part[2][r] + part[3][r]);
                gm[r] = 4 * kq + r <= li ? sc * e : 0.f;
            }
        }
#pragma unroll
        for (int c = 0; c < NC * NB; ++c)  // done before the wait starts
            asm volatile("" : "+v"(Sl[c]));
        // read the state, multiply-add, write it back, publish
        if constexpr (NW > 1) {
            f32_wait_counter(&L.done, k);
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int f4 = 0; f4 < NB; ++f4)
                    sp[c][f4] = L.S[c][f4][lane];
        }
        // element f = NB rr + nb of a lane's run is element rr of block nb
        auto next = [&](int c, int f) {
            const float4 &q = sp[c][f / 4];
            const float s = f % 4 == 0 ? q.x : f % 4 == 1 ? q.y : f % 4 == 2 ? q.z : q.w;
            return __builtin_fmaf(dl, s, Sl[c * NB + f % NB][f / NB]);
        };
        float4 sn[NC][NB];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int f4 = 0; f4 < NB; ++f4) {
                sn[c][f4] = make_float4(next(c, 4 * f4), next(c, 4 * f4 + 1), next(c, 4 * f4 + 2), next(c, 4 * f4 + 3));
                if constexpr (NW > 1)
                    L.S[c][f4][lane] = sn[c][f4];
            }
        if constexpr (NW > 1)
            f32_publish_counter(&L.done, k + 1, lane);
        auto keep_state = [&]() {
            if constexpr (NW == 1)
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int f4 = 0; f4 < NB; ++f4)
                        sp[c][f4] = sn[c][f4];
        };
        if (ckpt >= 0 || (roll && k == n_tiles - 1)) {
            void *to = roll ? const_cast<void *>(from) : a.state_out;
            const size_t at = (roll ? 0 : (size_t)ckpt * HP * N) + state_row;
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int f4 = 0; f4 < NB; ++f4)
                    state_store4(to, at + (size_t)16 * c * N + 4 * f4, sn[c][f4], st);
        }
        if (!y) {
            keep_state();
            continue;
        }
        const float4 ei4 = *reinterpret_cast<const float4 *>(&W.ei[4 * kq]);
        const float ei[4] = {ei4.x, ei4.y, ei4.z, ei4.w};
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            f32x4 Y0 = f32x4{0.f, 0.f, 0.f, 0.f}, Y1 = Y0;
#pragma unroll
            for (int f4 = 0; f4 < NB; ++f4) {
                Y0 = mfma_f32(Cf[4 * f4 + 0], sp[c][f4].x, Y0);
                Y1 = mfma_f32(Cf[4 * f4 + 1], sp[c][f4].y, Y1);
                Y0 = mfma_f32(Cf[4 * f4 + 2], sp[c][f4].z, Y0);
                Y1 = mfma_f32(Cf[4 * f4 + 3], sp[c][f4].w, Y1);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                Y0[r] = ei[r] * (Y0[r] + Y1[r]);
            const f32x4 before = Y0;
#pragma unroll
            for (int r = 0; r < 4; ++r)
                Y0 = mfma_f32(gm[r], xv[c][r], Y0);
            // a token whose x is not finite has reached every query of its channel, the earlier ones as 0 * inf: these
            // take the products without such tokens (between two such tokens of a tile an infinity becomes NaN)
            if (__builtin_expect(__any(!finite(Y0[0])), 0)) {
                int first = 16;
                f32x4 Y2 = before;
#pragma unroll
                for (int r = 3; r >= 0; --r)
                    first = !finite(xv[c][r]) ? 4 * kq + r : first;
                W.first_bad[lane] = first;
                lds_wait();
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    first = W.first_bad[16 * q + li] < first ? W.first_bad[16 * q + li] : first;
                lds_wait();
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    Y2 = mfma_f32(gm[r], finite(xv[c][r]) ? xv[c][r] : 0.f, Y2);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    Y0[r] = 4 * kq + r < first ? Y2[r] : Y0[r];
            }
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * kq + r < len)
                    y[((size_t)tok0 + 4 * kq + r) * HP + xcol + 16 * c] = __builtin_fmaf(Dh, xv[c][r], Y0[r]);
        }
        keep_state();
    }
}

// ================================================================ matrix cores, bf16 storage: split operands
// The same scan for bf16 x, dt, B, C and y.  B, C and x are bf16 already, so of every product only one factor is a
// 32-bit value (the decay-weighted x, the masked scores, the state), and a 32-bit value is exactly the sum of three
// bf16 ones (8 + 8 + 8 bits of its significand).  Three v_mfma_f32_16x16x32_bf16 therefore give the same products
// added up in fp32 as the fp32 instruction does, in 3/16 of its time, and the scores C.B take a single one.  Against
// 64 bits it is no further off than the fp32 instruction was.
//
// One workgroup per (sequence, head, NC slices of 16 channels); its waves take units of 32 tokens round-robin and each
// computes all of its unit, the state handed from wave to wave through LDS as in the fp32 kernel above.  A unit is a tile
// of the plan; the roll-forward cuts the sequence's tokens itself.
//
// Layouts (kq = lane / 16, li = lane % 16; an operand holds row or column li, k = 8 kq + e; a result element r is row
// 4 kq + r, column li).  Any order of the k index will do as long as both operands use the same one, so every operand is
// read from device memory in runs of neighbouring elements and what one product leaves in its result registers is what
// the next takes as an operand; nothing passes through LDS but the state and the tables of decay factors:
//   tokens     slot (kq, e) is token 16 (e / 4) + 4 kq + e % 4: the tokens whose results the lane holds
//   state      slot (kq, f) is state index 4 NB kq + f; row i of result block nb is state index NB i + nb
//   channels   column i of slice c is channel NC i + c of the workgroup's 16 NC
// With d_state 16 a lane holds four state indices per product and the other four slots take the second part of the
// split; the first 16 queries of a unit have only 16 keys and do the same.
//
// What bounds it: the vector ALUs that split and mask (counters: three to four times the cycles of the products).  Per call, this
// kernel against the fp32 instruction on the same storage: 32 heads x 64 channels, d_state 16, eight requests of 18 K
// tokens in all, 107 -> 67 us; roll-forward of three sequences of 17 to 256 tokens, 128 heads x 64 channels, d_state 128,
// 52 -> 35 us.
constexpr int kUnit = 32;
typedef __attribute__((ext_vector_type(8))) __bf16 split_bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 split_bf16x2;
typedef __attribute__((ext_vector_type(2))) float split_f32x2;
typedef __attribute__((ext_vector_type(2))) uint32_t split_u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t split_u32x4;

__device__ __forceinline__ f32x4 mfma_b16(uint4 a, uint4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(split_bf16x8, a), __builtin_bit_cast(split_bf16x8, b),
                                                   c, 0, 0, 0);
}
__device__ __forceinline__ uint32_t split_pack(float lo, float hi)  // two floats rounded to bf16
{
    const split_f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, split_bf16x2));
}
// the upper 16 bits of two words, the lower 16 bits of two words
__device__ __forceinline__ uint32_t upper2(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }
__device__ __forceinline__ uint32_t lower2(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x05040100u); }

// Two fp32 values as three pairs of bf16 whose sums they are: cut off after 8 bits of the significand, twice.
__device__ __forceinline__ void split3(float a, float b, uint32_t (&part)[3])
{
#pragma unroll
    for (int s = 0; s < 3; ++s) {
        const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
        part[s] = upper2(ua, ub);
        a -= __uint_as_float(ua & 0xffff0000u);
        b -= __uint_as_float(ub & 0xffff0000u);
    }
}
__device__ __forceinline__ void split3x8(const float (&v)[8], uint4 (&part)[3])
{
    uint32_t p[4][3];
#pragma unroll
    for (int d = 0; d < 4; ++d)
        split3(v[2 * d], v[2 * d + 1], p[d]);
#pragma unroll
    for (int s = 0; s < 3; ++s)
        part[s] = make_uint4(p[0][s], p[1][s], p[2][s], p[3][s]);
}

// Loads go through buffer descriptors: a uniform base and size, one 32-bit offset per lane and a uniform offset, so that
// no 64-bit address arithmetic runs on the vector ALUs.  Every access stays inside its descriptor.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t split_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}
// BYTES (2, 4, 8, or a multiple of 16) neighbouring bytes as words
template <int BYTES>
__device__ __forceinline__ void load_words(__amdgpu_buffer_rsrc_t r, uint32_t lane_off, uint32_t uniform_off, uint32_t *v)
{
    if (BYTES == 2) {
        v[0] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, (int)lane_off, (int)uniform_off, 0);
    } else if (BYTES == 4) {
        v[0] = __builtin_amdgcn_raw_buffer_load_b32(r, (int)lane_off, (int)uniform_off, 0);
    } else if (BYTES == 8) {
        const auto u = __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane_off, (int)uniform_off, 0);
        v[0] = u[0], v[1] = u[1];
    } else {
#pragma unroll
        for (int e = 0; e < BYTES / 16; ++e) {
            const auto u = __builtin_amdgcn_raw_buffer_load_b128(r, (int)(lane_off + 16 * e), (int)uniform_off, 0);
            v[4 * e] = u[0], v[4 * e + 1] = u[1], v[4 * e + 2] = u[2], v[4 * e + 3] = u[3];
        }
    }
}

// Four neighbouring elements of a cached state behind a descriptor (lane offset in elements), ST its storage type.
template <int ST> __device__ __forceinline__ float4 split_state_load4(__amdgpu_buffer_rsrc_t r, uint32_t elem)
{
    uint32_t u[4];
    if constexpr (ST == SSM_ST_F32) {
        load_words<16>(r, 4 * elem, 0, u);
        return make_float4(__uint_as_float(u[0]), __uint_as_float(u[1]), __uint_as_float(u[2]), __uint_as_float(u[3]));
    }
    load_words<8>(r, 2 * elem, 0, u);
    if constexpr (ST == SSM_ST_F16) {
        const st_f16x4 v = __builtin_bit_cast(st_f16x4, make_uint2(u[0], u[1]));
        return make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
    }
    return make_float4(__uint_as_float(u[0] << 16), __uint_as_float(u[0] & 0xffff0000u), __uint_as_float(u[1] << 16),
                       __uint_as_float(u[1] & 0xffff0000u));
}
template <int ST> __device__ __forceinline__ void split_state_store4(__amdgpu_buffer_rsrc_t r, uint32_t elem, float4 v)
{
    if constexpr (ST == SSM_ST_F32) {
        const split_u32x4 u = {__float_as_uint(v.x), __float_as_uint(v.y), __float_as_uint(v.z), __float_as_uint(v.w)};
        __builtin_amdgcn_raw_buffer_store_b128(u, r, (int)(4 * elem), 0, 0);
    } else if constexpr (ST == SSM_ST_F16) {
        const st_f16x4 h = {(_Float16)v.x, (_Float16)v.y, (_Float16)v.z, (_Float16)v.w};
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(split_u32x2, h), r, (int)(2 * elem), 0, 0);
    } else {
        const split_u32x2 u = {split_pack(v.x, v.y), split_pack(v.z, v.w)};
        __builtin_amdgcn_raw_buffer_store_b64(u, r, (int)(2 * elem), 0, 0);
    }
}

struct SplitWave {        // private to one wave
    double ell[kUnit];    // l_i log2(e)
    float ei[kUnit];      // e^{l_i}
    float wt[kUnit];      // e^{l_q - l_j} dt_j
    float dt[kUnit];
    int first_bad[64];
};
__device__ __forceinline__ const void *uniform_ptr(const void *p)
{
    const uint64_t u = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<const void *>(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(u >> 32)) << 32) |
                                          (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u));
}
template <int T> struct StateType {
    static constexpr int value = T;
};
template <int NB, int NC, int NW> struct SplitLds {
    float4 S[NC][NB][64];  // [slice][four of a lane's 4 NB state elements][lane]
    int done;
    int pad[3];
    SplitWave wv[NW];
};

// Waves per SIMD: what the registers of the common path leave room for.  Without the bound the paths for values that are
// not finite, which are all but never taken, would cost a wave (64 heads x 32 channels, d_state 16: 1.1 to 1.5 times the
// time); with it they spill a few registers of their own.
constexpr int split_waves_per_simd(int nb, int nc, int nw)
{
    return nb * nc <= 2 ? (nc == 2 && nw == 1 ? 3 : 4) : nb * nc == 4 && nc < 4 ? 3 : 2;
}
template <int NB, int NC, int NW>
__global__ __launch_bounds__(64 * NW, split_waves_per_simd(NB, NC, NW)) void ssm_scan_split_kernel(F32Args a)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    SplitLds<NB, NC, NW> &L = *reinterpret_cast<SplitLds<NB, NC, NW> *>(lds_raw);
    constexpr int N = 16 * NB, kRun = 4 * NB;          // d_state; state indices per lane
    constexpr int kSteps = NB == 1 ? 1 : NB / 2;       // products over the state indices, 32 at a time
    constexpr int kRowWords = kRun / 2;                // words of a lane's run of a row of B or C
    constexpr int kBtWords = NB == 1 ? 1 : NB / 2, kXWords = NC == 4 ? 2 : 1;
    const int H = a.H, P = a.P, G = a.G, st = a.state_dtype;
    const int slice = blockIdx.x % a.slices;
    const int h = (blockIdx.x / a.slices) % H;
    const int rank = a.first + (int)(blockIdx.x / (unsigned)(a.slices * H)), seq = a.order ? a.order[rank] : rank;
    const int g = h / (H / G);
    const int lane = threadIdx.x & 63, li = lane & 15, kq = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool roll = a.roll;
    const SsmSeq sq = a.seqs[seq];
    const void *from = uniform_ptr(a.init.of(seq));
    if (sq.tile_end <= sq.tile_begin || (roll && !from))
        return;  // nothing to scan; the whole workgroup leaves
    int tok_begin = 0, n_tok = 0, n_units = sq.tile_end - sq.tile_begin;
    if (roll) {
        const SsmTile last = a.tiles[sq.tile_end - 1];
        tok_begin = a.tiles[sq.tile_begin].tok0;
        n_tok = last.tok0 + last.len - tok_begin;
        n_units = (n_tok + kUnit - 1) / kUnit;
    }
    const unsigned char *x = static_cast<const unsigned char *>(a.x) + ((size_t)h * P + 16 * NC * slice) * 2;
    const unsigned char *Bg = static_cast<const unsigned char *>(a.B) + (size_t)g * N * 2;
    const unsigned char *Cg = static_cast<const unsigned char *>(a.C) + (size_t)g * N * 2;
    const bf16_t *dt = static_cast<const bf16_t *>(a.dt) + h;
    unsigned char *y = a.y ? static_cast<unsigned char *>(a.y) + ((size_t)h * P + 16 * NC * slice) * 2 : nullptr;
    const float Ah = a.A[h], Dh = a.D[h];
    const uint32_t gn_b = (uint32_t)G * N * 2, hp_b = (uint32_t)H * P * 2;  // bytes per token row
    // the workgroup's part of a cached state; the lane's: channel NC li + c, state indices 4 NB kq .. 4 NB kq + 4 NB - 1
    const size_t part_elem = ((size_t)h * P + 16 * NC * slice) * N;
    const int st_bytes = st == SSM_ST_F32 ? 4 : 2;
    const uint32_t lane_elem = NC * li * N + kRun * kq;
    auto state_part = [&](const void *base, size_t elem) {
        return split_rsrc(static_cast<const unsigned char *>(base) + (elem + part_elem) * st_bytes,
                          16u * NC * N * (uint32_t)st_bytes);
    };

    // operand of product s from a lane's run of a row; with d_state 16 the run fills four slots and `rest` the others
    auto row_operand = [&](const uint32_t (&r)[kRowWords], int s, bool twice) {
        if constexpr (NB == 1)
            return make_uint4(r[0], r[1], twice ? r[0] : 0u, twice ? r[1] : 0u);
        else
            return make_uint4(r[4 * s], r[4 * s + 1], r[4 * s + 2], r[4 * s + 3]);
    };

    // One wave alone keeps the state in its registers: what it starts from arrives while the first unit is computed.
    float4 sp[NC][NB];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int f4 = 0; f4 < NB; ++f4)
            sp[c][f4] = make_float4(0.f, 0.f, 0.f, 0.f);
    auto start_from = [&](auto type) {
        const __amdgpu_buffer_rsrc_t part = state_part(from, 0);
        if constexpr (NW == 1) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int f4 = 0; f4 < NB; ++f4)
                    sp[c][f4] = split_state_load4<decltype(type)::value>(part, lane_elem + c * N + 4 * f4);
            return;
        }
        for (int b = w; b < NC * NB; b += NW)
            L.S[b / NB][b % NB][lane] = split_state_load4<decltype(type)::value>(part, lane_elem + b / NB * N + 4 * (b % NB));
    };
    if (!from) {
        for (int b = w; NW > 1 && b < NC * NB; b += NW)
            L.S[b / NB][b % NB][lane] = make_float4(0.f, 0.f, 0.f, 0.f);
    } else if (st == SSM_ST_F32) {
        start_from(StateType<SSM_ST_F32>());
    } else if (st == SSM_ST_F16) {
        start_from(StateType<SSM_ST_F16>());
    } else {
        start_from(StateType<SSM_ST_BF16>());
    }
    if constexpr (NW > 1) {
        if (threadIdx.x == 0)
            L.done = 0;
        __syncthreads();  // the only one: the starting state and the counter are in place
    }

    SplitWave &W = L.wv[w];
    for (int k = w; k < n_units; k += NW) {
        int tok0, len, ckpt = -1;
        if (roll) {
            tok0 = tok_begin + kUnit * k;
            len = n_tok - kUnit * k < kUnit ? n_tok - kUnit * k : kUnit;
        } else {
            const SsmTile t = scalar_load(a.tiles + sq.tile_begin + k);
            tok0 = t.tok0, len = t.len, ckpt = t.ckpt_slot;
        }
        tok0 = __builtin_amdgcn_readfirstlane(tok0);
        len = __builtin_amdgcn_readfirstlane(len);
        ckpt = __builtin_amdgcn_readfirstlane(ckpt);
        // ---- the unit's operands as they come from device memory.  Rows past the end of a partial unit re-read its last
        // row: their weights are zero, and an x there that is not finite is treated like the last token's own.
        float dtl;
        uint32_t Cr[2][kRowWords], Br[2][kRowWords], Bt[8][kBtWords], xr[8][kXWords];
        {
            const uint32_t rows = (uint32_t)(len - 1);
            const __amdgpu_buffer_rsrc_t xs = split_rsrc(x + (size_t)tok0 * hp_b, rows * hp_b + 32 * NC);
            const __amdgpu_buffer_rsrc_t bs = split_rsrc(Bg + (size_t)tok0 * gn_b, rows * gn_b + 2 * N);
            const __amdgpu_buffer_rsrc_t cs = split_rsrc(Cg + (size_t)tok0 * gn_b, rows * gn_b + 2 * N);
            const __amdgpu_buffer_rsrc_t ds = split_rsrc(dt + (size_t)tok0 * H, (rows * H + 1) * 2);
            // row (own row of the lane) + up, at most the last one: a uniform part and a part per lane
            auto up_at = [&](uint32_t up, uint32_t stride) { return up < rows ? up * stride : rows * stride; };
            auto own_at = [&](uint32_t own, uint32_t up, uint32_t stride) {
                const uint32_t most = rows * stride - up_at(up, stride);
                return own < most ? own : most;
            };
            const int dt_tok = lane & (kUnit - 1);
            const uint32_t dt_raw = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(
                ds, (int)own_at(dt_tok * 2u * H, 0, 2u * H), 0, 0);
            dtl = dt_tok < len ? __uint_as_float(dt_raw << 16) : 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t up = 16 * (e >> 2) + (e & 3);
                load_words<2 * NC>(xs, own_at(4 * kq * hp_b, up, hp_b) + 2 * NC * li, up_at(up, hp_b), xr[e]);
                load_words<2 * NB>(bs, own_at(4 * kq * gn_b, up, gn_b) + 2 * NB * li, up_at(up, gn_b), Bt[e]);
            }
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const uint32_t own = own_at(li * gn_b, 16 * hf, gn_b) + 2 * kRun * kq;
                load_words<2 * kRun>(bs, own, up_at(16 * hf, gn_b), Br[hf]);
                load_words<2 * kRun>(cs, own, up_at(16 * hf, gn_b), Cr[hf]);
            }
        }
        // ---- decay factors.  Lanes 32..63 repeat lanes 0..31.
        float dl;
        {
            const double half = row_inclusive_sum((double)dtl * (double)Ah);  // tokens past the end add nothing
            const uint64_t u = __builtin_bit_cast(uint64_t, half);
            const uint64_t u15 = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(u >> 32), 15) << 32) |
                                 (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, 15);
            const double ell = 1.4426950408889634074 * (half + ((lane & 16) ? __builtin_bit_cast(double, u15) : 0.0));
            const uint64_t v = __builtin_bit_cast(uint64_t, ell);
            const uint64_t v31 = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), 31) << 32) |
                                 (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 31);
            const double last = __builtin_bit_cast(double, v31);
            dl = __builtin_amdgcn_exp2f((float)last);
            if (lane < kUnit) {
                W.ell[lane] = ell;
                W.dt[lane] = dtl;
                W.ei[lane] = __builtin_amdgcn_exp2f((float)ell);
                W.wt[lane] = __builtin_amdgcn_exp2f((float)(last - ell)) * dtl;
            }
        }
        lds_wait();
        // channel c of the lane's token e, and the operand of the products with x
        auto xval = [&](int c, int e) {
            const uint32_t u = xr[e][c >> 1];
            return __uint_as_float((c & 1) ? u & 0xffff0000u : u << 16);
        };
        auto xpair = [&](int c, int d) {
            return (c & 1) ? upper2(xr[2 * d][c >> 1], xr[2 * d + 1][c >> 1])
                           : lower2(xr[2 * d][c >> 1], xr[2 * d + 1][c >> 1]);
        };

        __builtin_amdgcn_sched_barrier(0);
        // ---- the unit's own state
        f32x4 Sl[NC * NB];  // [slice][block]
#pragma unroll
        for (int c = 0; c < NC * NB; ++c)
            Sl[c] = f32x4{0.f, 0.f, 0.f, 0.f};
        {
            uint4 bo[NB];
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                uint32_t b[4];
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    b[d] = (nb & 1) ? upper2(Bt[2 * d][nb >> 1], Bt[2 * d + 1][nb >> 1])
                                    : lower2(Bt[2 * d][nb >> 1], Bt[2 * d + 1][nb >> 1]);
                bo[nb] = make_uint4(b[0], b[1], b[2], b[3]);
            }
            const float4 w0 = *reinterpret_cast<const float4 *>(&W.wt[4 * kq]);
            const float4 w1 = *reinterpret_cast<const float4 *>(&W.wt[16 + 4 * kq]);
            const float wt[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                __builtin_amdgcn_sched_barrier(0);
                float v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    v[e] = wt[e] * xval(c, e);
                uint4 wx[3];
                split3x8(v, wx);
#pragma unroll
                for (int s = 2; s >= 0; --s)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        Sl[c * NB + nb] = mfma_b16(bo[nb], wx[s], Sl[c * NB + nb]);
            }
        }
        // A value that is not finite has no split, and times the zero of a part or of a row past the end it is NaN.  In B it
        // has reached every channel, in x every state index of its channel; what it has reached is summed token by token.
        {
            float z = 0.f;
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int nb = 0; nb < (c == 0 ? NB : 1); ++nb)
#pragma unroll
                    for (int rr = 0; rr < (c == 0 ? 4 : 1); ++rr)
                        z = __builtin_fmaf(Sl[c * NB + nb][rr], 0.f, z);
            if (__builtin_expect(__any(z != 0.f), 0)) {
                const __amdgpu_buffer_rsrc_t xs = split_rsrc(x + (size_t)tok0 * hp_b, (uint32_t)(len - 1) * hp_b + 32 * NC);
                const __amdgpu_buffer_rsrc_t bs = split_rsrc(Bg + (size_t)tok0 * gn_b, (uint32_t)(len - 1) * gn_b + 2 * N);
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        __builtin_amdgcn_sched_barrier(0);
                        f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma nounroll
                        for (int j = 0; j < len; ++j) {
                            uint32_t xw, bw;
                            load_words<2>(xs, 2 * NC * li + 2 * c, (uint32_t)j * hp_b, &xw);
                            const float v = W.wt[j] * __uint_as_float(xw << 16);
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                load_words<2>(bs, 2 * kRun * kq + 2 * (NB * r + nb), (uint32_t)j * gn_b, &bw);
                                sum[r] += v * __uint_as_float(bw << 16);
                            }
                        }
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            Sl[c * NB + nb][r] = finite(Sl[c * NB + nb][r]) ? Sl[c * NB + nb][r] : sum[r];
                    }
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // ---- masked, decayed scores as split operands: queries 0..15 have keys 0..15 (two parts share a product),
        // queries 16..31 all of them
        uint4 g_hm, g_l, g_hi[3];
        {
            f32x4 sc[3];  // queries / keys: first / first, second / first, second / second half
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                sc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < kSteps; ++s)
                    sc[b] = mfma_b16(row_operand(Br[b == 2], s, false), row_operand(Cr[b > 0], s, false), sc[b]);
            }
            const double e0 = W.ell[li], e1 = W.ell[16 + li];
            float v0[4], v1[8];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (r == 2)
                    __builtin_amdgcn_sched_barrier(0);
                const double k0 = W.ell[4 * kq + r], k1 = W.ell[16 + 4 * kq + r];
                const float d0 = W.dt[4 * kq + r], d1 = W.dt[16 + 4 * kq + r];
                const bool in = 4 * kq + r <= li;
                v0[r] = in ? sc[0][r] * (__builtin_amdgcn_exp2f((float)(e0 - k0)) * d0) : 0.f;
                v1[r] = sc[1][r] * (__builtin_amdgcn_exp2f((float)(e1 - k0)) * d0);
                v1[4 + r] = in ? sc[2][r] * (__builtin_amdgcn_exp2f((float)(e1 - k1)) * d1) : 0.f;
            }
            uint32_t p[2][3];
            split3(v0[0], v0[1], p[0]);
            split3(v0[2], v0[3], p[1]);
            g_hm = make_uint4(p[0][0], p[1][0], p[0][1], p[1][1]);
            g_l = make_uint4(p[0][2], p[1][2], 0u, 0u);
            split3x8(v1, g_hi);
        }
#pragma unroll
        for (int c = 0; c < NC * NB; ++c)  // done before the wait starts
            asm volatile("" : "+v"(Sl[c]));
        __builtin_amdgcn_sched_barrier(0);
        // ---- read the state, multiply-add, write it back, publish
        if constexpr (NW > 1) {
            f32_wait_counter(&L.done, k);
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int f4 = 0; f4 < NB; ++f4)
                    sp[c][f4] = L.S[c][f4][lane];
        }
        // element f = NB rr + nb of a lane's run is element rr of block nb
        auto next = [&](int c, int f) {
            const float4 &q = sp[c][f / 4];
            const float s = f % 4 == 0 ? q.x : f % 4 == 1 ? q.y : f % 4 == 2 ? q.z : q.w;
            return __builtin_fmaf(dl, s, Sl[c * NB + f % NB][f / NB]);
        };
        auto next4 = [&](int c, int f4) {
            return make_float4(next(c, 4 * f4), next(c, 4 * f4 + 1), next(c, 4 * f4 + 2), next(c, 4 * f4 + 3));
        };
        if constexpr (NW > 1) {
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int f4 = 0; f4 < NB; ++f4)
                    L.S[c][f4][lane] = next4(c, f4);
            __builtin_amdgcn_sched_barrier(0);
            f32_publish_counter(&L.done, k + 1, lane);
        }
        auto keep_state = [&]() {
            if constexpr (NW == 1)
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int f4 = 0; f4 < NB; ++f4)
                        sp[c][f4] = next4(c, f4);
        };
        if (ckpt >= 0 || (roll && k == n_units - 1)) {
            const __amdgpu_buffer_rsrc_t part =
                state_part(roll ? from : a.state_out, roll ? 0 : (size_t)ckpt * H * P * N);
            auto keep = [&](auto type) {
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int f4 = 0; f4 < NB; ++f4)
                        split_state_store4<decltype(type)::value>(part, lane_elem + c * N + 4 * f4, next4(c, f4));
            };
            if (st == SSM_ST_F32)
                keep(StateType<SSM_ST_F32>());
            else if (st == SSM_ST_F16)
                keep(StateType<SSM_ST_F16>());
            else
                keep(StateType<SSM_ST_BF16>());
        }
        if (!y) {
            keep_state();
            continue;
        }
        // ---- outputs, one channel of the lane after the other: element r of Y[ih] is token 16 ih + 4 kq + r
        auto intra = [&](const uint4 &xo, f32x4 &y0, f32x4 &y1) {
            const uint4 x2 = make_uint4(xo.x, xo.y, xo.x, xo.y);
            y0 = mfma_b16(g_l, x2, y0);
            y1 = mfma_b16(g_hi[2], xo, y1);
            y1 = mfma_b16(g_hi[1], xo, y1);
            y0 = mfma_b16(g_hm, x2, y0);
            y1 = mfma_b16(g_hi[0], xo, y1);
        };
        const float4 ei0 = *reinterpret_cast<const float4 *>(&W.ei[4 * kq]);
        const float4 ei1 = *reinterpret_cast<const float4 *>(&W.ei[16 + 4 * kq]);
        const f32x4 ei[2] = {{ei0.x, ei0.y, ei0.z, ei0.w}, {ei1.x, ei1.y, ei1.z, ei1.w}};
        float rows_z = 0.f;                 // NaN if an output of the first channel is not finite
        float Yf[2][8];                     // the present channel and the one before it
        uint32_t out[(NC + 1) / 2][8];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            __builtin_amdgcn_sched_barrier(0);
            f32x4 Y[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
            if constexpr (NB == 1) {
                uint32_t p[2][3];
                split3(sp[c][0].x, sp[c][0].y, p[0]);
                split3(sp[c][0].z, sp[c][0].w, p[1]);
                const uint4 s_hm = make_uint4(p[0][0], p[1][0], p[0][1], p[1][1]), s_l = make_uint4(p[0][2], p[1][2], 0u, 0u);
#pragma unroll
                for (int ih = 0; ih < 2; ++ih) {
                    const uint4 co = row_operand(Cr[ih], 0, true);
                    Y[ih] = mfma_b16(co, s_l, Y[ih]);
                    Y[ih] = mfma_b16(co, s_hm, Y[ih]);
                }
            } else {
#pragma unroll
                for (int s = 0; s < kSteps; ++s) {
                    const float4 s0 = sp[c][2 * s], s1 = sp[c][2 * s + 1];
                    const float v[8] = {s0.x, s0.y, s0.z, s0.w, s1.x, s1.y, s1.z, s1.w};
                    uint4 so[3];
                    split3x8(v, so);
#pragma unroll
                    for (int part = 2; part >= 0; --part)
#pragma unroll
                        for (int ih = 0; ih < 2; ++ih)
                            Y[ih] = mfma_b16(row_operand(Cr[ih], s, false), so[part], Y[ih]);
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e)
                Y[e >> 2][e & 3] *= ei[e >> 2][e & 3];
            const f32x4 in0 = Y[0], in1 = Y[1];
            intra(make_uint4(xpair(c, 0), xpair(c, 1), xpair(c, 2), xpair(c, 3)), Y[0], Y[1]);
            // an x or a state that is not finite has reached every query of its channel (the queries before such a token as
            // 0 * inf), a B or C that is not every channel of its queries
            float z = c == 0 ? 0.f : rows_z;
#pragma unroll
            for (int e = 0; e < 8; e += c == 0 ? 1 : 4)
                z = __builtin_fmaf(Y[e >> 2][e & 3], 0.f, z);
            if (c == 0)
                rows_z = z;
            if (__builtin_expect(__any(z != 0.f), 0)) {
                int first = kUnit;  // the channel's first such token
                uint32_t u[8];
#pragma unroll
                for (int e = 7; e >= 0; --e) {
                    const uint32_t raw = __float_as_uint(xval(c, e));
                    const bool nf = (raw & 0x7f800000u) == 0x7f800000u;
                    u[e] = nf ? 0u : raw;
                    first = nf ? 16 * (e >> 2) + (e & 3) : first;
                }
                first += 4 * kq;
                W.first_bad[lane] = first;
                lds_wait();
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    first = W.first_bad[16 * q + li] < first ? W.first_bad[16 * q + li] : first;
                lds_wait();
                first -= 4 * kq;
                f32x4 c0 = in0, c1 = in1;
                intra(make_uint4(upper2(u[0], u[1]), upper2(u[2], u[3]), upper2(u[4], u[5]), upper2(u[6], u[7])), c0, c1);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    Y[0][r] = r < first && finite(c0[r]) ? c0[r] : Y[0][r];
                    Y[1][r] = 16 + r < first && finite(c1[r]) ? c1[r] : Y[1][r];
                }
                // what is still not finite is infinite or NaN as the sum of its terms is: of a query 16 ih + 4 kq + r the lanes
                // 16 q + li hold the state and the tokens, the lanes 16 q + 4 kq + r the scores (their first parts will do)
                const __amdgpu_buffer_rsrc_t cs = split_rsrc(Cg + (size_t)tok0 * gn_b, (uint32_t)(len - 1) * gn_b + 2 * N);
#pragma nounroll
                for (int e = 0; e < 8; ++e) {
                    const int i = 16 * (e >> 2) + 4 * kq + (e & 3);
                    float inter = 0.f, sum = 0.f;
#pragma nounroll
                    for (int q = 0; q < 4; ++q) {
#pragma unroll
                        for (int f = 0; f < kRun; ++f) {
                            __builtin_amdgcn_sched_barrier(0);
                            const float4 &v = sp[c][f / 4];
                            const float s = f % 4 == 0 ? v.x : f % 4 == 1 ? v.y : f % 4 == 2 ? v.z : v.w;
                            uint32_t cw;
                            load_words<2>(cs, (i < len ? i : len - 1) * gn_b + 2 * f, 2 * kRun * q, &cw);
                            inter += __uint_as_float(cw << 16) * __shfl(s, 16 * q + li, 64);
                        }
#pragma unroll
                        for (int k2 = 0; k2 < 8; ++k2) {
                            __builtin_amdgcn_sched_barrier(0);
                            const uint32_t hi = e >= 4 ? (k2 < 2 ? g_hi[0].x : k2 < 4 ? g_hi[0].y : k2 < 6 ? g_hi[0].z : g_hi[0].w)
                                                       : (k2 < 2 ? g_hm.x : k2 < 4 ? g_hm.y : 0u);
                            const float g = __shfl(__uint_as_float((k2 & 1) ? hi & 0xffff0000u : hi << 16), 16 * q + 4 * kq + (e & 3), 64);
                            const float xv = __shfl(xval(c, k2), 16 * q + li, 64);
                            sum += 16 * (k2 >> 2) + 4 * q + (k2 & 3) <= i ? g * xv : 0.f;
                        }
                    }
                    const float v = W.ei[i] * inter + sum;
#pragma unroll
                    for (int k2 = 0; k2 < 8; ++k2)
                        Y[k2 >> 2][k2 & 3] = k2 == e && !finite(Y[k2 >> 2][k2 & 3]) ? v : Y[k2 >> 2][k2 & 3];
                }
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                Yf[c & 1][e] = __builtin_fmaf(Dh, xval(c, e), Y[e >> 2][e & 3]);
                if ((c & 1) || NC == 1)
                    out[c / 2][e] = split_pack(Yf[0][e], Yf[NC == 1 ? 0 : 1][e]);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        const __amdgpu_buffer_rsrc_t ys = split_rsrc(y + (size_t)tok0 * hp_b, (uint32_t)(len - 1) * hp_b + 32 * NC);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int up = 16 * (e >> 2) + (e & 3);
            if (4 * kq >= len - up)
                continue;
            const int own = (int)(4 * kq * hp_b + 2 * NC * li), row = (int)(up * hp_b);
            if constexpr (NC == 1) {
                __builtin_amdgcn_raw_buffer_store_b16((uint16_t)out[0][e], ys, own, row, 0);
            } else if constexpr (NC == 2) {
                __builtin_amdgcn_raw_buffer_store_b32(out[0][e], ys, own, row, 0);
            } else {
                const split_u32x2 both = {out[0][e], out[1][e]};
                __builtin_amdgcn_raw_buffer_store_b64(both, ys, own, row, 0);
            }
        }
        keep_state();
    }
}

// What a launch covers: `seqs` sequences, `busy` of them not empty, of `units` units (tiles of 16 tokens, units of 32) in
// all, `longest` in one.
struct F32Batch {
    int seqs, busy, longest;
    long long units;
};

// Waves per workgroup.  A workgroup's waves work on one sequence, so a long sequence wants many of them.  But waves a
// sequence has no units for only keep others off the compute unit, and in a launch that fills the GPU anyway waves come
// cheaper as workgroups of their own, with no hand-off between them.  So: as few as keep the longest sequence from
// outlasting the average of the `resident` waves that the GPU holds (by 4 : 3, or more than four waves, if not all of the
// workgroups then run at once, by 2 : 3), and at least four where up to three workgroups share a compute unit, which then read
// the states faster.  Against eight waves for every launch (sixteen with d_state 16 in fp32), per call: 600 sequences of one
// token, 32 heads x 64 channels, d_state 16, 328 -> 56 us in bf16 storage, 327 -> 45 us in fp32 (the vector-ALU kernel: 99
// and 98); 64 sequences of 100 tokens 43 -> 21 us and 57 -> 32 us; roll-forward of 64 sequences by 8 tokens, 80 heads x 64
// channels, d_state 128, 140 -> 74 us with fp16 states, 288 -> 107 us in fp32.
inline int scan_waves(const F32Batch &b, long long streams_per_seq, int resident, int least, int most)
{
    const long long wgs = b.busy * streams_per_seq, per_wave = (b.units * streams_per_seq + resident - 1) / resident;
    int nw = wgs <= 768 ? 4 : least;
    while (nw < most && nw < b.longest) {
        const bool in_turn = nw >= 4 && 2ll * nw * wgs > resident;  // workgroups of twice the waves would have to queue
        if ((in_turn ? 6 : 3) * nw * per_wave >= 4ll * b.longest)
            break;
        nw *= 2;
    }
#ifdef SSM_F32_WAVES  // the emulator's: a number of waves for every launch, 0: this rule
    if (SSM_F32_WAVES)
        nw = SSM_F32_WAVES < least ? least : SSM_F32_WAVES;
#endif
    return nw;
}

// A launch has fewer than 2^32 threads: a batch that needs more (tens of thousands of sequences) takes several.
#ifndef SSM_F32_MOST_THREADS
#define SSM_F32_MOST_THREADS (1ll << 31)
#endif
template <typename Launch> hipError_t in_launches(F32Args a, const F32Batch &b, int threads, Launch launch)
{
    const long long per_seq = (long long)a.H * a.slices;
    const long long most = SSM_F32_MOST_THREADS / (per_seq * threads);
    const int step = most < 1 ? 1 : most < b.seqs ? (int)most : b.seqs;
    for (; a.first < b.seqs; a.first += step) {
        const int n = b.seqs - a.first < step ? b.seqs - a.first : step;
        launch(a, dim3((unsigned)(n * per_seq)));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}
template <int NB, int NC, int NW> hipError_t launch_f32_nw(const F32Args &args, const F32Batch &b, hipStream_t stream)
{
    return in_launches(args, b, 64 * NW, [&](const F32Args &a, dim3 grid) {
        hipLaunchKernelGGL((ssm_scan_f32_kernel<NB, NC, NW>), grid, dim3(64 * NW), sizeof(F32Lds<NB, NC, NW>), stream, a);
    });
}
template <int NB, int NC> hipError_t launch_f32(const F32Args &a, const F32Batch &b, hipStream_t stream)
{
    // registers for about three waves on each of the 1024 SIMDs; with d_state 128 one wave alone is slow to read the state
    switch (scan_waves(b, (long long)a.H * a.slices, 3 * 1024, NB == 8 ? 2 : 1, NB == 1 ? 16 : 8)) {
    case 1: return launch_f32_nw<NB, NC, NB == 8 ? 2 : 1>(a, b, stream);
    case 2: return launch_f32_nw<NB, NC, 2>(a, b, stream);
    case 4: return launch_f32_nw<NB, NC, 4>(a, b, stream);
    case 8: return launch_f32_nw<NB, NC, 8>(a, b, stream);
    default: return launch_f32_nw<NB, NC, NB == 1 ? 16 : 8>(a, b, stream);
    }
}

template <int NB, int NC, int NW> hipError_t launch_split_nw(const F32Args &args, const F32Batch &b, hipStream_t stream)
{
    return in_launches(args, b, 64 * NW, [&](const F32Args &a, dim3 grid) {
        hipLaunchKernelGGL((ssm_scan_split_kernel<NB, NC, NW>), grid, dim3(64 * NW), sizeof(SplitLds<NB, NC, NW>), stream, a);
    });
}
template <int NB, int NC> hipError_t launch_split(const F32Args &a, const F32Batch &b, hipStream_t stream)
{
    // registers for two waves per SIMD where the state is large; sixteen waves would spill (94 instead of 67 us for the
    // packed batch above)
    switch (scan_waves(b, (long long)a.H * a.slices, 2 * 1024, 1, 8)) {
    case 1: return launch_split_nw<NB, NC, 1>(a, b, stream);
    case 2: return launch_split_nw<NB, NC, 2>(a, b, stream);
    case 4: return launch_split_nw<NB, NC, 4>(a, b, stream);
    default: return launch_split_nw<NB, NC, 8>(a, b, stream);
    }
}

template <int NB> hipError_t launch_f32_nc(F32Args &a, bool split, int nc, const F32Batch &b, hipStream_t stream)
{
    a.slices = a.P / (16 * nc);
    constexpr int kMost = NB <= 2 ? 4 : 2;  // four slices only with small states
    constexpr int kMostSplit = NB == 8 ? 1 : kMost;
    if (nc == 4)
        return split ? launch_split<NB, kMostSplit>(a, b, stream) : launch_f32<NB, kMost>(a, b, stream);
    if (nc == 2)
        return split ? launch_split<NB, kMostSplit < 2 ? 1 : 2>(a, b, stream) : launch_f32<NB, 2>(a, b, stream);
    return split ? launch_split<NB, 1>(a, b, stream) : launch_f32<NB, 1>(a, b, stream);
}

// ================================================================ vector ALUs, any shape
// One workgroup per (sequence, head); the [P,N] state lives in registers and is mirrored in LDS for the C.S products.
constexpr int kThreads = 256;
constexpr int kQ = kValuTileTokens;

template <typename IO, int EPT>
__global__ __launch_bounds__(kThreads) void ssm_scan_valu_kernel(ScanArgs a, StatePtrs from)
{
    const int tid = threadIdx.x;
    const int H = a.H, P = a.P, N = a.N, G = a.G;
    const int seq = blockIdx.x / H;
    const int h = blockIdx.x % H;
    const int g = h / (H / G);
    const int PN = P * N;
    const int NP1 = N + 1;

    extern __shared__ __align__(16) unsigned char lds_raw[];
    double *ell = reinterpret_cast<double *>(lds_raw);            // [q] inclusive sums of dt*A
    float *S_lds = reinterpret_cast<float *>(ell + kQ);           // [P][N+1]
    float *xs = S_lds + (size_t)P * NP1;                          // [q][P]
    float *Bs = xs + kQ * P;                                      // [q][N]
    float *Cs = Bs + kQ * N;                                      // [q][N]
    float *Gm = Cs + kQ * N;                                      // [q][q] masked scores
    float *dts = Gm + kQ * kQ;                                    // [q]
    float *wj = dts + kQ;                                         // [q] e^{l_last-l_j} dt_j
    float *ei = wj + kQ;                                          // [q] e^{l_i}

    const IO *x = static_cast<const IO *>(a.x);
    const IO *dt = static_cast<const IO *>(a.dt);
    const IO *Bg = static_cast<const IO *>(a.B);
    const IO *Cg = static_cast<const IO *>(a.C);
    IO *y = static_cast<IO *>(a.y);
    const float Ah = a.A[h];
    const float Dh = a.D[h];

    // running state: element e = tid + k*256 of this head's [P,N] block
    float acc[EPT];
    const void *init = from.of(seq);
    const int st = a.state_dtype;
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
        const int e = tid + k * kThreads;
        float v = 0.f;
        if (e < PN) {
            if (init)
                v = state_load(init, (size_t)h * PN + e, st);
            S_lds[(e / N) * NP1 + (e % N)] = v;
        }
        acc[k] = v;
    }

    const SsmSeq sq = a.seqs[seq];
    for (int ti = sq.tile_begin; ti < sq.tile_end; ++ti) {
        const SsmTile t = a.tiles[ti];
        const int len = t.len;
        const size_t tok0 = (size_t)t.tok0;

        if (tid < kQ)
            dts[tid] = tid < len ? IoTraits<IO>::load(dt + (tok0 + tid) * H + h) : 0.f;
        for (int idx = tid; idx < kQ * P; idx += kThreads) {
            const int i = idx / P, p = idx % P;
            xs[idx] = i < len ? IoTraits<IO>::load(x + ((tok0 + i) * H + h) * P + p) : 0.f;
        }
        for (int idx = tid; idx < kQ * N; idx += kThreads) {
            const int i = idx / N, n = idx % N;
            const size_t off = ((tok0 + i) * G + g) * N + n;
            Bs[idx] = i < len ? IoTraits<IO>::load(Bg + off) : 0.f;
            Cs[idx] = i < len ? IoTraits<IO>::load(Cg + off) : 0.f;
        }
        __syncthreads();

        if (tid < kQ) {
            double s = 0.0;
            for (int k = 0; k <= tid; ++k)
                s += (double)dts[k] * (double)Ah;
            ell[tid] = s;
        }
        __syncthreads();
        if (tid < kQ) {
            wj[tid] = tid < len ? expf((float)(ell[len - 1] - ell[tid])) * dts[tid] : 0.f;
            ei[tid] = expf((float)ell[tid]);
        }
        // masked, decayed scores: one (i, j) pair per thread
        {
            const int i = tid / kQ, j = tid % kQ;
            float v = 0.f;
            if (j <= i && i < len) {
                float dot = 0.f;
                for (int n = 0; n < N; ++n)
                    dot += Cs[i * N + n] * Bs[j * N + n];
                v = dot * expf((float)(ell[i] - ell[j])) * dts[j];
            }
            Gm[tid] = v;
        }
        __syncthreads();

        // outputs of the tile
        for (int idx = tid; idx < len * P; idx += kThreads) {
            const int i = idx / P, p = idx % P;
            float inter = 0.f;
            const float *Sp = S_lds + p * NP1;
            for (int n = 0; n < N; ++n)
                inter += Cs[i * N + n] * Sp[n];
            float intra = 0.f;
            for (int j = 0; j <= i; ++j)
                intra += Gm[i * kQ + j] * xs[j * P + p];
            const float v = ei[i] * inter + intra + Dh * xs[idx];
            IoTraits<IO>::store(y + ((tok0 + i) * H + h) * P + p, v);
        }
        __syncthreads();

        // state after the tile
        const float dlast = ei[len - 1];
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            const int e = tid + k * kThreads;
            if (e < PN) {
                const int p = e / N, n = e % N;
                float s = dlast * acc[k];
                for (int j = 0; j < len; ++j)
                    s += (wj[j] * xs[j * P + p]) * Bs[j * N + n];
                acc[k] = s;
                S_lds[p * NP1 + n] = s;
                if (t.ckpt_slot >= 0)
                    state_store(a.state_out, ((size_t)t.ckpt_slot * H + h) * PN + e, s, st);
            }
        }
        __syncthreads();
    }
}

template <typename IO>
hipError_t launch_ept(int ept, dim3 grid, size_t lds, hipStream_t stream, const ScanArgs &args)
{
#define SSM_LAUNCH(E)                                                                     \
    hipLaunchKernelGGL((ssm_scan_valu_kernel<IO, E>), grid, dim3(kThreads), lds, stream, args, \
                       state_ptrs_of(args.init_ptrs, args.host_ptrs, args.n_host_ptrs));        \
    break;
    switch (ept) {
    case 1: SSM_LAUNCH(1)
    case 2: SSM_LAUNCH(2)
    case 4: SSM_LAUNCH(4)
    case 8: SSM_LAUNCH(8)
    case 16: SSM_LAUNCH(16)
    default: SSM_LAUNCH(32)
    }
#undef SSM_LAUNCH
    return hipGetLastError();
}

}  // namespace

bool scan_f32_supports(const ssm_shape_t &s)
{
    const int n = s.d_state;
    return s.headdim % 16 == 0 && (n == 16 || n == 32 || n == 64 || n == 128);
}

// roll: the states behind init_ptrs / host_ptrs are advanced in place over the sequences' tokens.  Else the scan over the
// plan's tiles.  n_seqs: only so many of the plan's sequences, the longest ones (needs args.order unless it is all).
hipError_t launch_scan_f32(const ssm_plan *plan, const ScanArgs &args, bool roll, int n_seqs, hipStream_t stream)
{
    F32Args a;
    a.x = args.x, a.dt = args.dt, a.B = args.B, a.C = args.C;
    a.A = args.A, a.D = args.D;
    a.y = args.y;
    a.state_out = args.state_out;
    a.init = state_ptrs_of(args.init_ptrs, args.host_ptrs, args.n_host_ptrs);
    a.roll = roll;
    a.tiles = args.tiles;
    a.seqs = args.seqs;
    a.order = n_seqs < plan->batch ? args.order : nullptr;
    a.first = 0;
    a.H = args.H, a.P = args.P, a.G = args.G;
    a.state_dtype = args.state_dtype;
    const bool split = plan->shape.io_dtype == SSM_DT_BF16;
    const int nb = args.N / 16;
    const int busy = ssm_plan_longer_than(plan, 0);
    const long long streams = (long long)(busy < n_seqs ? busy : n_seqs) * args.H;
    int nc = ssm_f32_slices(split, args.N, args.P, streams);
#ifdef SSM_F32_SLICES  // the emulator's: so many for every launch, 0: the rule
    if (SSM_F32_SLICES)
        nc = SSM_F32_SLICES;
#endif
    // the scan's units are the plan's tiles; the roll-forward cuts the tokens itself
    const SsmSeq &lq = plan->seqs[plan->order[0]];
    F32Batch batch = {n_seqs, busy < n_seqs ? busy : n_seqs, lq.tile_end - lq.tile_begin, (long long)plan->tiles.size()};
    if (roll) {
        const int unit = split ? kUnit : kValuTileTokens;
        batch.longest = (ssm_plan_tokens(plan, plan->order[0]) + unit - 1) / unit;
        batch.units = 0;
        for (int r = 0; r < n_seqs && r < busy; ++r)
            batch.units += (ssm_plan_tokens(plan, plan->order[r]) + unit - 1) / unit;
    }
    switch (nb) {
    case 1: return launch_f32_nc<1>(a, split, nc, batch, stream);
    case 2: return launch_f32_nc<2>(a, split, nc, batch, stream);
    case 4: return launch_f32_nc<4>(a, split, nc, batch, stream);
    default: return launch_f32_nc<8>(a, split, nc, batch, stream);
    }
}

size_t ssm_valu_lds_bytes(int P, int N);

hipError_t launch_scan_valu(const ssm_plan *plan, const ScanArgs &args, hipStream_t stream)
{
    if (scan_f32_supports(plan->shape))
        return launch_scan_f32(plan, args, false, plan->batch, stream);
    const int PN = args.P * args.N;
    int ept = 1;
    while (ept * kThreads < PN)
        ept *= 2;
    const dim3 grid((unsigned)plan->n_workgroups);
    const size_t lds = ssm_valu_lds_bytes(args.P, args.N);
    if (plan->shape.io_dtype == SSM_DT_F32)
        return launch_ept<float>(ept, grid, lds, stream, args);
    return launch_ept<bf16_t>(ept, grid, lds, stream, args);
}
