// fp32 scan kernels: f32 or bf16 storage, all arithmetic in fp32 (decay exponents summed in fp64).  They are the path of
// the fp32 mode, of the shapes the fp16 / bf16 matrix-core kernel does not cover, and of the roll-forward over more
// than a few tokens.
//
// Both work tile by tile; per tile of q <= 16 tokens starting after token s, with l_i = A * sum_{k<=i} dt_k inside the
// tile:
//
//   y_i  = e^{l_i} (S_s C_i) + sum_{j<=i} (C_i.B_j) e^{l_i-l_j} dt_j x_j + D x_i
//   S_e  = e^{l_q} S_s + sum_j e^{l_q-l_j} dt_j x_j B_j^T
//
// which is the token recurrence of ssm_prefill.h unrolled over the tile.  Where d_state is 16, 32, 64 or 128 and headdim
// a multiple of 16 the contractions run on the matrix cores in fp32 (ssm_scan_f32_kernel); any other shape takes the
// vector ALUs (ssm_scan_valu_kernel).
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
// call: 80 heads x 64 channels, d_state 128, 2048 tokens in fp32 8180 -> 141 us; 32 heads x 64 channels, d_state 16, eight
// requests of 18 K tokens in all, bf16 storage, 2130 -> 109 us; 4 heads x 16 channels, d_state 16, 256 tokens 64 -> 12 us.
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
    int H, P, G, slices, state_dtype;
};

// n values (a multiple of 4, or 1 or 2) of the storage type as floats; p is aligned to the run's size, at most 16 bytes
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
template <int NV> __device__ __forceinline__ void load_run(const bf16_t *p, float *v)
{
    if (NV == 1) {
        v[0] = bf16_to_f32(*p);
    } else if (NV == 2) {
        const uint32_t u = *reinterpret_cast<const uint32_t *>(p);
        v[0] = __uint_as_float(u << 16), v[1] = __uint_as_float(u & 0xffff0000u);
    } else if (NV == 4) {
        const uint2 u = *reinterpret_cast<const uint2 *>(p);
        v[0] = __uint_as_float(u.x << 16), v[1] = __uint_as_float(u.x & 0xffff0000u);
        v[2] = __uint_as_float(u.y << 16), v[3] = __uint_as_float(u.y & 0xffff0000u);
    } else {
#pragma unroll
        for (int e = 0; e < NV; e += 8) {
            const uint4 u = *reinterpret_cast<const uint4 *>(p + e);
            const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                v[e + 2 * k] = __uint_as_float(w[k] << 16);
                v[e + 2 * k + 1] = __uint_as_float(w[k] & 0xffff0000u);
            }
        }
    }
}

// Four neighbouring elements of a cached state.
__device__ __forceinline__ float4 state_load4(const void *base, size_t idx, int st)
{
    if (st == SSM_ST_F32)
        return *reinterpret_cast<const float4 *>(static_cast<const float *>(base) + idx);
    return make_float4(state_load(base, idx, st), state_load(base, idx + 1, st), state_load(base, idx + 2, st),
                       state_load(base, idx + 3, st));
}
__device__ __forceinline__ void state_store4(void *base, size_t idx, float4 v, int st)
{
    if (st == SSM_ST_F32) {
        *reinterpret_cast<float4 *>(static_cast<float *>(base) + idx) = v;
        return;
    }
    state_store(base, idx, v.x, st);
    state_store(base, idx + 1, v.y, st);
    state_store(base, idx + 2, v.z, st);
    state_store(base, idx + 3, v.w, st);
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

struct F32Wave {          // private to one wave
    double ell[16];       // l_i
    float ei[16];         // e^{l_i}
    float wt[16];         // e^{l_q - l_j} dt_j
    float dt[16];
};
template <int NB, int NC, int NW> struct F32Lds {
    float4 S[NC][NB][64];  // [slice][four of a lane's 4 NB state elements][lane]
    int done;
    int pad[3];
    F32Wave wv[NW];
};

template <typename IO, int NB, int NC, int NW>
__global__ __launch_bounds__(64 * NW) void ssm_scan_f32_kernel(F32Args a)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    F32Lds<NB, NC, NW> &L = *reinterpret_cast<F32Lds<NB, NC, NW> *>(lds_raw);
    constexpr int N = 16 * NB;
    const int H = a.H, P = a.P, G = a.G, st = a.state_dtype;
    const int slice = blockIdx.x % a.slices;
    const int h = (blockIdx.x / a.slices) % H;
    const int seq = blockIdx.x / (a.slices * H);
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
    const IO *x = static_cast<const IO *>(a.x);
    const IO *dt = static_cast<const IO *>(a.dt);
    const IO *Bg = static_cast<const IO *>(a.B) + (size_t)g * N;
    const IO *Cg = static_cast<const IO *>(a.C) + (size_t)g * N;
    IO *y = static_cast<IO *>(a.y);
    const float Ah = a.A[h], Dh = a.D[h];
    // channel li of slice c, state indices 4 NB kq .. 4 NB kq + 4 NB - 1
    const size_t state_row = ((size_t)h * P + 16 * NC * slice + li) * N + 4 * NB * kq;
    const size_t GN = (size_t)G * N, HP = (size_t)H * P;
    const size_t xcol = (size_t)h * P + 16 * NC * slice + li;

    for (int b = w; b < NC * NB; b += NW) {
        const int c = b / NB, f4 = b % NB;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (from)
            v = state_load4(from, state_row + (size_t)16 * c * N + 4 * f4, st);
        L.S[c][f4][lane] = v;
    }
    if (threadIdx.x == 0)
        L.done = 0;
    __syncthreads();  // the only one: the starting state and the counter are in place

    F32Wave &W = L.wv[w];
    for (int k = w; k < n_tiles; k += NW) {
        int tok0, len, ckpt = -1;
        if (roll) {
            tok0 = tok_begin + 16 * k;
            len = n_tok - 16 * k < 16 ? n_tok - 16 * k : 16;
        } else {
            const SsmTile t = a.tiles[sq.tile_begin + k];
            tok0 = t.tok0, len = t.len, ckpt = t.ckpt_slot;
        }
        // rows past the end of a partial tile re-read its last row: their weights are zero
        const size_t row = (size_t)tok0 + (li < len ? li : len - 1);
        const float dtl = li < len ? IoTraits<IO>::load(dt + row * H + h) : 0.f;
        float Cf[4 * NB], Bf[4 * NB], Bt[4][NB], xv[NC][4];
        load_run<4 * NB>(Bg + row * GN + 4 * NB * kq, Bf);
        load_run<4 * NB>(Cg + row * GN + 4 * NB * kq, Cf);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const size_t tok = (size_t)tok0 + (4 * kq + r < len ? 4 * kq + r : len - 1);
            load_run<NB>(Bg + tok * GN + NB * li, Bt[r]);
#pragma unroll
            for (int c = 0; c < NC; ++c)
                xv[c][r] = IoTraits<IO>::load(x + tok * HP + xcol + 16 * c);
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
        f32_wait_counter(&L.done, k);
        // read the state, multiply-add, write it back, publish
        float4 sp[NC][NB];
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int f4 = 0; f4 < NB; ++f4)
                sp[c][f4] = L.S[c][f4][lane];
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
                L.S[c][f4][lane] = sn[c][f4];
            }
        f32_publish_counter(&L.done, k + 1, lane);
        if (ckpt >= 0 || (roll && k == n_tiles - 1)) {
            void *to = roll ? const_cast<void *>(from) : a.state_out;
            const size_t at = (roll ? 0 : (size_t)ckpt * HP * N) + state_row;
#pragma unroll
            for (int c = 0; c < NC; ++c)
#pragma unroll
                for (int f4 = 0; f4 < NB; ++f4)
                    state_store4(to, at + (size_t)16 * c * N + 4 * f4, sn[c][f4], st);
        }
        if (!y)
            continue;
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
#pragma unroll
            for (int r = 0; r < 4; ++r)
                Y0 = mfma_f32(gm[r], xv[c][r], Y0);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (4 * kq + r < len)
                    IoTraits<IO>::store(y + ((size_t)tok0 + 4 * kq + r) * HP + xcol + 16 * c,
                                        __builtin_fmaf(Dh, xv[c][r], Y0[r]));
        }
    }
}

template <typename IO, int NB, int NC>
hipError_t launch_f32(const F32Args &a, int batch, hipStream_t stream)
{
    constexpr int NW = NB == 1 ? 16 : 8;
    hipLaunchKernelGGL((ssm_scan_f32_kernel<IO, NB, NC, NW>), dim3((unsigned)batch * (unsigned)a.H * (unsigned)a.slices),
                       dim3(64 * NW), sizeof(F32Lds<NB, NC, NW>), stream, a);
    return hipGetLastError();
}

template <typename IO, int NB>
hipError_t launch_f32_nc(F32Args &a, int nc, int batch, hipStream_t stream)
{
    a.slices = a.P / (16 * nc);
    if (nc == 4)
        return launch_f32<IO, NB, NB <= 2 ? 4 : 2>(a, batch, stream);  // 4 slices only with small states
    if (nc == 2)
        return launch_f32<IO, NB, 2>(a, batch, stream);
    return launch_f32<IO, NB, 1>(a, batch, stream);
}

template <typename IO>
hipError_t launch_f32_nb(F32Args &a, int nb, int nc, int batch, hipStream_t stream)
{
    switch (nb) {
    case 1: return launch_f32_nc<IO, 1>(a, nc, batch, stream);
    case 2: return launch_f32_nc<IO, 2>(a, nc, batch, stream);
    case 4: return launch_f32_nc<IO, 4>(a, nc, batch, stream);
    default: return launch_f32_nc<IO, 8>(a, nc, batch, stream);
    }
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
// plan's tiles.
hipError_t launch_scan_f32(const ssm_plan *plan, const ScanArgs &args, bool roll, hipStream_t stream)
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
    a.H = args.H, a.P = args.P, a.G = args.G;
    a.state_dtype = args.state_dtype;
    // Slices of 16 channels per workgroup: more of them share the scores (4 nb of a tile's products), fewer leave more
    // workgroups.  Products per tile times rounds of 256 workgroups, the smaller the better.
    const int nb = args.N / 16, all = args.P / 16;
    long long streams = 0;
    for (const SsmSeq &q : plan->seqs)
        streams += q.tile_end > q.tile_begin;
    streams *= args.H;
    int nc = 1;
    long long best = 0;
    for (int c = 1; c <= (nb <= 2 ? 4 : 2); c *= 2) {
        if (all % c != 0)
            break;
        const long long rounds = (streams * (all / c) + 255) / 256, cost = rounds * (c * (8 * nb + 4) + 4 * nb);
        if (c == 1 || cost <= best)
            nc = c, best = cost;
    }
    if (plan->shape.io_dtype == SSM_DT_F32)
        return launch_f32_nb<float>(a, nb, nc, plan->batch, stream);
    return launch_f32_nb<bf16_t>(a, nb, nc, plan->batch, stream);
}

size_t ssm_valu_lds_bytes(int P, int N);

hipError_t launch_scan_valu(const ssm_plan *plan, const ScanArgs &args, hipStream_t stream)
{
    if (scan_f32_supports(plan->shape))
        return launch_scan_f32(plan, args, false, stream);
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
