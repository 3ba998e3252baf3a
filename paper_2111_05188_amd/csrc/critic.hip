// Critic (value network) forward over a time-major block of observations:
// V(x) = w3 . tanh(W2 tanh(W1 x + b1) + b2) + b3 for every row (t, e).
//
// A workgroup owns BM rows of one agent, numbered over its (step, env) pairs,
// so the weights it streams serve BM rows also where an agent has few envs.
//
// MFMA kernel (bf16, hidden widths 512 or 1024, observation rows of 1024
// columns).  Eight waves, two per SIMD; wave w owns output tiles
// w*OT .. w*OT+OT-1 of both hidden layers (OT = H / 128) for all
// BM = 512 / OT rows, a 4x8 or 8x4 register block of 16x16 fp32
// accumulators (128 registers).  The MFMA is
// v_mfma_f32_16x16x32_bf16 with A = a packed weight fragment (16 outputs x
// 32 inputs, streamed from L2 up to four k-steps ahead) and B = 32 inputs x 16 rows
// from LDS.  Layer 1 stages the observation block through LDS in chunks of
// 128 columns (double-buffered in LDS; the chunk after the next one is in
// flight while the current one is multiplied); h1 then replaces the staging
// buffers in LDS.  Layer 2's tanh outputs are rounded to bf16 and reduced
// with w3 straight from the accumulators: per lane, across the four lane
// groups of a tile, then across the eight waves in LDS, always in the same
// order, so the result is deterministic.
//
// Measured: 391 x 4,096 rows of 1001-512-512 in 2.21 ms, 1.12 PFLOP/s (2.38 ms
// with the staging loads ahead of the weights: each chunk then waited for
// HBM); 72 envs of four agents x 391 steps in 53 us (299 us with a block per
// step and agent: 18 of its 128 rows).  101 x 728 rows of 1001-1024-1024 in
// 0.315 ms (0.321).  (The 512-wide kernel is at its 256 registers and spills
// 8 of them, which the times include.)
//
// Every other shape (fp32, or bf16 of other widths) runs the tile kernel
// below.
#include <type_traits>

#include "device.hpp"
#include "internal.hpp"

// MFMA kernel configuration: waves per workgroup and 16x16 accumulator
// tiles per wave (each 4 registers).
#ifndef CRITIC_NW
#define CRITIC_NW 8
#endif
#ifndef CRITIC_ACC_TILES
#define CRITIC_ACC_TILES 32
#endif
#ifndef CRITIC_MIN_WAVES
#define CRITIC_MIN_WAVES 2
#endif


namespace tpk {

namespace {

typedef uint32_t u4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8 as_bf16x8(u4v v) { return __builtin_bit_cast(bf16x8, v); }

// Rows of workgroup b: BM (or the nrow left) of its agent's T epa rows,
// numbered over (step, env), so that few envs an agent still fill a block.
struct RowBlock {
    int agent, nrow, e0, epa;
    int64_t t0, E;
    // row r of the block in the [T][E] arrays
    __device__ __forceinline__ int64_t at(int r) const
    {
        const uint32_t x = (uint32_t)e0 + (uint32_t)r, t = x / (uint32_t)epa;
        return (t0 + t) * E + (int64_t)agent * epa + (x - t * (uint32_t)epa);
    }
};

__device__ __forceinline__ RowBlock row_block(const CriticArgs &A, int BM)
{
    RowBlock r;
    r.epa = A.envs_per_agent;
    r.E = A.E;
    const int64_t R = A.T * r.epa, bpa = (R + BM - 1) / BM;
    r.agent = (int)(blockIdx.x / bpa);
    const int64_t r0 = (int64_t)(blockIdx.x % bpa) * BM;
    r.nrow = (int)min((int64_t)BM, R - r0);
    r.t0 = r0 / r.epa;
    r.e0 = (int)(r0 % r.epa);
    return r;
}

// NW waves, each OT output tiles x RT row tiles of accumulators; KS1
// k-steps of 32 inputs in layer 1 (a multiple of 4).
template <int NW, int OT, int RT, int KS1>
__global__ __launch_bounds__(NW *WAVE, CRITIC_MIN_WAVES) void critic_mfma_kernel(CriticArgs A)
{
    constexpr int NTH = NW * WAVE;
    constexpr int H = 16 * NW * OT;    // hidden width (both layers)
    constexpr int BM = 16 * RT;        // rows per workgroup
    constexpr int KC = 128;            // columns per staged chunk (4 k-steps)
    constexpr int NCH = KS1 / 4;
    constexpr int LDX = KC + 8;        // staged row pitch (conflict-free reads)
    constexpr int LDH = H + 8;
    constexpr int KS2 = H / 32;
    constexpr int SPT = BM * (KC / 8) / NTH;   // 16-byte staging loads per thread
    static_assert(KS1 % 4 == 0 && KS2 % 4 == 0 && SPT >= 1, "shape");
    extern __shared__ __align__(16) uint8_t smem[];
    __bf16 *Xs = (__bf16 *)smem;       // [2][BM][LDX]
    __bf16 *H1s = (__bf16 *)smem;      // [BM][LDH] (after layer 1)
    constexpr size_t XBYTES = 2 * BM * LDX * 2, HBYTES = (size_t)BM * LDH * 2;
    float *vred = (float *)(smem + (XBYTES > HBYTES ? XBYTES : HBYTES));   // [NW][BM]

    const CriticLayout &P = A.lay;
    const int tid = threadIdx.x, lane = tid % WAVE;
    const int w = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const int r16 = lane & 15, kq = lane >> 4;
    const RowBlock rb = row_block(A, BM);
    const uint8_t *pk = A.packed + (size_t)rb.agent * P.agent_stride;

    // weight fragments in a ring of RS slots (64 registers)
    constexpr int RS = 16 / OT;
    static_assert(4 % RS == 0, "a chunk is whole rounds of the ring");
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)pk, (short)0, (int)P.agent_stride, 0x00020000);
    const int voff = lane * 16;
    const int base1 = (int)P.off_W[0] + w * OT * KS1 * 1024;
    const int base2 = (int)P.off_W[1] + w * OT * KS2 * 1024;
    bf16x8 wr[RS][OT];
    auto fetch1 = [&](int slot, int k) {
#pragma unroll
        for (int ot = 0; ot < OT; ++ot)
            wr[slot][ot] = as_bf16x8(__builtin_amdgcn_raw_buffer_load_b128(
                rsrc, voff, base1 + (ot * KS1 + k) * 1024, 0));
    };
    auto fetch2 = [&](int slot, int k) {
#pragma unroll
        for (int ot = 0; ot < OT; ++ot)
            wr[slot][ot] = as_bf16x8(__builtin_amdgcn_raw_buffer_load_b128(
                rsrc, voff, base2 + (ot * KS2 + k) * 1024, 0));
    };

    // observation staging: thread tid moves the 16-byte pieces tid + NTH i
    // of a 128-column chunk (row idx / 16, piece idx % 16); rows past the
    // block's last read its last row (never stored)
    const __bf16 *src[SPT];
#pragma unroll
    for (int i = 0; i < SPT; ++i) {
        const int idx = tid + NTH * i, row = min(idx >> 4, rb.nrow - 1), part = idx & 15;
        src[i] = (const __bf16 *)A.obs + (size_t)rb.at(row) * A.ld_obs + part * 8;
    }
    u4v st[SPT];
    auto load_chunk = [&](int c) {
#pragma unroll
        for (int i = 0; i < SPT; ++i)
            st[i] = __builtin_nontemporal_load((const u4v *)(src[i] + c * KC));
    };
    auto store_chunk = [&](int buf) {
#pragma unroll
        for (int i = 0; i < SPT; ++i) {
            const int idx = tid + NTH * i, row = idx >> 4, part = idx & 15;
            *(u4v *)(Xs + (size_t)buf * BM * LDX + row * LDX + part * 8) = st[i];
        }
    };

    load_chunk(0);
#pragma unroll
    for (int q = 0; q < RS; ++q) fetch1(q, q);
    store_chunk(0);
    load_chunk(NCH > 1 ? 1 : 0);
    __syncthreads();

    // ---- layer 1 ----------------------------------------------------------
    floatx4 acc[OT][RT];
    // one k-step: B fragments row tile by row tile (the next one read
    // while the current one is multiplied), each against the OT weights
    auto mma_kstep = [&](const __bf16 *xk, int ld, int slot) {
        bf16x8 x = *(const bf16x8 *)xk;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            bf16x8 xn;
            if (rt + 1 < RT) xn = *(const bf16x8 *)(xk + (rt + 1) * 16 * ld);
#pragma unroll
            for (int ot = 0; ot < OT; ++ot)
                acc[ot][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wr[slot][ot], x, acc[ot][rt],
                                                                      0, 0, 0);
            if (rt + 1 < RT) x = xn;
        }
    };
#pragma unroll
    for (int ot = 0; ot < OT; ++ot)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[ot][rt] = floatx4{0.f, 0.f, 0.f, 0.f};
    // Loads complete in order, so a wait for weights is a wait for every load
    // issued before them: a chunk's staging loads (which come from HBM) go out
    // after the weights of the next k-steps (RS = 4: of the whole next chunk),
    // and their own use is a chunk later.
    for (int c = 0; c < NCH; ++c) {
        const bool more = c + 1 < NCH;
        const __bf16 *xb = Xs + (size_t)(c & 1) * BM * LDX + r16 * LDX + kq * 8;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            mma_kstep(xb + 32 * q, LDX, q % RS);
            if (q + RS < 4 || more) fetch1(q % RS, c * 4 + q + RS);
            else fetch2(q % RS, q + RS - 4);
            if constexpr (OT == 4) __builtin_amdgcn_sched_barrier(0);
        }
        if (more) {
            store_chunk((c + 1) & 1);
            if (c + 2 < NCH) load_chunk(c + 2);
        }
        __syncthreads();
    }

    // h1 = tanh(acc + b1) in bf16, over the staging buffers
    {
        const float *b1 = (const float *)(pk + P.off_b[0]);
#pragma unroll
        for (int ot = 0; ot < OT; ++ot) {
            const int o = (w * OT + ot) * 16 + kq * 4;
            const floatx4 bv = *(const floatx4 *)(b1 + o);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                const bf16x4 h = {to_bf16(tanh_from_e2(NEG_2LOG2E * (acc[ot][rt][0] + bv[0]))),
                                  to_bf16(tanh_from_e2(NEG_2LOG2E * (acc[ot][rt][1] + bv[1]))),
                                  to_bf16(tanh_from_e2(NEG_2LOG2E * (acc[ot][rt][2] + bv[2]))),
                                  to_bf16(tanh_from_e2(NEG_2LOG2E * (acc[ot][rt][3] + bv[3])))};
                *(bf16x4 *)(H1s + (rt * 16 + r16) * LDH + o) = h;
            }
        }
    }
    __syncthreads();

    // ---- layer 2 (k-steps continue the fragment stream at KS1) -------------
#pragma unroll
    for (int ot = 0; ot < OT; ++ot)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[ot][rt] = floatx4{0.f, 0.f, 0.f, 0.f};
    {
        // layer-2 k-step ks sits in ring slot ks % RS
        const __bf16 *hb = H1s + r16 * LDH + kq * 8;
        for (int ks = 0; ks < KS2; ks += 4) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                mma_kstep(hb + (ks + q) * 32, LDH, q % RS);
                if (ks + q + RS < KS2) fetch2(q % RS, ks + q + RS);
                if constexpr (OT == 4) __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    // ---- h2 = bf16(tanh(acc + b2)); V = w3 . h2 + b3 ------------------------
    {
        const float *b2 = (const float *)(pk + P.off_b[1]);
        const float *w3 = (const float *)(pk + P.off_W[2]);
        float part[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) part[rt] = 0.f;
#pragma unroll
        for (int ot = 0; ot < OT; ++ot) {
            const int o = (w * OT + ot) * 16 + kq * 4;
            const floatx4 bv = *(const floatx4 *)(b2 + o);
            const floatx4 wv = *(const floatx4 *)(w3 + o);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float h = (float)to_bf16(tanh_from_e2(NEG_2LOG2E * (acc[ot][rt][i] + bv[i])));
                    part[rt] = fmaf(wv[i], h, part[rt]);
                }
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            part[rt] += __shfl_xor(part[rt], 16);
            part[rt] += __shfl_xor(part[rt], 32);
        }
        if (kq == 0)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) vred[w * BM + rt * 16 + r16] = part[rt];
    }
    __syncthreads();
    if (tid < rb.nrow) {
        float v = *(const float *)(pk + P.off_b[2]);
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) v += vred[ww * BM + tid];
        A.value[rb.at(tid)] = v;
    }
}

// ---------------------------------------------------------------------------
// Every other shape (fp32, or bf16 of other widths): the tile kernel.
//
// A workgroup takes BM = 16 RT rows of one agent.  Weights are
// MFMA fragments of 1 KiB ([tile of 16 outputs][k-block][64 lanes][16
// bytes]; a k-block is 16 fp32 or 32 bf16 inputs) streamed from L2 D blocks
// ahead; rows and the first hidden layer sit in LDS.  A wave owns OT output
// tiles at a time, OT x RT accumulators.  fp32 takes
// v_mfma_f32_16x16x4_f32, MFMA e on element e of every lane's 16 bytes.
// Where one round of the waves covers layer 1, the hidden rows take the
// observation rows' place (a third workgroup then fits a CU).
//
// fp32 is bound by its MFMAs: a year of the 30-stock daily workload (253 x
// 1,024 rows, 301-256-256) takes 0.71 ms, 104 TFLOP/s of the 153 a large
// fp32 product reaches; 0.68 ms without the tanh.  The kernel before it (one
// VALU thread an output, 16 rows a workgroup) took 2.26 ms, and 2.21 ms with
// bf16 rows, where this one takes 0.18 (1.00 against 0.11 at 298-128-352,
// 21.6 against 0.46 at 1001-768-768).  D weight blocks in flight: 2 for
// fp32 (4: 1% slower), 4 for bf16 (2: 5% slower, 8: 80%).  Two workgroups a
// CU, without the shared place: 0.75 ms; eight waves a workgroup: 0.71.
// ---------------------------------------------------------------------------
template <bool BF>
struct TileType {
    typedef float E;
};
template <>
struct TileType<true> {
    typedef __bf16 E;
};

constexpr int TILE_NW = 4;   // waves per workgroup

// One layer for this wave's tiles: h = tanh(W x + b) into hs, or, for the
// LAST one, part[rt] += w3 . h of this lane's outputs.
template <bool BF, int RT, int NW, int OT, bool LAST>
__device__ __forceinline__ void tile_layer(const uint8_t *W, const float *bias, const float *w3,
                                           int H, int NT, int KB, const uint8_t *xs, int ldx, uint8_t *hs,
                                           int ldh, float (&part)[RT], bool over, int wave, int lane)
{
    typedef typename TileType<BF>::E E;
    typedef E frag __attribute__((ext_vector_type(16 / sizeof(E))));
    typedef E e4 __attribute__((ext_vector_type(4)));
    constexpr int D = BF ? 4 : 2;
    const int r16 = lane & 15, kq = lane >> 4;
    const uint8_t *xb = xs + r16 * ldx + kq * 16;
    // `over`: hs takes xs's place, which every wave has read by the barrier
    // (one round; a wave without tiles computes the last one for nothing)
    for (int g0 = wave * OT; g0 < NT || over; g0 += NW * OT) {
        const uint8_t *wt[OT];
#pragma unroll
        for (int t = 0; t < OT; ++t) wt[t] = W + (size_t)min(g0 + t, NT - 1) * KB * 1024 + lane * 16;
        floatx4 acc[OT][RT];
#pragma unroll
        for (int t = 0; t < OT; ++t)
#pragma unroll
            for (int r = 0; r < RT; ++r) acc[t][r] = floatx4{0.f, 0.f, 0.f, 0.f};
        frag w[D][OT];
        auto load = [&](frag (&x)[OT], int k) {   // past the last block: the last again
            const int off = min(k, KB - 1) * 1024;
#pragma unroll
            for (int t = 0; t < OT; ++t) x[t] = *(const frag *)(wt[t] + off);
        };
        auto mma = [&](const frag (&x)[OT], int k) {
            frag v[RT];
#pragma unroll
            for (int r = 0; r < RT; ++r) v[r] = *(const frag *)(xb + r * 16 * ldx + k * 64);
            if constexpr (BF) {
#pragma unroll
                for (int r = 0; r < RT; ++r)
#pragma unroll
                    for (int t = 0; t < OT; ++t)
                        acc[t][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[t], v[r], acc[t][r], 0,
                                                                            0, 0);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int r = 0; r < RT; ++r)
#pragma unroll
                        for (int t = 0; t < OT; ++t)
                            acc[t][r] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[t][e], v[r][e],
                                                                             acc[t][r], 0, 0, 0);
            }
        };
#pragma unroll
        for (int d = 0; d < D; ++d) load(w[d], d);
        int k = 0;
        for (; k + D <= KB; k += D)
#pragma unroll
            for (int d = 0; d < D; ++d) {
                mma(w[d], k + d);
                load(w[d], k + d + D);
                __builtin_amdgcn_sched_barrier(0);   // the refill stays here
            }
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (k + d < KB) mma(w[d], k + d);
        if (over) __syncthreads();
#pragma unroll
        for (int t = 0; t < OT; ++t) {
            if (g0 + t >= NT) break;
            const int o = (g0 + t) * 16 + kq * 4;
            const floatx4 bv = *(const floatx4 *)(bias + o);
            floatx4 wv;
            if (LAST) wv = *(const floatx4 *)(w3 + o);
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                e4 h;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float z = acc[t][r][e] + bv[e];
                    h[e] = (E)(BF ? tanh_for_bf16<true>(z) : tanh_f32<true>(z));
                }
                // past the layer's outputs zeros, not what zero weights give
                // (NaN where an input is infinite); widths are multiples of 4
                if (o >= H) h = e4{};
                if (LAST) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) part[r] = fmaf(wv[e], (float)h[e], part[r]);
                } else {
                    *(e4 *)(hs + (r * 16 + r16) * ldh + o * (int)sizeof(E)) = h;
                }
            }
        }
        if (over) break;
    }
}

// tiles a wave takes at a time: the fewest tile slots over its rounds
__device__ __forceinline__ int tiles_per_wave(int NT, int NW)
{
    int best = 4, cost = 1 << 30;
    for (int ot = 4; ot >= 1; --ot) {
        const int c = (NT + NW * ot - 1) / (NW * ot) * ot;
        if (c < cost) {
            cost = c;
            best = ot;
        }
    }
    return best;
}

template <bool BF, int RT, int NW>
__global__ __launch_bounds__(NW *WAVE) void critic_tile_kernel(CriticArgs A, int ldx, int ldh,
                                                                 int over)
{
    typedef typename TileType<BF>::E E;
    constexpr int BM = 16 * RT, NTH = NW * WAVE, VE = 16 / (int)sizeof(E);
    extern __shared__ __align__(16) uint8_t smem[];
    const CriticLayout &P = A.lay;
    // rows and hidden rows (byte pitches); with `over` these in the place of those
    uint8_t *xs = smem, *hs = over ? xs : xs + BM * ldx;
    float *vred = (float *)(over ? xs + BM * max(ldx, ldh) : hs + BM * ldh);   // [NW][BM]
    const int tid = threadIdx.x, lane = tid % WAVE;
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    const RowBlock rb = row_block(A, BM);
    const uint8_t *pk = A.packed + (size_t)rb.agent * P.agent_stride;

    // observation rows into LDS, zeros from column S on
    const int pieces = P.K_pad / VE, S = P.S;
    for (int i = tid; i < BM * pieces; i += NTH) {
        const int r = i / pieces, c = i % pieces;
        typedef E pv __attribute__((ext_vector_type(16 / sizeof(E))));
        pv v = *(const pv *)((const E *)A.obs + (size_t)rb.at(min(r, rb.nrow - 1)) * A.ld_obs + c * VE);
        if (c * VE + VE > S)
#pragma unroll
            for (int e = 0; e < VE; ++e)
                if (c * VE + e >= S) v[e] = (E)0.f;
        *(pv *)(xs + r * ldx + c * 16) = v;
    }
    __syncthreads();
    const float *b1 = (const float *)(pk + P.off_b[0]), *b2 = (const float *)(pk + P.off_b[1]);
    const float *w3 = (const float *)(pk + P.off_W[2]);
    float part[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) part[r] = 0.f;
    auto layer = [&](auto last, int l, const float *b, const uint8_t *x, int ld) {
        constexpr bool LAST = decltype(last)::value;
        const uint8_t *W = pk + P.off_W[l];
        const int H = l == 0 ? P.H1 : P.H2, NT = P.NT[l], KB = P.KS[l];
        switch (tiles_per_wave(NT, NW)) {
        case 1: tile_layer<BF, RT, NW, 1, LAST>(W, b, w3, H, NT, KB, x, ld, hs, ldh, part, !LAST && over, wave, lane); break;
        case 2: tile_layer<BF, RT, NW, 2, LAST>(W, b, w3, H, NT, KB, x, ld, hs, ldh, part, !LAST && over, wave, lane); break;
        case 3: tile_layer<BF, RT, NW, 3, LAST>(W, b, w3, H, NT, KB, x, ld, hs, ldh, part, !LAST && over, wave, lane); break;
        default: tile_layer<BF, RT, NW, 4, LAST>(W, b, w3, H, NT, KB, x, ld, hs, ldh, part, !LAST && over, wave, lane); break;
        }
    };
    layer(std::false_type{}, 0, b1, xs, ldx);
    __syncthreads();
    layer(std::true_type{}, 1, b2, hs, ldh);
#pragma unroll
    for (int r = 0; r < RT; ++r) {
        part[r] += __shfl_xor(part[r], 16);
        part[r] += __shfl_xor(part[r], 32);
    }
    if (lane < 16)
#pragma unroll
        for (int r = 0; r < RT; ++r) vred[wave * BM + r * 16 + lane] = part[r];
    __syncthreads();
    if (tid < rb.nrow) {
        float v = *(const float *)(pk + P.off_b[2]);
#pragma unroll
        for (int w = 0; w < NW; ++w) v += vred[w * BM + tid];
        A.value[rb.at(tid)] = v;
    }
}

template <class K>
hipError_t launch_with_lds(K k, size_t nblk, int threads, size_t lds, const CriticArgs &a,
                           hipStream_t s)
{
    if (lds > LDS_LIMIT) return hipErrorInvalidConfiguration;
    if (nblk > 0x7fffffffULL) return hipErrorInvalidConfiguration;
    hipError_t e = hipFuncSetAttribute((const void *)k,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((unsigned)nblk), dim3(threads), lds, s, a);
    return hipGetLastError();
}

template <bool BF, int RT, int NW>
hipError_t launch_tile_cfg(const CriticArgs &a, int ldx, int ldh, int over, size_t lds, hipStream_t s)
{
    const int64_t R = a.T * a.envs_per_agent, nblk = (R + 16 * RT - 1) / (16 * RT) * a.n_agents;
    if (lds > LDS_LIMIT || nblk > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    auto k = critic_tile_kernel<BF, RT, NW>;
    const hipError_t e = hipFuncSetAttribute((const void *)k,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((unsigned)nblk), dim3(NW * WAVE), lds, s, a, ldx, ldh, over);
    return hipGetLastError();
}

template <bool BF>
hipError_t launch_tile(const CriticArgs &a, hipStream_t s)
{
    const CriticLayout &L = a.lay;
    const int esz = BF ? 2 : 4;
    // 16 bytes past whole k-blocks: rows 4 banks apart
    const int ldx = L.K_pad * esz + 16, ldh = L.KS[1] * 64 + 16;
    constexpr int NW = TILE_NW;
    const int over = L.NT[0] <= 4 * NW;
    auto lds = [&](int rt) {
        return (size_t)16 * rt * ((over ? (ldx > ldh ? ldx : ldh) : ldx + ldh) + NW * 4);
    };
    const auto blocks = [&](int rt) {
        return (a.T * a.envs_per_agent + 16 * rt - 1) / (16 * rt) * a.n_agents;
    };
    // the largest row tile with three workgroups' LDS on a CU (fragments are
    // used RT times) that still leaves two workgroups for every CU
    for (int rt : {4, 2}) {
        if (lds(rt) > LDS_LIMIT / 3 || blocks(rt) < 512) continue;
        if (rt == 4) return launch_tile_cfg<BF, 4, NW>(a, ldx, ldh, over, lds(rt), s);
        return launch_tile_cfg<BF, 2, NW>(a, ldx, ldh, over, lds(rt), s);
    }
    return launch_tile_cfg<BF, 1, NW>(a, ldx, ldh, over, lds(1), s);
}

}  // namespace

bool critic_mfma_shape(const CriticLayout &L)
{
    return L.dtype == TP_BF16 && L.H1 == L.H2 && (L.H1 == 512 || L.H1 == 1024) &&
           L.K_pad == 1024;
}

hipError_t launch_critic_value(const CriticArgs &a, hipStream_t s)
{
    const CriticLayout &L = a.lay;
    if (L.mfma) {
        constexpr int NW = CRITIC_NW;
        const int OT = L.H1 / (16 * NW), RT = CRITIC_ACC_TILES / OT, BM = 16 * RT;
        const size_t nblk = ((size_t)a.T * a.envs_per_agent + BM - 1) / BM * a.n_agents;
        const size_t xb = 2 * (size_t)BM * (128 + 8) * 2, hb = (size_t)BM * (L.H1 + 8) * 2;
        const size_t lds = (xb > hb ? xb : hb) + NW * (size_t)BM * 4;
        constexpr int T512 = 512 / (16 * NW), T1024 = 1024 / (16 * NW);
        if (L.H1 == 512)
            return launch_with_lds(critic_mfma_kernel<NW, T512, CRITIC_ACC_TILES / T512, 32>,
                                   nblk, NW * WAVE, lds, a, s);
        return launch_with_lds(critic_mfma_kernel<NW, T1024, CRITIC_ACC_TILES / T1024, 32>, nblk,
                               NW * WAVE, lds, a, s);
    }
    if (L.dtype == TP_BF16) return launch_tile<true>(a, s);
    return launch_tile<false>(a, s);
}

}  // namespace tpk
